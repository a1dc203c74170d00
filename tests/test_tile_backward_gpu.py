"""The gradient kernels that take sixteen increments at a time (sig_tile_backward_impl.h), where they can go wrong: paths that end inside
a tile or a span of tiles, channel counts that leave rows and letters of a block without a word, blocks that a workgroup takes
one after the other, stretches that do not begin at the start of their path.

Against the oracle's gradient.  An operand of a product is cut into pieces exactly and of the products of pieces at most 1.5 2^-23 of a term is left
out, so a sum of d terms is about as exact as in fp32; what adds up over a path are the roundings of the walk, some 2^-24 sqrt(increments) of the
largest term per level.  The bar of 1e-5 on the whole gradient is ten times what that gives at 300 increments (1e-6)."""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from oracle import sig_oracle as orc
from paper_2001_00706_amd.inputs import brownian_paths

pytestmark = pytest.mark.gpu

TOL = 1e-5


def gradient(x, g, N, basepoint=None, misalign=False):
    """(gradient of the points, of the basepoint)"""
    import torch
    xt, gt = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (x, g))
    bt = torch.from_numpy(basepoint).to("cuda:0") if isinstance(basepoint, np.ndarray) else bool(basepoint)
    if misalign:
        holder = torch.empty(gt.numel() + 1, dtype=gt.dtype, device=gt.device)
        holder[1:].copy_(gt.reshape(-1))
        gt = holder[1:].view(gt.shape)
    st = sig.sig_signature(xt, N, basepoint=bt)
    gp = torch.full_like(xt, float("nan"))
    gb = torch.full_like(bt, float("nan")) if isinstance(basepoint, np.ndarray) else None
    sig.sig_backward(xt, st, gt, N, basepoint=bt, grad_path=gp, **({"grad_basepoint": gb} if gb is not None else {}))
    torch.cuda.synchronize()
    return gp.cpu().numpy(), None if gb is None else gb.cpu().numpy()


def check(B, L, d, N, basepoint="none", sample=None, misalign=False, rounds=1):
    assert sig.sig_tile_rounds(B, L, d, N, basepoint=basepoint != "none", gradient=True) == rounds
    x = brownian_paths(B, L, d, seed=L + d) + np.float32(0.25)
    g = np.random.default_rng(B + L + d).standard_normal((B, orc.channels(d, N))).astype(np.float32)
    some = np.arange(B) if sample is None else np.asarray(sample)
    bp = {"none": None, "origin": True, "point": brownian_paths(B, 2, d, seed=7)[:, 1]}[basepoint]
    got, gb = gradient(x, g, N, bp, misalign)
    assert np.all(np.isfinite(got)), "gradient not fully written"
    xs = x[some].astype(np.float64)
    if basepoint == "point":
        want = orc.signature_backward(np.concatenate([bp[some][:, None].astype(np.float64), xs], axis=1), g[some], N)
        assert np.linalg.norm(gb[some] - want[:, 0]) <= TOL * np.linalg.norm(want)
        want = want[:, 1:]
    else:
        want = orc.signature_backward(xs, g[some], N, False, basepoint == "origin")
    diff = got[some] - want
    assert np.linalg.norm(diff) <= TOL * np.linalg.norm(want)
    single = np.linalg.norm(diff.reshape(len(some), -1), axis=1) / np.linalg.norm(want.reshape(len(some), -1), axis=1)
    assert single.max() <= 4 * TOL, single.max()


# 24 increments, whole tiles, one more and one less, spans of 64 and 128 and their neighbours
@pytest.mark.parametrize("L", [25, 33, 34, 64, 65, 66, 128, 129, 130, 257])
@pytest.mark.parametrize("d,N", [(4, 5), (7, 4), (11, 4)])
def test_lengths(L, d, N):
    check(3, L, d, N)


@pytest.mark.parametrize("basepoint", ["none", "origin", "point"])
@pytest.mark.parametrize("d,N", [(3, 4), (3, 6), (3, 8), (4, 4), (4, 6), (4, 7), (5, 4), (5, 6), (6, 4), (6, 5), (7, 5), (8, 4), (8, 5)]
                         + [(d, 4) for d in range(9, 17)] + [(9, 5), (12, 5)])
def test_channels_and_depths(d, N, basepoint):
    check(2, 41, d, N, basepoint)


@pytest.mark.parametrize("d,N", [(5, 7), (7, 6), (6, 7), (4, 8), (9, 6), (16, 5)])   # signatures of 30 000 scalars and more
def test_large_signatures(d, N):
    check(1, 40, d, N, "point")


# several blocks to a wavefront, one after the other (one round in twenty without any at most), for every number of last letters a block has; a single path
@pytest.mark.parametrize("B,L,d,N,rounds", [(600, 60, 4, 6, 2), (400, 129, 4, 7, 4), (64, 129, 4, 8, 2), (32, 128, 7, 7, 5), (64, 129, 7, 6, 2),
                                            (300, 129, 8, 5, 2), (300, 33, 9, 5, 7), (1, 700, 4, 4, 1), (1, 300, 13, 4, 1)])
def test_rounds_and_long_paths(B, L, d, N, rounds):
    check(B, L, d, N, sample=[0, B // 2, B - 1], rounds=rounds)


@pytest.mark.parametrize("d,N", [(4, 4), (6, 4), (10, 4)])
def test_unaligned_gradient(d, N):
    check(3, 50, d, N, misalign=True)


@pytest.mark.parametrize("d,N,chunks", [(9, 4, 3), (12, 4, 2), (16, 4, 4), (10, 5, 2)])
def test_stretches_are_walked_from_the_signature_they_are_handed(d, N, chunks):
    """From nine channels on the stretches of a path are rows of these kernels (of 8 increments, too few for them, and of 40)."""
    import torch
    for m in (8, 40):
        x = brownian_paths(2, m * chunks - 3, d, seed=m)
        g = np.random.default_rng(m).standard_normal((2, orc.channels(d, N))).astype(np.float32)
        xt, gt = (torch.from_numpy(a).to("cuda:0") for a in (x, g))
        got = sig.sig_backward_chunked(xt, gt, N, chunks).cpu().numpy()
        want = orc.signature_backward(x.astype(np.float64), g, N)
        assert np.linalg.norm(got - want) <= TOL * np.linalg.norm(want)


@pytest.mark.parametrize("d,N", [(4, 5), (8, 4), (12, 4)])
def test_infinite_gradient_stays_in_its_channels(d, N):
    """A word's gradient reaches the channels of its letters only, also where it is not a number."""
    B, L = 2, 40
    x = brownian_paths(B, L, d, seed=3)
    g = np.random.default_rng(3).standard_normal((B, orc.channels(d, N))).astype(np.float32)
    clean, _ = gradient(x, g, N)
    g[0, orc.channels(d, N) - 1] = np.inf      # the word of N times the last letter
    got, _ = gradient(x, g, N)
    assert not np.isfinite(got[0, :, d - 1]).any()
    np.testing.assert_array_equal(got[0, :, :d - 1], clean[0, :, :d - 1])
    np.testing.assert_array_equal(got[1], clean[1])


@pytest.mark.parametrize("B,L,d,N", [(40, 129, 5, 6), (32, 128, 7, 7), (20, 101, 7, 6), (8, 65, 9, 5)])
def test_gradient_is_as_exact_whatever_made_the_signature(B, L, d, N):
    """Without a word on where the signature comes from: one of the prefix tree, of stretches, or of a batch in parts, gives a gradient as exact as
    that of the scan's own, within what one seed differs from another (the roundings of another signature, walked back as they are, are off by 1.2 to
    1.45 times as much at these shapes); with it, the same bits."""
    import torch
    x = torch.from_numpy(brownian_paths(B, L, d, seed=1)).to("cuda:0")
    own = sig.sig_signature(x, N)
    g = torch.from_numpy(np.random.default_rng(1).standard_normal(tuple(own.shape)).astype(np.float32)).to("cuda:0")
    assert sig.sig_tile_rounds(B, L, d, N) == 1 and sig.sig_tile_rounds(B, L, d, N, gradient=True) >= 1
    want = sig.sig_backward(x.double(), sig.sig_signature(x.double(), N), g.double(), N)
    of = lambda s: float((sig.sig_backward(x, s, g, N).double() - want).norm() / want.norm())
    assert torch.equal(sig.sig_backward(x, own, g, N), sig.sig_backward(x, own, g, N, scanned=True))
    own_error = of(own)
    parts = torch.cat([sig.sig_signature(x[i:i + 3].contiguous(), N) for i in range(0, B, 3)])
    for other in (sig.sig_forward(x, N, variant=sig.SIG_VARIANT_TREE), sig.sig_forward_chunked(x, N, 16), parts):
        assert of(other) <= 1.1 * own_error
