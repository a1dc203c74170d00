"""The signature kernels that take sixteen increments at a time (sig_tile_forward_impl.h), where they can go wrong: paths that end inside a
tile or a span of tiles, channel counts that leave rows of a result without a word, a last workgroup with few wavefronts.

Against the oracle, level by level.  Operands are cut into pieces exactly and of the products of pieces at most 2^-21 of a term is left out, 2^-23 in the
mean; what adds up are the roundings of some n / 16 sums per entry, 2^-24 sqrt(n) of a level's largest terms.  5e-6 is ten times that for 300
increments, and is below what one lost increment of a path of 300 does to a level (1 / sqrt(300))."""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from oracle import sig_oracle as orc
from paper_2001_00706_amd.inputs import brownian_paths

pytestmark = pytest.mark.gpu

TOL = 5e-6


def check(B, L, d, N, basepoint="none", sample=None, misalign=False, tiles=1):
    """`misalign`: by four bytes, which leaves calls of 8 and 16 channels to the vector kernels."""
    import torch
    assert misalign or sig.sig_tile_rounds(B, L, d, N, basepoint=basepoint != "none") == tiles
    x = brownian_paths(B, L, d, seed=L + d) + np.float32(0.25)
    some = np.arange(B) if sample is None else np.asarray(sample)
    bp = {"none": None, "origin": True, "point": brownian_paths(B, 2, d, seed=7)[:, 1]}[basepoint]
    xt = torch.from_numpy(x).to("cuda:0")
    bt = torch.from_numpy(bp).to("cuda:0") if basepoint == "point" else bool(bp)
    out = torch.full((B * orc.channels(d, N) + 1,), float("nan"), device="cuda:0")[int(misalign):][:B * orc.channels(d, N)].view(B, -1)
    sig.sig_signature(xt, N, basepoint=bt, out=out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got)), "signature not fully written"
    xs = x[some].astype(np.float64)
    if basepoint == "point":
        xs = np.concatenate([bp[some][:, None].astype(np.float64), xs], axis=1)
    want = orc.signature(xs, N, False, basepoint == "origin")
    at = 0
    for k in range(1, N + 1):
        a, b = got[some, at:at + d ** k], want[:, at:at + d ** k]
        at += d ** k
        assert np.linalg.norm(a - b) <= TOL * np.linalg.norm(b), k


@pytest.mark.parametrize("L", [33, 34, 48, 49, 50, 64, 65, 66, 129, 300])
@pytest.mark.parametrize("d,N", [(5, 6), (7, 5), (9, 5)])
def test_lengths(L, d, N):
    check(3, L, d, N)


@pytest.mark.parametrize("basepoint", ["none", "origin", "point"])
@pytest.mark.parametrize("d,N", [(5, 6), (5, 7), (6, 6), (7, 5), (7, 6), (9, 5), (10, 5), (11, 5), (9, 6)])
def test_channels_and_depths(d, N, basepoint):
    check(2, 43, d, N, basepoint)


@pytest.mark.parametrize("B,L,d,N", [(40, 101, d, 4) for d in (9, 10, 11)] + [(90, 101, d, 4) for d in range(12, 16)]
                         + [(8, 40, d, 5) for d in range(12, 17)])   # enough wavefronts for twelve channels and more
def test_wide(B, L, d, N):
    check(B, L, d, N, "origin", sample=[0, 1, B - 1])


@pytest.mark.parametrize("d,N", [(5, 8), (6, 7), (7, 7), (8, 7), (12, 6)])
def test_large_signatures(d, N):
    check(1, 40, d, N, "point")


# eight and sixteen channels, whose matrix kernels want 16-byte alignment
@pytest.mark.parametrize("basepoint", ["none", "origin", "point"])
@pytest.mark.parametrize("B,L,d,N", [(2, 43, 8, 5), (2, 43, 8, 6), (3, 101, 8, 4), (90, 101, 16, 4)])
def test_unaligned(B, L, d, N, basepoint):
    check(B, L, d, N, basepoint, sample=[0, 1, B - 1], misalign=True)


# shapes beside those above that the matrix kernels of 8 and 16 channels and the prefix tree keep
@pytest.mark.parametrize("B,L,d,N,basepoint", [(2, 43, 8, 6, "none"), (2, 43, 8, 6, "origin"), (2, 43, 8, 6, "point"), (90, 101, 16, 4, "origin"),
                                               (1, 40, 6, 8, "point")])
def test_left_to_the_others(B, L, d, N, basepoint):
    check(B, L, d, N, basepoint, sample=[0, B - 1], tiles=0)


def test_a_point_that_is_not_a_number_stays_in_its_words():
    import torch
    x = torch.from_numpy(brownian_paths(1, 60, 7, seed=3)).to("cuda:0")
    x[0, 20, 6] = float("nan")
    s = sig.sig_signature(x, 5)[0].cpu().numpy()
    last = s[-7 ** 5:].reshape((7,) * 5)
    assert np.all(np.isfinite(last[:6, :6, :6, :6, :6])) and np.isnan(last[6, 0, 0, 0, 0]) and np.isnan(last[0, 0, 0, 0, 6])


@pytest.mark.parametrize("what", ["nan", "inf"])
@pytest.mark.parametrize("at", [0, 1, 30, 31, 32, 58, 59])
@pytest.mark.parametrize("d,N", [(7, 5), (5, 6), (9, 5)])
def test_what_is_finite(d, N, at, what):
    """The same scalars of signature and gradient are finite as in 64 bits (an infinite gradient may come out as NaN)."""
    import torch
    x = torch.from_numpy(brownian_paths(2, 60, d, seed=3)).to("cuda:0")
    x[0, at, 1] = float(what)
    s, want = sig.sig_signature(x, N), sig.sig_signature(x.double(), N)
    assert torch.equal(torch.isfinite(s), torch.isfinite(want))
    g = sig.sig_backward(x, s, torch.ones_like(s), N)
    assert torch.equal(torch.isfinite(g), torch.isfinite(sig.sig_backward(x.double(), want, torch.ones_like(want), N)))


# What overflows, is infinite or is no number: as one increment at a time.  The largest points make products of two increments overflow whose scalars
# are finite, an increment overflows between two finite points, sums overflow and infinities of both signs meet.
WILD = ["one channel", "far points", "largest", "inf", "last inf", "overflowing increment", "huge", "nan"]


def wild_path(kind, B, L, d):
    x = brownian_paths(B, L, d, seed=3)
    if kind == "one channel":
        x[1] = 1
        x[1, :, 0] = 1e20 * brownian_paths(1, L, 1, seed=3)[0, :, 0]
    elif kind == "far points":
        x[1, :, 0] *= 1e20
    elif kind == "largest":
        x[1, L // 2:, 1] = np.finfo(np.float32).max
    elif kind in ("inf", "nan"):
        x[1, L // 2, 1] = float(kind)
    elif kind == "last inf":
        x[1, -1, 1] = np.inf
    elif kind == "overflowing increment":
        x[1, :L // 2, 1], x[1, L // 2:, 1] = -3e38, 3e38
    elif kind == "huge":
        x[1] *= 1e9
    return x


def assert_wild_as(got, want):
    """Nothing that is finite, or infinite, one increment at a time is less than that (sums that come close to an overflow in another order may stay finite)."""
    assert not np.any(np.isfinite(want) & ~np.isfinite(got)) and not np.any(np.isnan(got) & ~np.isnan(want))
    infinite = np.isinf(got) & np.isinf(want)
    assert np.array_equal(got[infinite], want[infinite])


@pytest.mark.parametrize("kind", WILD)
@pytest.mark.parametrize("d,N", [(7, 5), (5, 6), (9, 5), (13, 4)])
def test_overflow_and_infinities_are_those_of_single_increments(d, N, kind):
    import torch
    B, L = 90 if d == 13 else 3, 100
    assert sig.sig_tile_rounds(B, L, d, N) == 1
    x = wild_path(kind, B, L, d)
    xt = torch.from_numpy(x).to("cuda:0")
    for basepoint in (False, True):
        got = sig.sig_forward(xt, N, basepoint=basepoint).cpu().numpy()
        want = sig.sig_forward(xt, N, basepoint=basepoint, variant=sig.SIG_VARIANT_TREE).cpu().numpy()
        assert_wild_as(got, want)
        for b in (0, B - 1):   # the other paths' results are not touched
            assert np.all(np.isfinite(got[b])) and np.linalg.norm(got[b] - want[b]) <= TOL * np.linalg.norm(want[b])
