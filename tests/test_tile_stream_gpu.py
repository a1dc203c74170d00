"""Stream mode with a lane per increment (sig_tile_stream.hip), where it can go wrong: paths that end inside or at the edge of sixty-four
increments, channel counts and depths with and without letters above a workgroup's words.

Against the oracle, level by level over all rows.  A scalar is a sum of n increments' terms by a tree over 64 lanes and a chain of n / 64, so it is
as exact as the one increment at a time of the other kernels: 2^-24 sqrt(n) of a level's terms per level, 5e-6 is ten times that at 300."""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from oracle import sig_oracle as orc
from paper_2001_00706_amd.inputs import brownian_paths
from tests.test_tile_forward_gpu import WILD, assert_wild_as, wild_path

pytestmark = pytest.mark.gpu

TOL = 5e-6


def check(B, L, d, N, basepoint="none"):
    import torch
    # (with fewer than 20 increments most lanes would have none: those calls, which the rule leaves to the other kernels, are here for its line)
    assert sig.sig_tile_rounds(B, L, d, N, stream=True, basepoint=basepoint != "none") == (L - (basepoint == "none") >= 20)
    x = brownian_paths(B, L, d, seed=L + d) + np.float32(0.25)
    bp = {"none": None, "origin": True, "point": brownian_paths(B, 2, d, seed=7)[:, 1]}[basepoint]
    xt = torch.from_numpy(x).to("cuda:0")
    bt = torch.from_numpy(bp).to("cuda:0") if basepoint == "point" else bool(bp)
    out = torch.full((B, L - (basepoint == "none"), orc.channels(d, N)), float("nan"), device="cuda:0")
    sig.sig_signature(xt, N, stream=True, basepoint=bt, out=out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got)), "rows not fully written"
    xs = x.astype(np.float64)
    if basepoint == "point":
        xs = np.concatenate([bp[:, None].astype(np.float64), xs], axis=1)
    want = orc.signature(xs, N, True, basepoint == "origin")
    at = 0
    for k in range(1, N + 1):
        a, b = got[..., at:at + d ** k], want[..., at:at + d ** k]
        at += d ** k
        assert np.linalg.norm(a - b) <= TOL * np.linalg.norm(b), k


@pytest.mark.parametrize("L", [2, 3, 16, 17, 18, 20, 21, 22, 33, 34, 64, 65, 66, 128, 129, 130, 300])
@pytest.mark.parametrize("d,N", [(4, 4), (5, 4), (3, 3)])
def test_lengths(L, d, N):
    check(2, L, d, N)


@pytest.mark.parametrize("basepoint", ["none", "origin", "point"])
@pytest.mark.parametrize("d,N", [(d, N) for d, most in ((2, 8), (3, 7), (4, 6), (5, 5), (6, 5), (7, 5)) for N in range(3, most + 1)])
def test_channels_and_depths(d, N, basepoint):
    check(2, 71, d, N, basepoint)


def test_a_point_that_is_not_a_number_stays_in_later_rows():
    import torch
    x = torch.from_numpy(brownian_paths(1, 130, 5, seed=3)).to("cuda:0")
    x[0, 70, 4] = float("nan")
    s = sig.sig_signature(x, 4, stream=True)[0].cpu().numpy()
    last = s[:, -5 ** 4:].reshape((-1,) + (5,) * 4)
    assert np.all(np.isfinite(s[:69])) and np.all(np.isfinite(last[:, :4, :4, :4, :4])) and np.all(np.isnan(last[69:, 4, 0, 0, 0]))


@pytest.mark.parametrize("d,N", [(2, 3), (2, 7), (3, 5), (4, 4), (5, 3), (5, 5), (7, 4)])
def test_begun_with_what_came_before(d, N):
    """The second half of a path on top of the first half's signature: the rows of the whole path."""
    import torch
    x = brownian_paths(3, 140, d, seed=d)
    xt = torch.from_numpy(x).to("cuda:0")
    first = sig.sig_signature(xt[:, :60].contiguous(), N)
    rows = sig.sig_signature(xt[:, 60:].contiguous(), N, stream=True, basepoint=xt[:, 59].contiguous(), initial=first)
    want = orc.signature(x.astype(np.float64), N, True)[:, 59:]
    at = 0
    for k in range(1, N + 1):
        a, b = rows[..., at:at + d ** k].cpu().numpy(), want[..., at:at + d ** k]
        at += d ** k
        assert np.linalg.norm(a - b) <= TOL * np.linalg.norm(b), k


@pytest.mark.parametrize("what", ["nan", "inf"])
@pytest.mark.parametrize("at", [0, 20, 63, 64, 65, 100, 129])
@pytest.mark.parametrize("d,N", [(4, 4), (5, 3), (2, 6)])
def test_what_is_finite(d, N, at, what):
    import torch
    x = torch.from_numpy(brownian_paths(2, 130, d, seed=3)).to("cuda:0")
    x[0, at, 1] = float(what)
    rows = sig.sig_signature(x, N, stream=True)
    assert torch.equal(torch.isfinite(rows), torch.isfinite(sig.sig_signature(x.double(), N, stream=True)))


# on both sides of the longest path that is taken, by the number of paths; longer ones go in chunks
@pytest.mark.parametrize("B,d,N,longest", [(1, 3, 4, 1000), (16, 2, 3, 2000), (65, 4, 3, 3000), (40, 3, 6, 1500), (130, 3, 5, 1059), (2, 6, 4, 1500)])
def test_long_streams(B, d, N, longest):
    import torch
    for L in (longest + 1, longest + 2):
        assert sig.sig_tile_rounds(B, L, d, N, stream=True) == (L == longest + 1)
        x = brownian_paths(B, L, d, seed=d)
        some = [0, 1, 63, 64, L // 2, L - 2]
        got = sig.sig_signature(torch.from_numpy(x).to("cuda:0"), N, stream=True)[:2, some].cpu().numpy()
        want = orc.signature(x[:2].astype(np.float64), N, True)[:, some]
        for sl in orc.level_slices(d, N):
            assert np.linalg.norm(got[..., sl] - want[..., sl]) <= TOL * (L / 300) ** 0.5 * np.linalg.norm(want[..., sl])


@pytest.mark.parametrize("kind", WILD)
@pytest.mark.parametrize("d,N", [(2, 5), (3, 4), (4, 5), (5, 4), (7, 3)])
def test_overflow_and_infinities_are_those_of_single_increments(d, N, kind):
    import torch
    B, L = 3, 120   # (streams of 128 increments and more are cut into chunks by the prefix-tree kernels)
    x = wild_path(kind, B, L, d)
    xt = torch.from_numpy(x).to("cuda:0")
    for basepoint in (False, True):
        assert sig.sig_tile_rounds(B, L, d, N, stream=True, basepoint=basepoint) == 1
        got = sig.sig_forward(xt, N, stream=True, basepoint=basepoint).cpu().numpy()
        want = sig.sig_forward(xt, N, stream=True, basepoint=basepoint, variant=sig.SIG_VARIANT_TREE).cpu().numpy()
        assert_wild_as(got, want)
        for b in (0, 2):
            assert np.all(np.isfinite(got[b])) and np.linalg.norm(got[b] - want[b]) <= TOL * np.linalg.norm(want[b])


@pytest.mark.parametrize("what", ["inf", "nan", "large"])
def test_what_came_before_is_not_finite(what):
    """`initial` with an infinity, a NaN or scalars that overflow in the products: as a product per row makes them."""
    import torch
    d, N, L = 4, 4, 100
    x = torch.from_numpy(np.abs(brownian_paths(2, L, d, seed=3)).cumsum(1)).to("cuda:0")
    before = sig.sig_forward(x, N)
    if what == "large":
        before[1] *= 3e38 / before[1].abs().max()
    else:
        before[1, 1] = float(what)
    assert sig.sig_tile_rounds(2, L, d, N, stream=True) == 1
    got = sig.sig_signature(x, N, stream=True, initial=before).cpu().numpy()
    rows = sig.sig_forward(x, N, stream=True)
    want = torch.stack([sig.sig_combine(before, rows[:, i].contiguous(), d, N) for i in range(L - 1)], 1).cpu().numpy()
    assert np.linalg.norm(got[0] - want[0]) <= TOL * np.linalg.norm(want[0])
    finite = np.isfinite(want[1])
    assert np.array_equal(np.isfinite(got[1]), finite) and np.array_equal(np.isnan(got[1]), np.isnan(want[1]))
