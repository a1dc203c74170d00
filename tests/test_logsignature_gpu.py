"""GPU parity of `sig_log`, `sig_lyndon_gather` and `sig_logsignature` with the fp64 oracle
(paper sections 2.3, 4.3, appendix A.2).

The logarithm adds and subtracts products of the signature's levels, which largely cancel, so its
rounding error is measured against the size of the terms summed: per level k,
||got_k - want_k|| <= tol * sum_m (1/m) sum_{k_1+..+k_m = k} ||Sig_{k_1}|| ... ||Sig_{k_m}||
(the power series of section 2.3 with every level replaced by its norm).
"""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from oracle import sig_oracle as orc
from paper_2001_00706_amd.inputs import WORKLOADS, brownian_paths, uniform_paths, workload_paths

pytestmark = pytest.mark.gpu

TOL = {np.float32: 1e-4, np.float64: 1e-10}


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


def term_scale(sig_ref, d, N):
    """Per level, the sum of the norms of the terms of the power series of the logarithm."""
    n = np.array([0.0] + [np.linalg.norm(sig_ref[..., sl]) for sl in orc.level_slices(d, N)])
    total, power = np.zeros(N + 1), np.zeros(N + 1)
    power[0] = 1.0
    for m in range(1, N + 1):
        power = np.convolve(power, n)[:N + 1]
        total += power / m
    return total[1:]


def assert_log_close(got, want, sig_ref, d, N, dt):
    got = np.asarray(got, dtype=np.float64)
    for sl, scale in zip(orc.level_slices(d, N), term_scale(sig_ref, d, N)):
        err = np.linalg.norm(got[..., sl] - want[..., sl])
        assert err <= TOL[dt] * (scale if scale > 0 else 1.0), (err, scale)


SHAPES = [(3, 9, 2, 6), (2, 6, 3, 5), (4, 12, 4, 4), (2, 5, 4, 6), (2, 4, 7, 3), (3, 5, 1, 4), (2, 6, 5, 1),
          (1, 20, 2, 8), (2, 5, 8, 4), (2, 7, 2, 9), (1, 5, 3, 9), (1, 6, 2, 10)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,L,d,N", SHAPES)
def test_log_of_signatures(B, L, d, N, dtype):
    x = brownian_paths(B, L, d, seed=L * d + N).astype(dtype)
    s = orc.signature(x, N)
    got = host(sig.sig_log(dev(s.astype(dtype)), d, N))
    assert_log_close(got, orc.tensor_log(s.astype(dtype), d, N), s, d, N, dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,L,d,N", SHAPES)
def test_logsignature_words_and_expand(B, L, d, N, dtype):
    x = uniform_paths(B, L, d, seed=3 * L + d, lo=-0.5, hi=0.5).astype(dtype)
    idx = orc.lyndon_indices(d, N)
    for stream, basepoint in [(False, False), (True, True)]:
        s = orc.signature(x, N, stream, basepoint)
        full = orc.tensor_log(s, d, N)
        got_full = host(sig.sig_logsignature(dev(x), N, stream=stream, basepoint=basepoint, mode="expand"))
        assert_log_close(got_full, full, s, d, N, dtype)
        got = host(sig.sig_logsignature(dev(x), N, stream=stream, basepoint=basepoint))
        assert got.shape[-1] == sig.sig_logsignature_channels(d, N) == len(idx)
        # the gather itself is exact
        np.testing.assert_array_equal(got, got_full[..., idx])


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["float32", "float64"])
def test_benchmark_shape_every_row(dtype):
    """1024 signatures of d = 4, N = 6 (the shape `bench.py --op logsignature` times): the logarithm of every row and
    the whole logsignature pipeline on every path, against the oracle."""
    w = WORKLOADS[1]
    x = workload_paths(w).astype(dtype)
    s = orc.signature(x, w.N)
    want = orc.tensor_log(s.astype(dtype), w.d, w.N)
    got = host(sig.sig_log(dev(s.astype(dtype)), w.d, w.N))
    assert_log_close(got, want, s, w.d, w.N, dtype)
    # row by row as well: a row computed from another row's data would pass a batch-wide norm only by luck
    for r in range(0, w.B, 37):
        assert_log_close(got[r:r + 1], want[r:r + 1], s[r:r + 1], w.d, w.N, dtype)
    idx = orc.lyndon_indices(w.d, w.N)
    words = host(sig.sig_logsignature(dev(x), w.N))
    full = orc.tensor_log(s, w.d, w.N)
    scale = term_scale(s, w.d, w.N)
    pos = 0
    for k, sl in enumerate(orc.level_slices(w.d, w.N)):
        cols = [i for i, off in enumerate(idx) if sl.start <= off < sl.stop]
        err = np.linalg.norm(words[:, cols] - full[:, [idx[i] for i in cols]])
        assert err <= TOL[dtype] * scale[k], (k + 1, err, scale[k])
        pos += len(cols)
    assert pos == len(idx) == words.shape[1]


def test_inverted_logsignature_is_minus_the_logsignature():
    # log(g^{-1}) = -log(g) (section 2.3 defines the inverted logsignature as log(Sig^{-1}))
    x = dev(brownian_paths(3, 10, 3, seed=2).astype(np.float64))
    a = host(sig.sig_logsignature(x, 4, inverse=True))
    b = host(sig.sig_logsignature(x, 4))
    np.testing.assert_allclose(a, -b, rtol=1e-9, atol=1e-12)


def test_many_rows_and_a_large_state():
    # 300 stream rows; and d = 8, N = 5 (37 448 scalars per row, several passes over 32 768-word levels)
    x = brownian_paths(2, 151, 3, seed=8)
    s = orc.signature(x, 4, stream=True)
    got = host(sig.sig_log(dev(s.astype(np.float32)), 3, 4))
    assert_log_close(got, orc.tensor_log(s.astype(np.float32), 3, 4), s, 3, 4, np.float32)
    y = brownian_paths(2, 9, 8, seed=9)
    s = orc.signature(y, 5)
    got = host(sig.sig_log(dev(s.astype(np.float32)), 8, 5))
    assert_log_close(got, orc.tensor_log(s.astype(np.float32), 8, 5), s, 8, 5, np.float32)


def test_log_refuses_to_work_in_place_and_empty_batches_are_fine():
    import torch
    s = torch.zeros((2, 6), device="cuda:0")
    with pytest.raises(ValueError):
        sig.sig_log(s, 2, 2, out=s)
    lib = sig.load_library()
    assert lib.sig_log(s.data_ptr(), 2, 2, 2, sig.SIG_F32, s.data_ptr(), 0) == sig.SIG_ERR_INVALID_ARG
    e = torch.zeros((0, 6), device="cuda:0")
    assert sig.sig_log(e, 2, 2).shape == (0, 6)
    assert sig.sig_lyndon_gather(e, 2, 2).shape == (0, 3)


# the kernels for a shape known at compile time, in LDS (d = 2, 3, 4, 8) and, too deep or too large for them, the one that
# forms a word by itself, with and without a compiled-in channel count; beyond depth 9 all words and a gather; one row and
# a number of words that is no multiple of a workgroup's
@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("rows,d,N", [(1, 2, 2), (130, 3, 6), (3, 4, 6), (2, 8, 4), (2, 4, 7), (5, 5, 5), (1, 7, 4), (3, 9, 2),
                                      (2, 12, 3), (3, 2, 9), (2, 2, 10), (4, 6, 1), (3, 1, 4)])
def test_kept_words_are_those_of_the_whole_logarithm(rows, d, N, dtype):
    s = dev(orc.signature(uniform_paths(rows, 6, d, seed=rows + d + N, lo=-0.5, hi=0.5), N).astype(dtype))
    got = sig.sig_log_words(s, d, N)
    np.testing.assert_array_equal(host(got), host(sig.sig_log(s, d, N))[..., orc.lyndon_indices(d, N)])
    assert sig.sig_log_words(s[:0], d, N).shape == (0, got.shape[-1])


def test_logsignature_gradient_in_one_node():
    """The gradient of the operation as a whole equals that of its parts in sequence, with an inverse and a basepoint tensor."""
    import torch
    for d, N, stream, inverse, mode in [(3, 4, False, False, "words"), (5, 3, True, True, "words"), (2, 5, False, True, "expand")]:
        x = dev(uniform_paths(3, 7, d, seed=d, lo=-0.5, hi=0.5)).requires_grad_(True)
        b = dev(uniform_paths(3, 1, d, seed=d + 1, lo=-0.5, hi=0.5)[:, 0]).requires_grad_(True)
        out = sig.logsignature(x, N, stream=stream, basepoint=b, inverse=inverse, mode=mode)
        parts = sig.signature_to_logsignature(sig.signature(x, N, stream=stream, basepoint=b, inverse=inverse), d, N, mode=mode)
        assert torch.equal(out, parts)
        w = torch.randn_like(out)
        for got, want in zip(torch.autograd.grad(out, (x, b), w), torch.autograd.grad(parts, (x, b), w)):
            assert torch.equal(got, want)
