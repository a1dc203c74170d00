"""GPU parity of `sig_log_backward`, `sig_lyndon_scatter` and the differentiable `logsignature` with the fp64
oracle (paper sections 2.3, 4.3, 5.3).

The gradient of the logarithm is, like the logarithm, an alternating sum of products that largely cancel, so its
rounding error is measured against the size of the terms summed.  That size comes from the oracle too: at -|x|
with cotangent |g| every term of the series has the same sign, so the oracle's gradient there is, scalar by scalar,
the sum of the absolute values of the terms.
"""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from oracle import sig_oracle as orc
from paper_2001_00706_amd.inputs import WORKLOADS, brownian_paths, workload_paths

pytestmark = pytest.mark.gpu

TOL = {np.float32: 1e-5, np.float64: 1e-13}


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


def assert_grad_close(got, want, scale, d, N, dt):
    got = np.asarray(got, dtype=np.float64)
    for sl in orc.level_slices(d, N):
        err = np.linalg.norm(got[..., sl] - want[..., sl])
        bound = np.linalg.norm(scale[..., sl])
        assert err <= TOL[dt] * (bound if bound > 0 else 1.0), (err, bound)


# rows, d, N: matrices of at most 256 columns only (2^8, 3^5, 5^3, 9^2), wider ones (2^9, 4^5, 7^3, 8^3), a single
# letter, depths 1 and 2, and a channel count without a compiled-in divisor
SHAPES = [(3, 2, 9), (2, 2, 10), (5, 3, 6), (2, 4, 6), (3, 5, 4), (2, 7, 4), (4, 1, 5), (3, 6, 1), (3, 4, 2),
          (2, 8, 4), (3, 9, 3), (1, 3, 7), (7, 2, 3)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("rows,d,N", SHAPES)
def test_gradient_of_the_logarithm(rows, d, N, dtype):
    x = orc.signature(1.5 * brownian_paths(rows, 8, d, seed=rows + 10 * d + N), N).astype(dtype)
    g = np.random.default_rng(N * 100 + d).standard_normal(x.shape).astype(dtype)
    got = host(sig.sig_log_backward(dev(x), dev(g), d, N))
    want = orc.tensor_log_backward(x, g, d, N)
    scale = orc.tensor_log_backward(-np.abs(x.astype(np.float64)), np.abs(g.astype(np.float64)), d, N)
    assert_grad_close(got, want, scale, d, N, dtype)


def test_gradient_of_the_logarithm_of_arbitrary_elements_and_leading_dimensions():
    # not only signatures; leading dimensions are flattened into rows
    d, N = 3, 5
    S = orc.channels(d, N)
    rng = np.random.default_rng(1)
    x, g = 0.5 * rng.standard_normal((2, 3, S)), rng.standard_normal((2, 3, S))
    got = host(sig.sig_log_backward(dev(x), dev(g), d, N))
    scale = orc.tensor_log_backward(-np.abs(x), np.abs(g), d, N)
    assert got.shape == x.shape
    assert_grad_close(got, orc.tensor_log_backward(x, g, d, N), scale, d, N, np.float64)


def test_two_calls_give_identical_bits():
    d, N = 4, 6
    x = orc.signature(brownian_paths(6, 9, d, seed=2), N).astype(np.float32)
    g = np.random.default_rng(0).standard_normal(x.shape).astype(np.float32)
    a = host(sig.sig_log_backward(dev(x), dev(g), d, N))
    b = host(sig.sig_log_backward(dev(x), dev(g), d, N))
    assert np.array_equal(a, b)


def horner_r2(x, d, N, words, fma):
    """R_2 of log(1 + x) = x - x R_2 .. at the given words (rows of letters), by Horner's rule in the precision of `fma`."""
    K = words.shape[1]
    power = d ** np.arange(K, -1, -1)

    def at(i, j):   # x at letters i .. j - 1
        idx = words[:, i:j] @ power[K - (j - i) + 1:]
        return x[orc.level_slices(d, N)[j - i - 1].start + idx]

    r = {}   # R_m at the suffix from letter i on
    for m in range(N, 1, -1):
        new = {}
        for i in range(max(0, K - (N - m + 1)), K):
            acc = x.dtype.type((1 if m & 1 else -1) / x.dtype.type(m)) * at(i, K)
            for j in range(K - 1, i, -1):
                acc = fma(at(i, j), r[j], acc)
            new[i] = acc
        r = new
    return r[0]


# The gradient with respect to x[0] of the word 0 w alone, where w does not contain the letter 0, is R_2[w] and nothing else: the
# error of these factors of the gradient is no larger than that of Horner's rule step by step.  The same additions in the
# same order: 1.1 leaves room for a few sums fused the other way round; sums of powers instead are off by 1.2 to 1.8
# times as much.  A channel count with and without a compiled-in divisor.
@pytest.mark.parametrize("d,N", [(3, 8), (3, 9), (5, 6), (6, 5), (9, 4)])
def test_right_factors_are_as_accurate_as_horners_rule(d, N):
    x = orc.signature(brownian_paths(1, 100, d, seed=d + N), N).astype(np.float32)[0]
    words = np.stack(np.meshgrid(*[np.arange(1, d)] * (N - 1), indexing="ij"), -1).reshape(-1, N - 1)[:512]
    g = np.zeros((len(words), len(x)), dtype=np.float32)
    level = orc.level_slices(d, N)[N - 1].start
    g[np.arange(len(words)), level + words @ d ** np.arange(N - 2, -1, -1)] = 1
    assert sig.sig_log_backward_workspace_bytes(len(words), d, N, sig.SIG_F32) > 0   # the kernels that form the factors first
    got = host(sig.sig_log_backward(dev(np.tile(x, (len(words), 1))), dev(g), d, N))[:, 0]
    exact = horner_r2(x.astype(np.float64), d, N, words, lambda a, b, c: a * b + c)
    model = horner_r2(x, d, N, words, lambda a, b, c: (a.astype(np.float64) * b + c).astype(np.float32))
    assert model.dtype == np.float32
    assert np.linalg.norm(got - exact) <= 1.1 * np.linalg.norm(model - exact)


def test_scatter_is_the_transpose_of_gather():
    d, N = 3, 5
    idx = orc.lyndon_indices(d, N)
    g = np.random.default_rng(3).standard_normal((4, 2, len(idx)))
    got = host(sig.sig_lyndon_scatter(dev(g), d, N))
    want = np.zeros((4, 2, orc.channels(d, N)))
    want[..., idx] = g
    assert np.array_equal(got, want)


# a workgroup per row up to 8192 scalars (d = 2, N = 12 has 8190 and d = 90, N = 2 has 8190), two launches beyond (8372)
@pytest.mark.parametrize("rows,d,N", [(3, 2, 12), (2, 90, 2), (3, 91, 2), (1, 1, 3)])
def test_scatter_on_both_sides_of_the_row_limit(rows, d, N):
    import torch
    idx = orc.lyndon_indices(d, N)
    g = np.random.default_rng(5).standard_normal((rows, len(idx))).astype(np.float32)
    out = torch.full((rows, orc.channels(d, N)), 7.0, device="cuda:0")
    want = np.zeros(tuple(out.shape), dtype=np.float32)
    want[..., idx] = g
    assert np.array_equal(host(sig.sig_lyndon_scatter(dev(g), d, N, out=out)), want)


def test_workspace_is_checked():
    import torch
    d, N = 4, 7     # 21 844 scalars per signature: the chain of launches, which needs a workspace
    x = dev(orc.signature(brownian_paths(2, 5, d, seed=1), N))
    need = sig.sig_log_backward_workspace_bytes(2, d, N, sig.SIG_F64)
    assert need > 0
    short = torch.empty(need - 1, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(sig.SigError):
        sig.sig_log_backward(x, x.clone(), d, N, workspace=short)
    assert sig.sig_log_backward_workspace_bytes(2, d, 1, sig.SIG_F64) == 0
    assert sig.sig_log_backward_workspace_bytes(2, 2, 4, sig.SIG_F64) == 0      # single launch, everything in LDS


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["float32", "float64"])
def test_both_routes_agree_on_the_same_shape(dtype):
    # d = 3, N = 7 (3279 scalars): 8 signatures go through the single-launch kernel (no workspace), 300 through the
    # chain of launches (workspace); in fp64 the working set of a signature exceeds the LDS and both take the chain
    d, N = 3, 7
    code = sig.SIG_F32 if dtype == np.float32 else sig.SIG_F64
    assert sig.sig_log_backward_workspace_bytes(300, d, N, code) > 0
    assert (sig.sig_log_backward_workspace_bytes(8, d, N, code) == 0) == (dtype == np.float32)
    x = orc.signature(brownian_paths(300, 6, d, seed=12), N).astype(dtype)
    g = np.random.default_rng(4).standard_normal(x.shape).astype(dtype)
    many = host(sig.sig_log_backward(dev(x), dev(g), d, N))
    few = host(sig.sig_log_backward(dev(x[:8]), dev(g[:8]), d, N))
    want = orc.tensor_log_backward(x[:8], g[:8], d, N)
    scale = orc.tensor_log_backward(-np.abs(x[:8].astype(np.float64)), np.abs(g[:8].astype(np.float64)), d, N)
    assert_grad_close(few, want, scale, d, N, dtype)
    assert_grad_close(many[:8], want, scale, d, N, dtype)
    want = orc.tensor_log_backward(x, g, d, N)
    scale = orc.tensor_log_backward(-np.abs(x.astype(np.float64)), np.abs(g.astype(np.float64)), d, N)
    assert_grad_close(many, want, scale, d, N, dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("rows,d,N", [(5, 2, 2), (300, 2, 9), (3, 2, 10), (70, 4, 3), (9, 4, 6), (2, 8, 2), (40, 8, 3), (3, 8, 4)])
def test_power_of_two_channels_take_one_launch_at_any_batch_size(rows, d, N, dtype):
    # d = 2, 4, 8: the gather form of the single-launch kernel whenever a signature's working set fits the LDS (all of
    # these do, in both precisions: the largest, d = 4, N = 6 in fp64, takes 140 KB)
    code = sig.SIG_F32 if dtype == np.float32 else sig.SIG_F64
    assert sig.sig_log_backward_workspace_bytes(rows, d, N, code) == 0
    x = orc.signature(1.3 * brownian_paths(rows, 7, d, seed=rows + d + N), N).astype(dtype)
    g = np.random.default_rng(rows + N).standard_normal(x.shape).astype(dtype)
    got = host(sig.sig_log_backward(dev(x), dev(g), d, N))
    want = orc.tensor_log_backward(x, g, d, N)
    scale = orc.tensor_log_backward(-np.abs(x.astype(np.float64)), np.abs(g.astype(np.float64)), d, N)
    assert_grad_close(got, want, scale, d, N, dtype)
    for r in range(0, rows, 17):
        assert_grad_close(got[r:r + 1], want[r:r + 1], scale[r:r + 1], d, N, dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("rows", [1024, 256])
def test_benchmark_shape_every_row(rows, dtype):
    """d = 4, N = 6 at 1024 rows is what `bench.py --op logsignature_backward` times: one launch, with 61 KB of LDS per
    signature in fp32 and 140 KB in fp64.  Every row against the oracle, batch-wide and row by row."""
    w = WORKLOADS[1]
    code = sig.SIG_F32 if dtype == np.float32 else sig.SIG_F64
    need = sig.sig_log_backward_workspace_bytes(rows, w.d, w.N, code)
    assert need == 0
    x = orc.signature(workload_paths(w)[:rows], w.N).astype(dtype)
    g = np.random.default_rng(w.seed).standard_normal(x.shape).astype(dtype)
    got = host(sig.sig_log_backward(dev(x), dev(g), w.d, w.N))
    want = orc.tensor_log_backward(x, g, w.d, w.N)
    scale = orc.tensor_log_backward(-np.abs(x.astype(np.float64)), np.abs(g.astype(np.float64)), w.d, w.N)
    assert_grad_close(got, want, scale, w.d, w.N, dtype)
    for r in range(0, rows, 29):
        assert_grad_close(got[r:r + 1], want[r:r + 1], scale[r:r + 1], w.d, w.N, dtype)


def test_logsignature_gradient_on_the_benchmark_shape():
    """The whole gradient of the logsignature (scatter, logarithm, signature) with respect to the path on all 1024
    paths of d = 4, N = 6, L = 128, in fp32, against the oracle's."""
    import torch
    w = WORKLOADS[1]
    x = workload_paths(w)
    n_words = len(orc.lyndon_indices(w.d, w.N))
    g = np.random.default_rng(w.seed + 1).standard_normal((w.B, n_words)).astype(np.float32)
    p = dev(x).requires_grad_(True)
    sig.logsignature(p, w.N).backward(dev(g))
    got = host(p.grad).astype(np.float64)
    want = orc.logsignature_backward(x, g, w.N)
    err = np.linalg.norm((got - want).reshape(w.B, -1), axis=1)
    den = np.linalg.norm(want.reshape(w.B, -1), axis=1)
    assert np.linalg.norm(err) <= 1e-4 * np.linalg.norm(den), np.linalg.norm(err) / np.linalg.norm(den)
    assert np.max(err / den) <= 5e-4, np.max(err / den)


@pytest.mark.parametrize("stream", [False, True])
@pytest.mark.parametrize("B,L,d,N", [(3, 7, 2, 5), (2, 6, 3, 4), (2, 9, 4, 4)])
def test_logsignature_is_differentiable_in_the_path(B, L, d, N, stream):
    import torch
    x = brownian_paths(B, L, d, seed=L + N).astype(np.float64)
    n_inc = L - 1
    w = len(orc.lyndon_indices(d, N))
    g = np.random.default_rng(5).standard_normal((B, n_inc, w) if stream else (B, w))
    p = dev(x).requires_grad_(True)
    out = sig.logsignature(p, N, stream=stream)
    np.testing.assert_allclose(host(out.detach()), orc.logsignature(x, N, stream=stream), rtol=0, atol=1e-11)
    out.backward(dev(g))
    want = orc.logsignature_backward(x, g, N, stream=stream)
    np.testing.assert_allclose(host(p.grad), want, rtol=1e-9, atol=1e-10)


def test_gradcheck_through_the_logsignature_in_both_modes():
    import torch
    x = dev(brownian_paths(2, 5, 2, seed=9).astype(np.float64)).requires_grad_(True)
    assert torch.autograd.gradcheck(lambda p: sig.logsignature(p, 4), (x,), eps=1e-6, atol=1e-7, rtol=1e-6)
    assert torch.autograd.gradcheck(lambda p: sig.logsignature(p, 3, stream=True, mode="expand"), (x,), eps=1e-6,
                                    atol=1e-7, rtol=1e-6)
    s = dev(orc.signature(brownian_paths(2, 5, 2, seed=9), 3)).requires_grad_(True)
    assert torch.autograd.gradcheck(lambda t: sig.signature_to_logsignature(t, 2, 3), (s,), eps=1e-6, atol=1e-7,
                                    rtol=1e-6)


def test_threads_that_launch_one_kernel_with_different_lds():
    # the single-launch kernel takes 72 KB of LDS at d = N = 5 and 124 at d = 6, N = 5, where the runtime wants to be told beforehand
    import threading
    import torch
    calls = []
    for d in (5, 6):
        s, g = (torch.randn((3, orc.channels(d, 5)), generator=torch.Generator().manual_seed(d + i)).to("cuda:0") for i in (0, 1))
        calls.append((s, g, d, sig.sig_log_backward(s, g, d, 5)))
    torch.cuda.synchronize()
    failed = []

    def work(s, g, d, want):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                outs = [sig.sig_log_backward(s, g, d, 5) for _ in range(100)]
                torch.cuda.current_stream().synchronize()
                assert all(torch.equal(out, want) for out in outs)
        except Exception as e:
            failed.append(e)

    threads = [threading.Thread(target=work, args=c) for c in calls for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


# a workgroup per signature with everything in LDS: every depth of the odd channel counts that have such a kernel, and the last steps of
# signatures too large for it (their first steps go by the matrices); few and many rows
@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("rows,d,N", [(3, 3, 3), (300, 3, 4), (2, 3, 5), (3, 3, 6), (300, 3, 7), (3, 3, 8), (2, 3, 9), (300, 5, 3), (3, 5, 4), (300, 5, 5),
                                      (2, 5, 6), (2, 5, 7), (3, 6, 3), (300, 6, 4), (3, 6, 5), (2, 6, 6), (300, 7, 3), (3, 7, 4), (2, 7, 5),
                                      (2, 4, 7), (2, 4, 8), (2, 8, 5), (2, 8, 6)] + [(3, d, 3) for d in range(9, 17)] +
                         [(2, 9, 4), (300, 11, 4), (2, 16, 4), (2, 9, 5)])
def test_elements_in_lds(rows, d, N, dtype):
    x = orc.signature(1.3 * brownian_paths(rows, 7, d, seed=rows + d + N), N).astype(dtype)
    g = np.random.default_rng(rows + N).standard_normal(x.shape).astype(dtype)
    got = host(sig.sig_log_backward(dev(x), dev(g), d, N))
    some = np.arange(0, rows, 37)
    want = orc.tensor_log_backward(x[some], g[some], d, N)
    scale = orc.tensor_log_backward(-np.abs(x[some].astype(np.float64)), np.abs(g[some].astype(np.float64)), d, N)
    assert_grad_close(got[some], want, scale, d, N, dtype)


# more signatures than workgroups of 256 and of 512 threads, or two threads a scalar, make up a grid (less than 2^32 threads): all alike but for
# their first scalar
@pytest.mark.parametrize("rows,d,N", [((1 << 24) + 3, 3, 3), ((1 << 23) + 3, 9, 3), (160001, 4, 7)])
def test_more_signatures_than_a_grid_holds(rows, d, N):
    import torch
    S, some = orc.channels(d, N), torch.tensor([0, 1, 1 << 17, rows // 2, rows - 1])   # (all below the smallest count)
    s1, g1 = (torch.randn(S, generator=torch.Generator().manual_seed(i)).to("cuda:0") * 0.3 for i in (0, 1))
    s, g, out = (torch.empty((rows, S), device="cuda:0") for _ in range(3))
    s[:], g[:] = s1, g1
    s[:, 0] = (torch.arange(rows, device="cuda:0") % 1021) / 1021
    sig.sig_log_backward(s, g, d, N, out=out)
    want = sig.sig_log_backward(s[some].contiguous(), g[some].contiguous(), d, N)
    assert torch.equal(out[some], want)
    assert torch.equal(out[rows - 1021:], out[rows - 2042:rows - 1021])   # the rows that leave the same rest
