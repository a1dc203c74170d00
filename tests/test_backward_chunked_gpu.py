"""Parity of `sig_backward_chunked` (the gradient of few long paths, walked back stretch by stretch) with the CPU oracle's
gradient, through the C ABI."""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from oracle import sig_oracle as orc
from paper_2001_00706_amd import binding
from paper_2001_00706_amd.inputs import brownian_paths, uniform_paths

pytestmark = pytest.mark.gpu

TOL = {np.float32: 1e-4, np.float64: 1e-9}


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def chunked(x, g, N, chunks, basepoint=False, grad_basepoint=None):
    import torch
    xt = dev(x)
    gp = torch.full_like(xt, float("nan"))
    sig.sig_backward_chunked(xt, dev(g), N, chunks, basepoint=basepoint, grad_path=gp, grad_basepoint=grad_basepoint)
    torch.cuda.synchronize()
    return gp.cpu().numpy()


def check(x, N, chunks, basepoint=False, seed=0):
    dt = x.dtype.type
    B, L, d = x.shape
    S = orc.channels(d, N)
    g = np.random.default_rng(seed + L + 7 * d + N).standard_normal((B, S)).astype(dt)
    got = chunked(x, g, N, chunks, basepoint)
    assert np.all(np.isfinite(got)), "gradient not fully written"
    want = orc.signature_backward(x, g, N, False, basepoint)
    err = np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want)
    assert err <= TOL[dt], err
    per_path = np.linalg.norm((got - want).reshape(B, -1), axis=1) / np.linalg.norm(want.reshape(B, -1), axis=1)
    assert per_path.max() <= 5 * TOL[dt], per_path.max()


# the stretches land on different gradient kernels: the walk that forms its products by itself (d = 2..8, N = 3..9), as paths of their own
# the d = 16, N = 4 kernel, the one for many channels (d = 20) and the generic one (d = 3, N = 10)
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,L,d,N,chunks", [
    (2, 65, 3, 4, 4), (3, 64, 4, 4, 8), (1, 130, 2, 6, 16), (2, 41, 5, 3, 5), (1, 100, 4, 6, 7), (2, 50, 16, 4, 4),
    (1, 33, 20, 3, 3), (2, 30, 6, 5, 6), (1, 40, 3, 10, 4), (4, 20, 8, 3, 2), (1, 300, 4, 5, 32), (2, 19, 3, 3, 18),
    # depth 2 (a stretch is not a path of its own: the closed form of the depth-2 gradient must step aside) and depth 1
    (1, 64, 4, 2, 2), (2, 300, 32, 2, 16), (5, 9, 64, 2, 4), (33, 64, 16, 2, 7), (2, 100, 1, 2, 8), (3, 50, 48, 2, 5),
    (2, 40, 5, 1, 4), (1, 30, 1, 1, 3),
])
def test_stretches_walked_back_side_by_side(B, L, d, N, chunks, dtype):
    check(brownian_paths(B, L, d, seed=L + d).astype(dtype), N, chunks)


# the tree of products (depth 2, depth 10, d = 12 and 13): counts next to powers of two (a last node without a neighbour on one or several
# levels), the first counts whose rounds no longer fit the single launch at the top (8192 scalars of a path: 1365 | 1366 signatures at d = 2,
# N = 2, 146 | 147 at d = 7, 4 | 5 at d = 2, N = 10), levels moved as vectors (d = 4, 8, 12), as whole groups of siblings (d = 2, 3, 5, 6, 7) and word by
# word (d = 13).  From d = 2 to 8 at N = 3 and 4 the same counts on the walk that forms its products by itself.
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,L,d,N,chunks", [
    (2, 138, 3, 4, 137), (3, 70, 3, 4, 69), (2, 69, 3, 4, 68), (1, 35, 3, 4, 17), (1, 258, 2, 3, 257), (2, 66, 4, 4, 65),
    (2, 25, 4, 4, 24), (2, 26, 4, 4, 25), (2, 21, 7, 3, 20), (1, 22, 7, 3, 21), (1, 66, 13, 2, 33), (2, 24, 13, 3, 23), (1, 40, 12, 3, 13), (2, 35, 7, 3, 34), (1, 47, 7, 4, 23),
    (1, 1366, 2, 2, 1365), (1, 1367, 2, 2, 1366), (2, 684, 3, 2, 683), (2, 410, 4, 2, 409), (2, 411, 4, 2, 410), (1, 275, 5, 2, 274), (1, 197, 6, 2, 196),
    (2, 147, 7, 2, 146), (2, 148, 7, 2, 147), (3, 18, 7, 2, 17), (1, 115, 8, 2, 114), (2, 5, 2, 10, 4), (1, 12, 2, 10, 5), (1, 8, 3, 10, 7),
])
def test_tree_of_products(B, L, d, N, chunks, dtype):
    check(brownian_paths(B, L, d, seed=L + d).astype(dtype), N, chunks)


# Every kernel of the walk over stretches (d = 2..8 at N = 3..9), with the products from LDS and from memory, whole and short last
# stretches, against the walk in one piece (both within the same distance of the oracle); 2 paths of words that share a
# workgroup, or span several.
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("d", [2, 3, 4, 5, 6, 7, 8])
def test_stretches_of_every_shape(d, dtype):
    for N in range(3, 10):
        S = orc.channels(d, N)
        if S > 1_100_000:
            continue
        x = brownian_paths(2, 12, d, seed=d + N).astype(dtype)
        g = np.random.default_rng(N).standard_normal((2, S)).astype(dtype)
        whole = sig.sig_backward(dev(x), sig.sig_signature(dev(x), N), dev(g), N).cpu().numpy().astype(np.float64)
        for chunks in (2, 3, 11):
            got = chunked(x, g, N, chunks)
            assert np.linalg.norm(got - whole) <= 2 * TOL[dtype] * np.linalg.norm(whole), (N, chunks)


# counts around the lines where stretches are joined to nodes of 8: 16 and 17 with the products from LDS (d = 3, N = 4), 8 and 9 from
# memory (d = 5, N = 6), nodes of nodes (130 and 71), a last node of one stretch; many paths to a workgroup, with an origin in front
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,L,d,N,chunks,basepoint", [
    (5, 17, 3, 4, 16, False), (5, 18, 3, 4, 17, False), (3, 131, 3, 4, 130, False), (2, 9, 5, 6, 8, False), (2, 10, 5, 6, 9, False),
    (1, 72, 5, 6, 71, False), (37, 19, 2, 3, 5, True), (37, 18, 2, 3, 17, True), (3, 32, 8, 4, 9, True),
])
def test_nodes_of_stretches(B, L, d, N, chunks, basepoint, dtype):
    check(brownian_paths(B, L, d, seed=L).astype(dtype) + dtype(0.2 * basepoint), N, chunks, basepoint=basepoint)


# the workspace's layout: exactly the bytes asked for, what lies behind them stays as it was
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,L,d,N,chunks", [(2, 11, 3, 3, 4), (3, 131, 2, 4, 65), (2, 601, 4, 5, 600), (1, 72, 5, 6, 71), (3, 40, 8, 4, 9), (1, 30, 7, 5, 8),
                                            (2, 30, 9, 3, 4)])
def test_the_workspace_asked_for_is_all_that_is_used(B, L, d, N, chunks, dtype):
    import torch
    code = sig.SIG_F32 if dtype == np.float32 else sig.SIG_F64
    x = brownian_paths(B, L, d, seed=L).astype(dtype)
    g = np.random.default_rng(L).standard_normal((B, orc.channels(d, N))).astype(dtype)
    need = sig.sig_backward_chunked_workspace_bytes(B, L, d, N, False, chunks, code)
    room = torch.full((need + (1 << 20),), 91, dtype=torch.uint8, device="cuda:0")
    got = sig.sig_backward_chunked(dev(x), dev(g), N, chunks, workspace=room[:need])
    want = orc.signature_backward(x, g, N, False, False)
    assert np.linalg.norm(got.cpu().numpy() - want) <= TOL[dtype] * np.linalg.norm(want)
    assert bool((room[need:] == 91).all())


def test_a_path_with_nan_spoils_no_other():
    x = brownian_paths(40, 21, 3, seed=1).astype(np.float32)
    g = np.random.default_rng(2).standard_normal((40, orc.channels(3, 4))).astype(np.float32)
    want = chunked(x, g, 4, 4)
    x[7, 9] = np.nan
    got = chunked(x, g, 4, 4)
    assert np.isnan(got[7]).any() and np.array_equal(np.delete(got, 7, 0), np.delete(want, 7, 0))


def test_stretches_two_to_a_workgroup():
    # 111 paths in 7 stretches are 777 rows of d = 4, N = 6, an odd number (the kernel of that shape takes whole paths only:
    # test_gradient_on_both_sides_of_the_register_resident_kernels_lines)
    check(brownian_paths(111, 29, 4, seed=2).astype(np.float32), 6, 7)


# Many paths: products one after the other from 16 MB of signatures on where they do not fit the LDS (d = 12, N = 4: 22 620 scalars, d = 16, N = 4),
# from 4 MB on where they go word by word (d = 13, N = 3: 2379; d = 20, N = 3: 8420); one path fewer takes the tree.  (At d = 7 and 8 as many
# paths on the walk that forms its products by itself.)  The whole against the gradient in one piece (both within the same
# distance of the oracle), a few paths against the oracle.
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("d,N,line,chunks", [(7, 5, 16, 2), (7, 5, 16, 5), (13, 3, 4, 3), (20, 3, 4, 4), (8, 5, 16, 4), (12, 4, 16, 3), (16, 4, 16, 4)])
def test_products_in_chains(d, N, line, chunks, dtype):
    S = orc.channels(d, N)
    at = -(-(line << 20) // (S * np.dtype(dtype).itemsize))
    for B in (at, at - 1):
        x = brownian_paths(B, 11, d, seed=d).astype(dtype)
        g = np.random.default_rng(d).standard_normal((B, S)).astype(dtype)
        got = chunked(x, g, N, chunks)
        xt = dev(x)
        whole = sig.sig_backward(xt, sig.sig_signature(xt, N), dev(g), N).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - whole) <= 2 * TOL[dtype] * np.linalg.norm(whole)
        some = [0, B // 2, B - 1]
        want = orc.signature_backward(x[some], g[some], N, False, False)
        assert np.linalg.norm(got[some] - want) <= TOL[dtype] * np.linalg.norm(want)


def test_fastest_count():
    h = sig.sig_backward_chunks_fastest
    for B, L, d, N in ((1, 65537, 4, 6), (2, 4000, 6, 3), (32, 801, 8, 4)):
        chunks = h(B, L, d, N)
        assert chunks >= 4 and chunks & (chunks - 1) == 0 and (L - 1) // chunks >= 16
        assert sig.sig_backward_chunked_workspace_bytes(B, L, d, N, False, chunks) <= 2 << 30
    assert h(1024, 128, 4, 6) == 1 and h(1, 100000, 4, 2) == 1 and h(1, 100, 4, 4) == 1   # many, depth 2, short
    assert h(2, 1, 3, 4) == 0 and h(1, 100, 0, 4) == 0
    check(brownian_paths(2, 1500, 3, seed=4), 4, h(2, 1500, 3, 4))


@pytest.mark.parametrize("B,L,d,N,chunks", [(2, 64, 3, 4, 4), (1, 65, 4, 4, 8), (3, 30, 5, 3, 7), (2, 9, 2, 5, 9)])
def test_with_the_origin_as_basepoint(B, L, d, N, chunks):
    check(brownian_paths(B, L, d, seed=3).astype(np.float64) + 0.3, N, chunks, basepoint=True)
    check(brownian_paths(B, L, d, seed=4) + np.float32(0.3), N, chunks, basepoint=True)


def test_with_a_basepoint_value_and_its_gradient():
    import torch
    B, L, d, N = 3, 45, 3, 4
    x = brownian_paths(B, L, d, seed=5).astype(np.float64) + 0.1
    bp = uniform_paths(B, 1, d, seed=6)[:, 0].astype(np.float64)
    g = np.random.default_rng(1).standard_normal((B, orc.channels(d, N)))
    bt = dev(bp)
    gb = torch.full_like(bt, float("nan"))
    got = chunked(x, g, N, 6, basepoint=bt, grad_basepoint=gb)
    want = orc.signature_backward(np.concatenate([bp[:, None], x], axis=1), g, N)
    np.testing.assert_allclose(got, want[:, 1:], rtol=1e-9, atol=1e-11)
    np.testing.assert_allclose(gb.cpu().numpy(), want[:, 0], rtol=1e-9, atol=1e-11)


def test_more_stretches_than_increments_and_stretches_that_do_not_divide_the_path():
    # 10 increments: 4 stretches of 3, 3, 3, 1; 64 asked for: 10 stretches of one increment
    for chunks in (4, 64, 3, 2):
        check(brownian_paths(2, 11, 3, seed=chunks).astype(np.float64), 4, chunks)
    check(brownian_paths(1, 2, 4, seed=9).astype(np.float64), 3, 2)   # a single increment


def test_the_hinted_count_on_a_long_path():
    B, L, d, N = 1, 4097, 4, 4
    chunks = sig.sig_backward_chunks_hint(B, L, d, N)
    assert chunks > 1
    check(brownian_paths(B, L, d, seed=12), N, chunks)
    check(brownian_paths(B, L, d, seed=13).astype(np.float64), N, chunks)
    assert sig.sig_backward_chunks_hint(1024, 128, 4, 6) == 1 and sig.sig_backward_chunks_hint(1, 100000, 4, 2) == 1


@pytest.mark.parametrize("refused", [0, 1, 2])
def test_autograd_takes_the_stretches_for_a_long_path(monkeypatch, refused):
    """... as many as are fastest; where there is no memory for these, as few as the hint, and then none."""
    import torch
    B, L, d, N = 2, 4097, 3, 4
    fastest, hint = (h(B, L, d, N, False, sig.SIG_F64) for h in (sig.sig_backward_chunks_fastest, sig.sig_backward_chunks_hint))
    assert fastest > hint > 1
    asked, call = [], binding.sig_backward_chunked

    def sig_backward_chunked(path, grad_out, depth, chunks, **kw):
        asked.append(chunks)
        if len(asked) <= refused:
            raise torch.OutOfMemoryError("no memory")
        return call(path, grad_out, depth, chunks, **kw)

    monkeypatch.setattr(binding, "sig_backward_chunked", sig_backward_chunked)
    x = brownian_paths(B, L, d, seed=8).astype(np.float64)
    w = np.random.default_rng(9).standard_normal((B, orc.channels(d, N)))
    xt = dev(x).requires_grad_(True)
    (sig.signature(xt, N) * dev(w)).sum().backward()
    assert asked == [fastest, hint][:refused + 1]
    want = orc.signature_backward(x, w, N)
    np.testing.assert_allclose(xt.grad.cpu().numpy(), want, rtol=1e-8, atol=1e-10)


def test_same_result_twice_and_inputs_untouched():
    import torch
    x = dev(brownian_paths(2, 200, 4, seed=2))
    g = dev(np.random.default_rng(3).standard_normal((2, orc.channels(4, 5))).astype(np.float32))
    x0, g0 = x.clone(), g.clone()
    a = sig.sig_backward_chunked(x, g, 5, 8).clone()
    b = sig.sig_backward_chunked(x, g, 5, 8)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(x, x0) and torch.equal(g, g0)


def test_invalid_arguments_and_short_workspace():
    import torch
    x = dev(brownian_paths(2, 50, 3, seed=1))
    g = dev(np.zeros((2, orc.channels(3, 4)), dtype=np.float32))
    for chunks in (0, 1, 70000):
        with pytest.raises(sig.SigError):
            sig.sig_backward_chunked(x, g, 4, chunks)
        assert sig.sig_backward_chunked_workspace_bytes(2, 50, 3, 4, False, chunks) == -1
    need = sig.sig_backward_chunked_workspace_bytes(2, 50, 3, 4, False, 4)
    assert need > 0
    with pytest.raises(sig.SigError):
        sig.sig_backward_chunked(x, g, 4, 4, workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda:0"))
    assert sig.sig_backward_chunks_hint(2, 1, 3, 4) == 0
