"""The autograd nodes in C++ against the Python functions that serve every other call, and what is handed back to these."""
import numpy as np
import pytest

import paper_2001_00706_amd as sig
from paper_2001_00706_amd import autograd
from paper_2001_00706_amd.inputs import brownian_paths

pytestmark = pytest.mark.gpu


def both(monkeypatch, call):
    """`call()` through the C++ nodes and through the Python functions; whether the former took it."""
    taken = []
    node = autograd._transform

    def spy(*args):
        out = node(*args)
        taken.append(out is not NotImplemented)
        return out

    monkeypatch.setattr(autograd, "_transform", spy)
    got = call()
    monkeypatch.setattr(autograd, "_transform", lambda *args: NotImplemented)
    want = call()
    monkeypatch.setattr(autograd, "_transform", node)
    return got, want, taken


def same(got, want):
    import torch
    assert len(got) == len(want)
    for g, w in zip(got, want):
        assert (g is None) == (w is None)
        if g is not None:
            assert g.dtype == w.dtype and g.shape == w.shape and g.stride() == w.stride() and torch.equal(g, w)


# (stretches forward and backward among them: 1 x 600 points)
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("op", ["signature", "words", "expand"])
@pytest.mark.parametrize("B,L,d,N,stream,basepoint,inverse", [
    (3, 20, 3, 4, False, "none", False), (3, 20, 3, 4, True, "zero", False), (2, 9, 5, 3, False, "point", True),
    (2, 9, 2, 5, True, "point", True), (1, 600, 4, 4, False, "none", False), (1, 600, 3, 3, False, "point", True),
    (4, 12, 17, 2, False, "none", False), (2, 1, 2, 3, False, "zero", False),
])
def test_the_same_as_the_python_functions(monkeypatch, B, L, d, N, stream, basepoint, inverse, op, dtype):
    import torch
    x = torch.from_numpy(brownian_paths(B, L, d, seed=L).astype(dtype)).to("cuda:0")
    bp = torch.from_numpy(brownian_paths(1, B + 1, d, seed=1)[0, 1:].astype(dtype)).to("cuda:0")

    def call():
        xt = x.clone().requires_grad_(True)
        bt = bp.clone().requires_grad_(True) if basepoint == "point" else basepoint == "zero"
        kw = dict(stream=stream, basepoint=bt, inverse=inverse)
        out = sig.signature(xt, N, **kw) if op == "signature" else sig.logsignature(xt, N, mode=op, **kw)
        w = torch.from_numpy(np.random.default_rng(3).standard_normal(tuple(out.shape)).astype(dtype)).to("cuda:0")
        grads = torch.autograd.grad(out, [xt] + ([bt] if basepoint == "point" else []), w)
        with torch.no_grad():
            plain = sig.signature(x, N, **dict(kw, basepoint=bp if basepoint == "point" else kw["basepoint"]))
        return [out.detach(), plain, *grads]

    sig.logsignature(x, N, basepoint=True)   # the table of the kept words
    got, want, taken = both(monkeypatch, call)
    assert taken == [True, True]
    same(got, want)


def test_views_of_paths_basepoints_and_gradients(monkeypatch):
    import torch
    x = torch.from_numpy(brownian_paths(6, 11, 4, seed=5)).to("cuda:0")

    def call():
        xt = x.clone().requires_grad_(True)
        bt = x[0, :4].clone().requires_grad_(True)   # [4, 4]
        one = sig.signature(xt.transpose(1, 2), 3)   # 4 points of 11 channels
        two = sig.signature(xt[::2, :, 1:], 3, basepoint=bt.t()[:3, 1:])
        grads = [one.detach()[:1].expand_as(one), two.detach().t().contiguous().t()]
        return [one.detach(), two.detach(), *torch.autograd.grad([one, two], [xt, bt], grads)]

    got, want, taken = both(monkeypatch, call)
    assert taken == [True, True]
    same(got, want)


def test_what_is_handed_back(monkeypatch):
    import torch
    x = torch.from_numpy(brownian_paths(2, 9, 3, seed=5)).to("cuda:0")
    refused = [lambda: sig.signature(x.cpu(), 3), lambda: sig.signature(x.half(), 3), lambda: sig.signature(x[0], 3), lambda: sig.signature(x, 0),
               lambda: sig.signature(x, 33), lambda: sig.signature(x[:, :1], 3), lambda: sig.signature(x, 3, basepoint=x[:1, 0]),
               lambda: sig.signature(x, 3, basepoint=x[:, 0].double()), lambda: sig.logsignature(x.cpu(), 3), lambda: sig.signature(None, 3),
               lambda: sig.logsignature(x, 3, mode="brackets")]
    for call in refused:
        kinds = []
        for node in (autograd._transform, lambda *args: NotImplemented):
            with monkeypatch.context() as m:
                m.setattr(autograd, "_transform", node)
                with pytest.raises(Exception) as info:
                    call()
            kinds.append((info.type, str(info.value)))
        assert kinds[0] == kinds[1]
    for call in (lambda: sig.signature(x, np.int64(3)), lambda: sig.signature(x, 3, stream=1), lambda: sig.signature(x, 3, basepoint=1),
                 lambda: sig.signature(x[:0], 3), lambda: sig.signature(torch.zeros(1, 4097, 2, device="cuda:0"), 2)):
        got, want, taken = both(monkeypatch, lambda: [call()])
        assert taken == [False]
        same(got, want)


def test_depths_that_are_no_python_int(monkeypatch):
    # the table of the kept words is looked up by depth, and an array has no hash
    import torch
    x = torch.from_numpy(brownian_paths(2, 9, 3, seed=5)).to("cuda:0")
    want = sig.logsignature(x, 4)
    for depth in (np.array(4), np.int64(4), torch.tensor(4), 4.0):
        got, again, taken = both(monkeypatch, lambda: [sig.logsignature(x, depth)])
        assert not any(taken)
        same(got, again)
        same(got, [want])


def test_depths_beyond_the_kept_words_alone_are_scanned_once(monkeypatch):
    # sig_log_words ends at depth 9: the node is not asked for what it would hand back with the signature already formed
    import torch
    x = torch.from_numpy(brownian_paths(2, 9, 2, seed=5)).to("cuda:0")
    for depth, asked in ((9, [True]), (10, []), (11, [])):
        sig.logsignature(x, depth)   # the table of the kept words
        got, want, taken = both(monkeypatch, lambda: [sig.logsignature(x, depth)])
        assert taken == asked
        same(got, want)


def test_engine_semantics():
    import torch
    x = torch.from_numpy(brownian_paths(2, 9, 3, seed=5)).to("cuda:0").requires_grad_(True)
    assert not sig.signature(x.detach(), 3).requires_grad
    with torch.no_grad():
        assert not sig.signature(x, 3).requires_grad
    out = sig.signature(x, 3)
    g = torch.ones_like(out)
    first = torch.autograd.grad(out, x, g, retain_graph=True)[0]
    assert torch.equal(first, torch.autograd.grad(out, x, g)[0])
    with pytest.raises(RuntimeError, match="second time"):
        torch.autograd.grad(out, x, g)
    # what is saved goes through the hooks, and is watched for changes in place
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(t.shape) or t.cpu(), lambda t: t.to("cuda:0")):
        hooked = sig.signature(x, 3)
    assert len(packed) == 2 and torch.equal(torch.autograd.grad(hooked, x, g)[0], first)
    changed = sig.signature(x, 3)
    with torch.no_grad():
        changed.mul_(2)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        torch.autograd.grad(changed, x, g)
    # a stream of its own
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        on_s = torch.autograd.grad(sig.signature(x, 3), x, g)[0]
    s.synchronize()
    assert torch.equal(on_s, first)


def test_threads_on_streams_of_their_own():
    import threading
    import torch
    paths = [torch.from_numpy(brownian_paths(3, 60 + 7 * i, 4, seed=i)).to("cuda:0") for i in range(4)]

    def call(path):
        x = path.clone().requires_grad_(True)
        out = sig.logsignature(x, 4)
        return out.detach(), torch.autograd.grad(out, x, torch.ones_like(out))[0]

    want = [call(p) for p in paths]
    torch.cuda.synchronize()
    failed = []

    def work(path, w):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                got = [call(path) for _ in range(30)]
                torch.cuda.current_stream().synchronize()
                for g in got:
                    same(g, w)
        except Exception as e:
            failed.append(e)

    threads = [threading.Thread(target=work, args=a) for a in zip(paths, want)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


def test_transforms_and_forward_gradients_as_before(monkeypatch):
    import torch
    x = torch.from_numpy(brownian_paths(2, 9, 3, seed=5)).to("cuda:0")
    assert autograd._transform(x.cpu(), 3, False, False, False, 0, None) is NotImplemented
    # under vmap the node hands the call back, and torch.autograd.Function says that it has no rule for it
    asked = []
    node = autograd._transform
    monkeypatch.setattr(autograd, "_transform", lambda *args: asked.append(node(*args)) or asked[-1])
    with pytest.raises(RuntimeError, match="vmap"):
        torch.func.vmap(lambda p: sig.signature(p.unsqueeze(0), 3))(x)
    assert asked == [NotImplemented]
    monkeypatch.setattr(autograd, "_transform", node)
    import torch.autograd.forward_ad as fw
    with fw.dual_level():
        dual = fw.make_dual(x.clone().requires_grad_(True), torch.ones_like(x))
        assert autograd._transform(dual, 3, False, False, False, 0, None) is NotImplemented


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("B,L,d,N", [(1, 4, 2, 3), (5, 9, 3, 4), (3, 6, 12, 2)])
def test_path_query_in_the_node(B, L, d, N, dtype):
    """The node's interval gives the bits of the Python function's, and leaves to it what is not plain."""
    import torch
    from paper_2001_00706_amd import binding
    from paper_2001_00706_amd.autograd import _interval
    x = torch.from_numpy(brownian_paths(B, L, d, seed=L)).to("cuda:0", getattr(torch, dtype))
    p = sig.Path(x, N)
    rows = p._sig[0]
    for start, end in ((1, 2), (1, L - 1), (L - 2, L - 1)):
        got = _interval(rows, start, end, d, N)
        assert got is not NotImplemented and torch.equal(got, binding.sig_interval(rows, start, end, d, N))
        assert torch.equal(p.signature(start, end), got)
    for args in ((rows, 0, 2, d, N), (rows, 2, 2, d, N), (rows, 1, L, d, N), (rows, 1, 2, d + 1, N), (rows, 1, 2, d, 0), (rows, 1, 2, d, 10 ** 30),
                 (rows.cpu(), 1, 2, d, N), (rows.transpose(0, 1), 1, 2, d, N), (rows.half(), 1, 2, d, N), (rows, True, 2, d, N), (rows, 1, 2, d)):
        assert _interval(*args) is NotImplemented
