"""The work this library is used for, as cases to be timed: signatures and logsignatures of batches of paths, with and
without their gradients, in final and in stream mode, few long paths, double precision, and intervals of stored paths.

Paths are Brownian sample paths, `x_1 = 0`, increments `N(0, 1/L)` per channel; gradients of the loss with respect to an
output are standard normal.  All calls go through the package's torch entry points (`signature`, `logsignature`, `Path`)."""
import math

import numpy as np
import torch

import paper_2001_00706_amd as sig

DTYPES = {"float32": torch.float32, "float64": torch.float64}


def _case(name, op, B, L, d, N, dtype="float32", stream=False, basepoint="none", train=False, queries=0):
    """`op`: "signature", "logsignature" or "path"; `basepoint`: "none", "zero" (the origin) or "point" (one per path);
    `train`: the gradient with respect to the path (and to the basepoint points) as well; `queries`: intervals asked of
    a `Path`."""
    return {"name": name, "op": op, "B": B, "L": L, "d": d, "N": N, "dtype": dtype, "stream": stream,
            "basepoint": basepoint, "train": train, "queries": queries}


def listed():
    return [
        # one small request, as a service that computes features of one short series answers it: latency
        _case("tiny", "signature", 32, 16, 2, 4),
        # features of a large batch of ordinary series, the benchmark's default shape
        _case("batch_d4n6", "signature", 1024, 128, 4, 6),
        # training through the largest signature of the paper's benchmark grid (section 6.1: 32 paths of 128 points, d = N = 7)
        _case("train_d7n7", "signature", 32, 128, 7, 7, train=True),
        # training on many channels, the benchmark's largest shape
        _case("train_d16n4", "signature", 256, 1024, 16, 4, train=True),
        # every prefix signature of a batch (expanding windows), the benchmark's stream shape
        _case("stream_d4n5", "signature", 128, 256, 4, 5, stream=True),
        # a recurrent or convolutional layer reads every prefix signature and is trained through it; odd length
        _case("train_stream_d5n4", "signature", 64, 101, 5, 4, stream=True, basepoint="zero", train=True),
        # logsignature features of a batch: the dimension-reduced form most models are fed with; ragged sizes
        _case("log_d5n5", "logsignature", 500, 101, 5, 5, basepoint="point"),
        # training through the logsignature at a point of the paper's grid (32 paths of 128 points, N = 7)
        _case("train_log_d5n7", "logsignature", 32, 128, 5, 7, train=True),
        # a mini-batch of an ordinary logsignature model, trained
        _case("train_log_d6n4", "logsignature", 256, 100, 6, 4, basepoint="zero", train=True),
        # one long record (a day of ticks, an audio clip) trained through as a whole
        _case("train_long_d4n6", "signature", 1, 65537, 4, 6, train=True),
        # double precision, as used where gradients are checked or paths are nearly straight
        _case("train_f64_d4n5", "signature", 128, 128, 4, 5, dtype="float64", train=True),
        # an online service: prefix signatures of stored series, new points appended, intervals queried
        _case("path_d4n4", "path", 32, 401, 4, 4, queries=8),
    ]


def _fmas(d, N):
    return sum((N - i + 1) * d ** i for i in range(2, N + 1))


def _channels(d, N):
    return sum(d ** k for k in range(1, N + 1))


def _increments(case):
    return case["L"] - (case["basepoint"] == "none")


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the same kinds: batches of 1 to 2048 paths, 8 to 1100 points (a single path or two up to 60 000), 2 to 16
    channels, depths 2 to 8, the signature up to a million scalars."""
    while True:
        op = rng.choice(["signature"] * 5 + ["logsignature"] * 3 + ["path"])
        long = op == "signature" and rng.random() < 0.15
        stream = op == "signature" and not long and rng.random() < 0.35
        train = op != "path" and rng.random() < 0.55
        B = rng.randint(1, 2) if long else _log_uniform(rng, 8, 64) if op == "path" else _log_uniform(rng, 1, 2048)
        L = _log_uniform(rng, 2000, 60000) if long else _log_uniform(rng, 60, 600) if op == "path" \
            else _log_uniform(rng, 8, 1100)
        d = _log_uniform(rng, 2, 16)
        N = rng.randint(2, 8)
        case = _case("", op, B, L, d, N, dtype="float64" if rng.random() < 0.15 else "float32", stream=stream,
                     basepoint=rng.choice(["none", "zero", "point"]) if op != "path" else "none", train=train,
                     queries=rng.randint(2, 12) if op == "path" else 0)
        del case["name"]
        S = _channels(d, N)
        flops = 2 * _fmas(d, N) * B * _increments(case) * (2 if case["dtype"] == "float64" else 1)
        rows = B * _increments(case) if stream or op == "path" else B
        scalars = rows * S
        # within the listed cases' reach: arithmetic, size of the outputs, length of the chain of increments
        if S > 1_000_000 or flops > (4e9 if long else 9e9) or scalars > 40_000_000:
            continue
        if op == "path" and S > 5000:
            continue
        if case["dtype"] == "float64" and S > 100_000:
            continue
        if op == "logsignature" and B * S * N > 60_000_000:
            continue
        return case


def _lyndon(d, N):
    """Lyndon words of length 1..N over 0..d-1, ordered by length, then lexicographically, as flat offsets."""
    found = [[] for _ in range(N + 1)]
    word = [-1]
    while word:
        word[-1] += 1
        found[len(word)].append(tuple(word))
        m = len(word)
        while len(word) < N:
            word.append(word[len(word) - m])
        while word and word[-1] == d - 1:
            word.pop()
    offsets, base = [], 0
    for k in range(1, N + 1):
        for w in sorted(found[k]):
            at = 0
            for letter in w:
                at = at * d + letter
            offsets.append(base + at)
        base += d ** k
    return offsets


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device=gen.device, dtype=torch.float64).to(DTYPES[dtype])


def _output_shape(case):
    B, d, N = case["B"], case["d"], case["N"]
    width = sig.sig_logsignature_channels(d, N) if case["op"] == "logsignature" else _channels(d, N)
    return (B, _increments(case), width) if case["stream"] else (B, width)


def prepare(case, seed, device="cuda"):
    gen = torch.Generator(device=device).manual_seed(seed)
    B, L, d = case["B"], case["L"], case["d"]
    steps = torch.randn((B, L, d), generator=gen, device=device, dtype=torch.float64) / math.sqrt(L)
    steps[:, 0] = 0
    path = steps.cumsum(1).to(DTYPES[case["dtype"]])
    state = {"case": case, "path": path}
    if case["op"] == "path":
        cut = max(2, 3 * L // 4)
        state["first"], state["new"] = path[:, :cut].contiguous(), path[:, cut:].contiguous()
        rng = np.random.default_rng(seed)
        intervals = []
        for _ in range(case["queries"]):
            a, b = sorted(int(i) for i in rng.choice(L, 2, replace=False))
            intervals.append((a, b))
        state["intervals"] = intervals
    if case["basepoint"] == "point":
        state["basepoint"] = _normal(gen, (B, d), case["dtype"]) / math.sqrt(L)
    if case["train"]:
        state["grad_out"] = _normal(gen, _output_shape(case), case["dtype"])
        state["path"].requires_grad_(True)
        if "basepoint" in state:
            state["basepoint"].requires_grad_(True)
    return state


def run(state):
    case = state["case"]
    if case["op"] == "path":
        path = sig.Path(state["first"], case["N"])
        path.update(state["new"])
        return [path.signature(a, b) for a, b in state["intervals"]]
    basepoint = state.get("basepoint", case["basepoint"] == "zero")
    transform = sig.signature if case["op"] == "signature" else sig.logsignature
    out = transform(state["path"], case["N"], stream=case["stream"], basepoint=basepoint)
    if not case["train"]:
        return out
    wanted = [state["path"]] + ([state["basepoint"]] if "basepoint" in state else [])
    return [out.detach(), *torch.autograd.grad(out, wanted, state["grad_out"])]


def work(case):
    B, L, d, N, n = case["B"], case["L"], case["d"], case["N"], _increments(case)
    S, M = _channels(d, N), _fmas(d, N)
    size = 8 if case["dtype"] == "float64" else 4
    scalars, flops = B * L * d, 0
    # the fused multiply-exponentiate of every increment; depth 2 in closed form: one contraction over the increments
    forward = 2 * d * d + 5 * d if N == 2 and not case["stream"] else 2 * M + d * (2 * N - 1)
    backward = 2 * d * d + 5 * d if N == 2 and not case["stream"] else 7 * M + 5 * N * d - S
    if case["op"] == "path":
        cut = max(2, 3 * L // 4)
        # what the later queries read is written: the signature of every prefix, and one product per query
        scalars += B * (L - 1) * S + case["queries"] * 3 * B * S
        flops += B * (L - 1) * forward + 2 * B * (case["queries"] + L - cut) * sum((k - 1) * d ** k for k in range(2, N + 1))
        return {"bytes": scalars * size, "flops": flops}
    out = math.prod(_output_shape(case))
    scalars += out + (B * d if case["basepoint"] == "point" else 0)
    flops += B * n * forward
    if case["op"] == "logsignature":
        # Horner's rule for the logarithm: the last round only at the words that are kept
        rounds = sum((k - 1) * d ** k * 2 for m in range(2, N) for k in range(2, N - m + 2))
        kept = sum(2 * (k - 1) * d ** k / k for k in range(2, N + 1))
        rows = B * n if case["stream"] else B
        flops += rows * (rounds + kept) * (3 if case["train"] else 1)
    if case["train"]:
        scalars += out + B * L * d + (B * d if case["basepoint"] == "point" else 0)
        flops += B * n * backward
    return {"bytes": scalars * size, "flops": int(flops)}


def tolerance(case):
    """About four times the largest error against 64-bit arithmetic seen over the listed cases and draws of each kind; the
    largest difference, which is found among the smallest coefficients of the top level, likewise.  The logarithm and
    the product of a signature with an inverse cancel; a gradient walked back along tens of thousands of increments
    adds up their rounding."""
    if case["dtype"] == "float64":
        return {"rel": 2.5e-13, "max": 2e-11}
    if case["op"] == "logsignature":
        return {"rel": 1e-4, "max": 6e-2} if case["N"] > 6 else {"rel": 2e-5, "max": 4e-3}
    if case["train"] and case["L"] > 2000:
        return {"rel": 1e-4, "max": 2e-3}
    if case["op"] == "path":
        return {"rel": 5e-5, "max": 1e-3}
    if case["train"]:
        return {"rel": 2e-5, "max": 4e-4}
    return {"rel": 2.5e-6, "max": 1.5e-4}


# ---- the same in 64 bits, by definition: exponentials of the increments, products in the truncated tensor algebra ----

def _exp(z, N):
    levels = [z]
    for k in range(2, N + 1):
        levels.append((levels[-1].unsqueeze(-1) * z.unsqueeze(-2)).flatten(-2) / k)
    return levels


def _mul(a, b):
    out = []
    for k in range(len(a)):
        total = a[k] + b[k]
        for j in range(k):
            total = total + (a[j].unsqueeze(-1) * b[k - 1 - j].unsqueeze(-2)).flatten(-2)
        out.append(total)
    return out


def _log(x):
    """log(1 + x) by Horner's rule; a product of two elements without constant term starts at level 2."""
    N = len(x)
    r = [v / N for v in x]
    for m in range(N - 1, 0, -1):
        new = []
        for k in range(N):
            total = x[k] / m
            for j in range(k):
                total = total - (x[j].unsqueeze(-1) * r[k - 1 - j].unsqueeze(-2)).flatten(-2)
            new.append(total)
        r = new
    return r


def _signature64(points, N, stream):
    z = points[:, 1:] - points[:, :-1]
    if stream:
        rows, state = [], None
        for s in range(z.shape[1]):
            e = _exp(z[:, s], N)
            state = e if state is None else _mul(state, e)
            rows.append(torch.cat(state, -1))
        return torch.stack(rows, 1)
    parts = _exp(z, N)   # neighbours joined pairwise
    while parts[0].shape[1] > 1:
        pairs = parts[0].shape[1] // 2
        joined = _mul([v[:, 0:2 * pairs:2] for v in parts], [v[:, 1:2 * pairs:2] for v in parts])
        parts = [torch.cat([v, w[:, 2 * pairs:]], 1) for v, w in zip(joined, parts)]
    return torch.cat([v[:, 0] for v in parts], -1)


def _split(x, d, N):
    return list(x.split([d ** k for k in range(1, N + 1)], -1))


def exact(case, seed, device="cuda"):
    state = prepare(case, seed, device)
    B, d, N, n = case["B"], case["d"], case["N"], _increments(case)
    if case["op"] == "path":
        path = state["path"].double()
        return [_signature64(path[:, a:b + 1], N, False) for a, b in state["intervals"]]
    keep = torch.tensor(_lyndon(d, N), device=device) if case["op"] == "logsignature" else None
    at_a_time = max(1, int(2e8 / (n * _channels(d, N))))
    outs, grads, grads_bp = [], [], []
    for b in range(0, B, at_a_time):
        rows = slice(b, b + at_a_time)
        points = state["path"].detach()[rows].double().requires_grad_(case["train"])
        base, wanted = None, [points]
        if case["basepoint"] == "zero":
            base = torch.zeros_like(points[:, 0])
        elif case["basepoint"] == "point":
            base = state["basepoint"].detach()[rows].double().requires_grad_(case["train"])
            wanted.append(base)
        all_points = points if base is None else torch.cat([base.unsqueeze(1), points], 1)
        out = _signature64(all_points, N, case["stream"])
        if keep is not None:
            out = torch.cat(_log(_split(out, d, N)), -1)[..., keep]
        if case["train"]:
            found = torch.autograd.grad(out, wanted, state["grad_out"][rows].double())
            grads.append(found[0])
            grads_bp.extend(found[1:])
        outs.append(out.detach())
    if not case["train"]:
        return torch.cat(outs)
    return [torch.cat(outs), torch.cat(grads), *([torch.cat(grads_bp)] if grads_bp else [])]
