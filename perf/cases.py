"""The work whose speed matters to a program that uses this library: Y = X W + b with a ternary W, through the Python
binding, over the range of shapes, densities and options the library is used with.

X and b are drawn uniform in [-1, 1) or standard normal, W as independent entries with P(+1) = P(-1) = density / 2
(the recipe of synth_inputs.py, drawn on the GPU here because the inputs are made many times).
"""
import math

import torch

import paper_2510_06957_amd as tg

LARGEST = 4096 * 8192 * 8192          # M * K * N of the largest listed case
LARGEST_MATRIX = 8192 * 8192          # K * N


def _case(name, M, K, N, density, dist, call="tstgemm", prelu="none", own_workspace=False):
    # call: the entry point; prelu: "none", "one" slope or one per "column"; own_workspace (M > 64): the program uploads
    # the row sets alone and brings the scratch memory itself (one buffer for many matrices) instead of the default upload
    return dict(name=name, M=M, K=K, N=N, density=density, dist=dist, call=call, prelu=prelu, own_workspace=own_workspace)


def listed():
    return [
        # one token through a feed-forward projection: the smallest M, the weights are read once
        _case("decode-1", 1, 4096, 11008, 0.5, "normal"),
        # a small batch of tokens through the same layer
        _case("decode-8", 8, 4096, 11008, 0.5, "normal"),
        # one token with the weights in five-entries-per-byte form, the entry point for finite X
        _case("decode-1-packed", 1, 4096, 11008, 0.5, "normal", call="packed"),
        # a few tokens through a layer with odd sizes and a fused activation: launch latency and remainders
        _case("decode-5-ragged", 5, 2053, 1531, 0.25, "normal", prelu="column"),
        # the smallest benchmark configuration: latency of a batched call
        _case("batch-64-tiny", 64, 512, 512, 0.5, "uniform"),
        # a batch in a serving loop that must not allocate
        _case("batch-32-noalloc", 32, 4096, 4096, 0.25, "normal", call="noalloc"),
        # the deepest shape of the paper's sweep over K (M = 64, N = 4096)
        _case("batch-64-deep", 64, 16384, 4096, 0.5, "uniform"),
        # a prompt of ordinary length, the library's headline configuration
        _case("prefill-256", 256, 4096, 4096, 0.5, "uniform"),
        # the same with few non-zeros
        _case("prefill-256-sparse", 256, 4096, 4096, 0.125, "normal"),
        # odd sizes, activation, the caller's own workspace
        _case("prefill-777-ragged", 777, 3001, 2999, 0.25, "normal", prelu="one", own_workspace=True),
        # the largest batch, dense and very sparse weights
        _case("batch-4096", 4096, 8192, 8192, 0.5, "uniform", own_workspace=True),
        _case("batch-4096-sparse", 4096, 8192, 8192, 0.0625, "uniform", own_workspace=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A shape of the same ranges: M from 1 to 4096, K and N from 512 to 16384, density 1/16 to 1/2."""
    M = _log_int(rng, 1, 4096)
    while True:
        K, N = _log_int(rng, 512, 16384), _log_int(rng, 512, 16384)
        if rng.random() < 0.5:        # half of the sizes are multiples of 64, as layer sizes are; the others fall anywhere
            K, N = K // 64 * 64, N // 64 * 64
        if K * N <= LARGEST_MATRIX and M * K * N <= LARGEST:
            break
    density = rng.choice([0.0625, 0.125, 0.25, 0.5])
    if density == 0.5 and M * K * N > LARGEST // 2:
        density = 0.25
    call = rng.choice(["tstgemm", "tstgemm", "packed" if M <= 8 else "noalloc"])
    prelu = rng.choice(["none", "none", "one", "column"]) if call == "tstgemm" else "none"
    return dict(M=M, K=K, N=N, density=density, dist=rng.choice(["uniform", "normal"]), call=call, prelu=prelu,
                own_workspace=call == "tstgemm" and M > 64 and rng.random() < 0.5)


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed * 1000003 + 17)
    M, K, N, d = case["M"], case["K"], case["N"], case["density"]
    u = torch.rand((K, N), generator=g, device="cuda")
    W = (u < d / 2).to(torch.int8) - ((u >= d / 2) & (u < d)).to(torch.int8)
    del u

    def dense(*shape):
        if case["dist"] == "normal":
            return torch.randn(shape, generator=g, device="cuda")
        return torch.rand(shape, generator=g, device="cuda") * 2 - 1

    X, b = dense(M, K), dense(N)
    alpha = None
    if case["prelu"] != "none":       # slopes of a trained PReLU lie around 0.25
        alpha = 0.1 + 0.3 * torch.rand(1 if case["prelu"] == "one" else N, generator=g, device="cuda")
    return W, X, b, alpha


def prepare(case, seed):
    W, X, b, alpha = _inputs(case, seed)
    M, K, N = case["M"], case["K"], case["N"]
    t = tg.tcsc_build(W.cpu().numpy())
    state = dict(call=case["call"], X=X, b=b, alpha=alpha, t=t, Y=None, ws=None)
    if case["own_workspace"]:
        tg.tcsc_upload(t, forms=tg.FORM_ROWSETS)
        state["ws"] = torch.empty(tg.tstgemm_workspace_bytes(M, K, N)[1], dtype=torch.uint8, device="cuda")
    else:
        tg.tcsc_upload(t)
    if case["call"] == "noalloc":
        state["Y"] = torch.empty((M, N), device="cuda")
    return state


def run(state):
    X, t, b = state["X"], state["t"], state["b"]
    if state["call"] == "packed":
        return tg.tstgemm_packed(X, t, b)
    if state["call"] == "noalloc":
        return tg.tstgemm_noalloc(X, t, b, state["Y"])
    if state["ws"] is not None:
        return tg.tstgemm(X, t, b, alpha=state["alpha"], workspace=state["ws"])
    return tg.tstgemm(X, t, b, alpha=state["alpha"])


def work(case):
    """Bytes: X, b and Y once, W once in the smaller of two bits per entry and two bytes per non-zero.  Operations: one
    add per non-zero and row of X, and one per output for the bias."""
    M, K, N = case["M"], case["K"], case["N"]
    nnz = case["density"] * K * N
    return {"bytes": 4 * (M * K + M * N + N) + min(K * N / 4, 2 * nnz), "flops": M * nnz + M * N}


def tolerance(case):
    # 32-bit sums of n = K * density signed terms, added one after the other: measured 1.1e-6 at n = 4096 and 4.1e-7 at
    # n = 512 (M = 4096; the largest difference 10 times that), 1e-7 where a sum is cut into many short ones
    rel = max(6e-7, 7e-8 * math.sqrt(case["K"] * case["density"]))
    return {"rel": rel, "max": 10 * rel}


def exact(case, seed):
    W, X, b, alpha = _inputs(case, seed)
    Y = X.double() @ W.double() + b.double()
    if alpha is not None:
        Y = torch.where(Y > 0, Y, alpha.double() * Y)
    return Y
