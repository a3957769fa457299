"""k_matrix with X in digits (6-bit floats, one exponent for 32 entries of a row), which calls large enough take: every number
of planes, tiles that go back to bf16 planes beside tiles that do not, remainders of rows, entries and columns, K slices and
slabs, against float64 products."""
import numpy as np
import pytest

import paper_2510_06957_amd as tg

pytestmark = pytest.mark.gpu

# Calls that take digits, on each tile, K whole and sliced (tests/test_host_api_digits.py has the list); rows one more than a tile and
# parts of one, K at a block's edge, inside one and odd, columns of a part of a tile
SHAPES = [(1025, 4161, 17950), (4097, 2047, 9000), (1471, 16380, 4100), (777, 16380, 5900), (1300, 16380, 3600), (2049, 8129, 4500)]


def problem(M, K, N, seed, values, density=0.5):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.rand((K, N), generator=g, device="cuda")
    W = (u < density / 2).to(torch.int8) - ((u >= density / 2) & (u < density)).to(torch.int8)
    if values == "normal":
        X = torch.randn((M, K), generator=g, device="cuda")
    elif values == "uniform":
        X = torch.rand((M, K), generator=g, device="cuda") * 2 - 1
    elif values == "int":
        X = torch.randint(-100, 101, (M, K), generator=g, device="cuda").float()
    else:   # bf16: activations that come out of a 16-bit layer
        X = torch.randn((M, K), generator=g, device="cuda").bfloat16().float()
    b = torch.randint(-8, 9, (N,), generator=g, device="cuda").float()
    t = tg.tcsc_upload(tg.tcsc_build(W.cpu().numpy()), forms=tg.FORM_ROWSETS)
    assert N == 64 or tg.tstgemm_query_digits(t, M, workspace(M, K, N).numel())
    return W.double(), X, b, t


def workspace(M, K, N):
    import torch
    return torch.empty(tg.tstgemm_workspace_bytes(M, K, N)[1], dtype=torch.uint8, device="cuda")


# Bound on the error: the sums of the upper digits and of the lower are rounded once per 64 rows of W (in bf16 planes twice per
# 16), so it does not depend on how large one entry is beside another; measured at 3e-8 of sum |X W|.
TIGHT = 1e-6


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("values", ["normal", "uniform", "int", "bf16"])
def test_planes(M, K, N, values):
    W, X, b, t = problem(M, K, N, 900 + M, values)
    Y = tg.tstgemm(X, t, b, workspace=workspace(M, K, N)).double()
    E = X.double() @ W + b.double()
    if values == "int":
        assert (Y == E).all()
    else:
        A = X.double().abs() @ W.abs() + b.double().abs()
        assert ((Y - E).abs() <= TIGHT * A).all()
        assert (Y - E).norm() <= 1e-7 * E.norm()


def test_every_entry_alone():
    """One entry of W in a column: an output is an entry of X, exactly."""
    import torch
    M, K = 4800, 4160
    perm = np.random.default_rng(910).permutation(K)
    W = np.zeros((K, K), np.int8)
    W[perm, np.arange(K)] = 1
    t = tg.tcsc_upload(tg.tcsc_build(W), forms=tg.FORM_ROWSETS)
    g = torch.Generator(device="cuda").manual_seed(911)
    ws = workspace(M, K, K)
    assert tg.tstgemm_query_digits(t, M, ws.numel())
    for values in ("powers", "normal", "full"):
        if values == "powers":
            # +-2^e, and a third of them one less in the last place.  Seven planes hold multiples of 2^(E - 33), E the exponent of
            # the largest entry (0 here): an entry of exponent e has multiples of 2^(e - 23), so all is held from e = -10 on,
            # which is what one less than 2^-9 has
            e = torch.randint(-9, 1, (M, K), generator=g, device="cuda").float()
            X = torch.exp2(e) * torch.where(torch.rand((M, K), generator=g, device="cuda") < 0.5, -1.0, 1.0)
            X[:, ::3] = torch.nextafter(X[:, ::3], torch.zeros_like(X[:, ::3]))
            X[:, ::32] = 1.0
        elif values == "normal":
            X = torch.randn((M, K), generator=g, device="cuda")
        else:                      # all 24 bits set at random, large scale
            X = (torch.randint(2**23, 2**24, (M, K), generator=g, device="cuda") * 2.0**40).float()
        Y = tg.tstgemm(X, t, None, workspace=ws)
        want = X[:, torch.from_numpy(perm).cuda()]
        assert torch.equal(Y, want)


@pytest.mark.parametrize("values", ["feature 1e8", "feature 1e10", "feature 1e12", "feature 1.7e18", "feature 1e30", "one 1e12", "one 1e30",
                                    "floor", "few -20", "few -25", "few -30", "few -40", "block"])
def test_entries_beside_larger_ones(values):
    """Large entries of X, mostly under zero weights, beside ordinary ones: no output loses a bit of the small entries to them, so
    the bound of ordinary X holds for every output."""
    import torch
    M, K, N = 2300, 4161, 8200
    W, X, b, t = problem(M, K, N, 960, "normal", 1 / 16)
    g = torch.Generator(device="cuda").manual_seed(961)
    kind, size = (values + " 0").split()[:2]
    if kind == "feature":            # one column of X: a number, a time, a mark
        X[:, 100] = float(size)
    elif kind == "one":
        X[5, 100] = float(size)
    elif kind == "floor":            # ones beside a floor of 1e-11
        X = torch.where(torch.rand((M, K), generator=g, device="cuda") < 0.5, torch.ones_like(X), torch.full_like(X, 1e-11))
    elif kind == "few":              # of 32 entries mostly zeros, one of 1.5, some in [1, 2) times 2^e
        u = torch.rand((M, K), generator=g, device="cuda")
        X = torch.where(u < 0.25, (1 + torch.rand((M, K), generator=g, device="cuda")) * 2.0 ** int(size), torch.zeros_like(X))
        X[:, ::32] = 1.5
    else:                            # whole numbers, every other 32 of them times 2^60: each block of 32 fits by itself
        X = torch.randint(-100, 101, (M, K), generator=g, device="cuda").float()
        X *= torch.exp2((torch.arange(K, device="cuda") // 32 % 2 * 60).float())
        W[torch.arange(K, device="cuda") // 32 % 2 == 1, : N // 2] = 0
        t = tg.tcsc_upload(tg.tcsc_build(W.to(torch.int8).cpu().numpy()), forms=tg.FORM_ROWSETS)
        assert tg.tstgemm_query_digits(t, M, workspace(M, K, N).numel())
    Y = tg.tstgemm(X, t, b, workspace=workspace(M, K, N)).double()
    E = X.double() @ W + b.double()
    A = X.double().abs() @ W.abs() + b.double().abs()
    assert ((Y - E).abs() <= TIGHT * A).all()


@pytest.mark.parametrize("M,K,N", [(1025, 4161, 17950), (777, 16380, 5900)])
def test_tiles_that_digits_do_not_hold(M, K, N):
    """Rows with entries too far apart, beyond the exponents' range, infinite or NaN: their tiles go back to bf16 planes (and
    from there, where a sum is not finite, to the sums of any X); the others keep their digits.  What no infinity or NaN
    reaches is right, what one reaches is not finite."""
    import torch
    W, X, b, t = problem(M, K, N, 920, "uniform")
    g = torch.Generator(device="cuda").manual_seed(921)
    X[70] *= torch.exp2(torch.randint(-60, 20, (K,), generator=g, device="cuda").float())
    X[3] *= 1e-36
    X[140] *= 1e33
    X[150, 100], X[150, K - 1], X[151, K - 1] = float("inf"), float("-inf"), float("nan")
    X[190, 0] = float("nan")
    Y = tg.tstgemm(X, t, b, workspace=workspace(M, K, N)).double()
    bad = ~torch.isfinite(X)
    E = X.double().masked_fill(bad, 0) @ W + b.double()
    A = X.double().abs().masked_fill(bad, 0) @ W.abs() + b.double().abs()
    reached = (bad.double() @ W.abs()) > 0
    assert torch.equal(~torch.isfinite(Y), reached) and reached.any()
    assert ((Y - E).abs() <= TIGHT * A)[~reached].all()


@pytest.mark.parametrize("M,K,N", [(4097, 2047, 9000), (1471, 16380, 4100), (777, 16380, 5900), (1300, 16380, 3600)])
def test_one_entry_gives_a_tile_up(M, K, N):
    """k_digits gives the rest of a run of units up where one is not held: every other tile of rows has one such entry, at the
    start of K, at its end and between, beside tiles that keep their digits; the workspace holds noise before."""
    import torch
    W, X, b, t = problem(M, K, N, 970, "uniform")
    blocks = (K + 63) // 64
    for i in range(0, (M + 63) // 64, 2):
        kb = (0, blocks - 1, blocks // 2, 7, 8, 9, blocks - 2, 3)[i // 2 % 8]
        k, m = min(64 * kb + 37, K - 1), min(64 * i + 5 * i % 64, M - 1)
        X[m, k] = 1.2345678e-15
    ws = workspace(M, K, N)
    ws.random_(0, 256)
    Y = tg.tstgemm(X, t, b, workspace=ws).double()
    E = X.double() @ W + b.double()
    A = X.double().abs() @ W.abs() + b.double().abs()
    assert ((Y - E).abs() <= TIGHT * A).all()
    assert torch.equal(Y, tg.tstgemm(X, t, b, workspace=ws).double())


def slab_workspace(M, K, slabs):
    """Bytes for X in digits in so many slabs, the last of them the shortest."""
    return int(-(-M // 64) * -(-K // 64) * 22529 / slabs * 1.06) // 256 * 256


# (more slabs than one, last slabs of fewer tiles, last tiles of fewer rows, K at a block's edge and inside)
SLABS = [(5000, 4100, 9100, 2), (4000, 4161, 17950, 3), (8090, 4160, 8100, 2)]


@pytest.mark.parametrize("M,K,N,slabs", SLABS)
def test_slabs_of_rows(M, K, N, slabs):
    """A workspace that holds only some of the tiles in digits: the same results as with room for all, to the bit, also where a tile
    of the first and one of the last slab go back to bf16 planes."""
    import torch
    W, X, b, t = problem(M, K, N, 930, "uniform")
    X[7, K // 2] = X[M - 1, K - 1] = 1.2345678e-15
    Y = tg.tstgemm(X, t, b, workspace=workspace(M, K, N))
    E = X.double() @ W + b.double()
    A = X.double().abs() @ W.abs() + b.double().abs()
    assert ((Y.double() - E).abs() <= TIGHT * A).all()
    size = slab_workspace(M, K, slabs)
    assert tg.tstgemm_query_digits(t, M, size) and size < -(-M // 64) * -(-K // 64) * 22529
    ws = torch.full((size + 256,), 77, dtype=torch.uint8, device="cuda")
    assert torch.equal(tg.tstgemm(X, t, b, workspace=ws[:size]), Y) and (ws[size:] == 77).all()
    # and down to the least that a call needs, which digits do without
    least = tg.tstgemm_workspace_bytes(M, K, N)[0]
    Z = tg.tstgemm(X, t, b, workspace=ws[:least])
    assert ((Z.double() - E).abs() <= TIGHT * A).all()


@pytest.mark.parametrize("M,K,N,slabs", [(5000, 4100, 9100, 1), (5000, 4100, 9100, 2), (4000, 4161, 17950, 3)])
def test_events_around_the_last_slab(M, K, N, slabs):
    """The pair of events of a call brackets the products of the last slab, without k_digits and the other slabs."""
    import torch
    W, X, b, t = problem(M, K, N, 980, "uniform")
    ws = torch.empty(slab_workspace(M, K, slabs), dtype=torch.uint8, device="cuda")
    assert tg.tstgemm_query_digits(t, M, ws.numel())
    pair, whole = ([torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(2))
    for e in pair:
        e.record()
    shares = []
    for _ in range(5):
        whole[0].record()
        Y = tg.tstgemm(X, t, b, workspace=ws, events=pair)
        whole[1].record()
        torch.cuda.synchronize()
        shares.append(pair[0].elapsed_time(pair[1]) / whole[0].elapsed_time(whole[1]))
    # (of the whole, k_digits is about a tenth)
    assert 0.6 / slabs < sorted(shares)[2] < (1.0, 0.65, 0.5)[slabs - 1], shares


@pytest.mark.parametrize("count", ["one", "column"])
def test_prelu_and_rows_behind_y(count):
    import torch
    M, K, N = 2300, 4161, 8200
    W, X, b, t = problem(M, K, N, 940, "int")
    alpha = torch.exp2(torch.randint(-3, 3, (1 if count == "one" else N,), device="cuda").float())
    out = torch.full((M + 2, N), float("nan"), device="cuda")
    Y = tg.tstgemm(X, t, b, Y=out[:M], alpha=alpha, workspace=workspace(M, K, N)).double()
    E = X.double() @ W + b.double()
    assert (Y == torch.where(E > 0, E, alpha.double() * E)).all()
    assert torch.isnan(out[M:]).all()


def test_under_graph_capture():
    """Recorded once and replayed on new X, with eager work in between: the number of planes follows the X of the replay."""
    import torch
    M, K, N = 4097, 2047, 9000
    W, X, b, t = problem(M, K, N, 950, "int")
    ws, Y = workspace(M, K, N), torch.empty((M, N), device="cuda")
    tg.tstgemm(X, t, b, Y, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tg.tstgemm(X, t, b, Y, workspace=ws)
    for seed, values in enumerate(("normal", "int", "uniform", "wide", "int")):
        _, Xs, _, _ = problem(M, K, 64, 951 + seed, "normal" if values == "wide" else values)
        if values == "wide":
            Xs[::64] *= torch.exp2(torch.arange(K, device="cuda") % 60 - 30.0)
        X.copy_(Xs)
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        E = X.double() @ W + b.double()
        A = X.double().abs() @ W.abs() + b.double().abs()
        assert ((Y.double() - E).abs() <= TIGHT * A).all(), values
