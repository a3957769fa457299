"""The matrix-core kernels (X cut into three bf16 planes) through the ordinary entry points: sizes at the edges of their
tiles and steps, X that their planes cannot hold, and the same calls through the list and row-set kernels, against the
oracle element by element."""
import numpy as np
import pytest

import oracle
import paper_2510_06957_amd as tg
import synth_inputs as si
from gpu_util import assert_close, gpu_tstgemm

pytestmark = pytest.mark.gpu

# Sums of at most K terms in fp32, each product exact: bounded by K 2^-24 of sum |X W| in any order, and measured at
# 1e-7 of the result's norm.  The walk of the lists is held to 1e-5 of sum |X W| (gpu_util); here a tenth of it, which a
# lost third plane (2^-16 = 1.5e-5 of every entry) cannot pass.
TIGHT = 1e-6


def tight(Y, Yd, A, what):
    err = np.abs(Y.astype(np.float64) - Yd)
    assert np.all(err <= TIGHT * A), f"{what}: {np.max(err / A):.2e}"


# rows: 32- and 64-row tiles and one more or less; K: below, at and above steps of 32, blocks of 64, groups and slices of
# them, not a multiple of 4; N: columns of a fragment, of a tile, odd.  Every tile shape is taken with K whole and in slices
# (test_host_api.py has the list).
EDGES = [(11, 1, 1), (31, 31, 33), (32, 32, 32), (33, 33, 31), (64, 64, 64), (63, 65, 130), (65, 127, 63), (17, 257, 300),
         (100, 515, 129), (129, 1027, 257), (255, 2050, 255), (257, 64, 1025), (40, 8195, 100), (700, 333, 700), (1025, 100, 513),
         (1300, 4100, 5000), (2049, 2053, 4100), (36, 985, 23), (297, 2355, 1685), (777, 3001, 2999), (255, 4033, 4031),
         (1410, 1529, 1955), (640, 4099, 4099)]


@pytest.mark.parametrize("M,K,N", EDGES)
def test_tile_edges(M, K, N):
    W, X, b = si.make_inputs(M, K, N, 0.5, "normal", seed=700 + M + K + N)
    ot = oracle.tcsc_build(W)
    Yd, A, _ = oracle.tstgemm(X, ot, b)
    Y, h = gpu_tstgemm(W, X, b)
    tight(Y, Yd, A, f"{M}x{K}x{N}")
    _, Xi, _ = si.make_inputs(M, K, N, 0.5, "int8", seed=701 + M)
    Yi, _ = gpu_tstgemm(W, Xi, b, handle=h)
    assert np.array_equal(Yi, oracle.tstgemm(Xi, ot, b)[0].astype(np.float32))
    # the same call through the kernels that walk lists and row sets
    other = dict(wide_lists=True) if M <= 8 else dict(list_walk=1) if M <= 64 else dict(cols_per_wave=4)
    Yo, _ = gpu_tstgemm(W, X, b, handle=h, **other)
    assert np.all(np.abs(Yo.astype(np.float64) - Y) <= 1.1e-5 * A)


# rows of X around every instance of the small kernel (2, 5, 8, 10); groups of 256 rows of W for four and for eight
# wavefronts, fewer and more than these, not a multiple of 4; one to four tiles of 16 columns per workgroup, and more
@pytest.mark.parametrize("M", range(1, 11))
@pytest.mark.parametrize("K,N", [(1, 1), (65, 33), (1023, 17), (1029, 40), (2307, 31), (4097, 16), (300, 16400), (1500, 5000),
                                 (1300, 9000), (1280, 13000), (1281, 20000)])
def test_few_rows(M, K, N):
    W, X, b = si.make_inputs(M, K, N, 0.75, "normal", seed=710 + M + K)
    ot = oracle.tcsc_build(W)
    Yd, A, _ = oracle.tstgemm(X, ot, b)
    # the row sets and (M > 8) what else the call asks for; then the lists alone
    t = tg.tcsc_upload(tg.tcsc_build(W), forms=tg.FORM_ROWSETS | tg.FORM_CUTS | tg.FORM_WORKSPACE)
    Y, _ = gpu_tstgemm(W, X, b, handle=t)
    tight(Y, Yd, A, f"{M}x{K}x{N}")
    Xi = np.random.default_rng(712).integers(-8, 9, (M, K)).astype(np.float32)
    Yi, _ = gpu_tstgemm(W, Xi, b, handle=t)
    assert np.array_equal(Yi, oracle.tstgemm(Xi, ot, b)[0].astype(np.float32))
    if M <= 8:
        Yo, _ = gpu_tstgemm(W, X, b, handle=tg.tcsc_upload(tg.tcsc_build(W), forms=tg.FORM_LISTS16))
        assert_close(Yo, Yd, A, f"{M}x{K}x{N} lists")


# the base-3 codes: pieces of 80 rows, groups of four of them, four and eight wavefronts, K in and beyond its last byte
@pytest.mark.parametrize("M", range(1, 9))
@pytest.mark.parametrize("K,N", [(1, 1), (79, 17), (81, 16), (319, 33), (320, 40), (1283, 31), (1601, 5000), (2563, 9000),
                                 (700, 16400), (1290, 13000), (5121, 70)])
def test_packed_codes(M, K, N):
    import torch
    W, X, b = si.make_inputs(M, K, N, 0.5, "normal", seed=790 + M + K)
    ot = oracle.tcsc_build(W)
    Yd, A, _ = oracle.tstgemm(X, ot, b)
    t = tg.tcsc_upload(tg.tcsc_build(W), forms=tg.FORM_PACKED)
    bd = torch.from_numpy(b).cuda()
    Xi = np.random.default_rng(791).integers(-8, 9, (M, K)).astype(np.float32)
    Ydi = oracle.tstgemm(Xi, ot, b)[0].astype(np.float32)
    tight(tg.tstgemm_packed(torch.from_numpy(X).cuda(), t, bd).cpu().numpy(), Yd, A, f"{M}x{K}x{N}")
    assert np.array_equal(tg.tstgemm_packed(torch.from_numpy(Xi).cuda(), t, bd).cpu().numpy(), Ydi)
    # the kernel on the vector ALU, which a request for parts of K still gets
    assert np.array_equal(tg.tstgemm_packed(torch.from_numpy(Xi).cuda(), t, bd, k_slices=1).cpu().numpy(), Ydi)
    # finite, but beyond what the scaled planes hold
    Xl = np.ldexp(Xi, 112).astype(np.float32)
    Yl = tg.tstgemm_packed(torch.from_numpy(Xl).cuda(), t, None).cpu().numpy()
    Ye = np.ldexp(oracle.tstgemm(Xi, ot, None)[0], 112)
    assert np.array_equal(Yl.astype(np.float64), Ye)


def _same(Y, Yd):
    """Equal in what is not finite; else within the tolerance of the finite part of the sum."""
    return np.array_equal(np.isnan(Y), np.isnan(Yd)) and np.array_equal(np.isposinf(Y), np.isposinf(Yd)) \
        and np.array_equal(np.isneginf(Y), np.isneginf(Yd))


@pytest.mark.parametrize("M,K,N", [(3, 300, 70), (8, 1500, 40), (40, 300, 70), (40, 4100, 200), (300, 333, 130)])
@pytest.mark.parametrize("alpha", [None, 0.25])
def test_infinities_and_nans(M, K, N, alpha):
    """X with infinities and NaNs: exactly the outputs whose lists hold them are not finite, as a plain sum gives it."""
    W, X, b = si.make_inputs(M, K, N, 0.25, "normal", seed=720 + M + K)
    rng = np.random.default_rng(721)
    for v in (np.inf, -np.inf, np.nan):
        X[rng.integers(0, M, 2), rng.integers(0, K, 2)] = v
    X[0, 5], X[0, K - 1] = np.inf, np.inf
    Yd = np.zeros((M, N))
    for m in range(M):
        used = np.where(W != 0, X[m][:, None].astype(np.float64) * W, 0.0)
        with np.errstate(invalid="ignore"):
            Yd[m] = used.sum(axis=0)
    with np.errstate(invalid="ignore"):
        A = np.where(np.isfinite(Yd), np.abs(np.where(np.isfinite(X), X, 0)).astype(np.float64) @ np.abs(W), 0) + np.abs(b)
        Yd = Yd + b
        if alpha is not None:
            Yd = np.where(Yd > 0, Yd, alpha * Yd)
    Y, _ = gpu_tstgemm(W, X, b, alpha=alpha)
    assert np.isfinite(Yd).any() and not np.isfinite(Yd).all()
    assert _same(Y, Yd)
    ok = np.isfinite(Yd)
    assert np.all(np.abs(Y[ok] - Yd[ok]) <= 1e-5 * A[ok])


@pytest.mark.parametrize("M,K,N", [(1, 65, 17), (5, 2100, 70), (10, 300, 5000), (17, 65, 40), (40, 4100, 200), (64, 512, 512),
                                   (130, 4100, 70), (300, 333, 130), (700, 300, 1100)])
def test_infinities_beside_numbers_of_any_size(M, K, N):
    """Rows of integers times powers of two from the smallest float to where the sums just fit, one of them mixed, each with
    an infinity under a weight that is zero in most columns: there the result is exact (the mixed row: within the bound of
    an fp32 sum); where the weight is not zero, the infinity of its sign, or NaN where two of them meet."""
    W, X, _ = si.make_inputs(M, K, N, 0.5, "int8", seed=750 + M + K)
    W[K // 3] = 0
    W[K // 3, ::7], W[K // 3, 3::7] = 1, -1
    W[K - 1] = W[K // 3] * np.where(np.arange(N) % 2, 1, -1)
    exponents = np.array([0, -149, 116, -100, 62, 70, 100, -126])[np.arange(M) % 8]
    X = np.ldexp(X.astype(np.float64), exponents[:, None])
    mixed = np.arange(M) % 8 == 5
    X[mixed, ::2] = np.ldexp(X[mixed, ::2], -140)
    X[:, K - 1] = 0
    Xc = X.copy()
    Xc[:, K // 3] = 0
    Yd, A = Xc @ W, np.abs(Xc) @ np.abs(W)
    sign = np.where(np.arange(M) % 3, 1.0, -1.0)
    X[:, K // 3] = sign * np.inf
    X[::4, K - 1] = np.inf
    with np.errstate(invalid="ignore"):
        for k in (K // 3, K - 1):
            held = np.isinf(X[:, k])[:, None] & (W[k] != 0)[None, :]
            Yd[held] += (X[:, k][:, None] * np.where(W[k] == 0, 1, W[k]))[held]
    Y, h = gpu_tstgemm(W, X.astype(np.float32), None)
    assert np.isfinite(Yd).any() and np.isinf(Yd).any() and _same(Y, Yd)
    ok = np.isfinite(Yd)
    exact = ok & ~mixed[:, None]
    assert np.array_equal(Y[exact].astype(np.float64), Yd[exact])
    assert np.all(np.abs(Y[ok] - Yd[ok]) <= TIGHT * A[ok])
    # the list and row-set kernels agree
    other = dict(wide_lists=True) if M <= 8 else dict(list_walk=1) if M <= 64 else dict(cols_per_wave=4)
    assert _same(gpu_tstgemm(W, X.astype(np.float32), None, handle=h, **other)[0], Yd)


@pytest.mark.parametrize("M,K,N,every_row", [(1, 4096, 4096, True), (8, 4096, 4096, False), (256, 4096, 4096, False),
                                             (1024, 1024, 4096, True)])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 1e35])
def test_x_that_is_not_finite_does_not_stall_a_call(M, K, N, every_row, value):
    """What X holds must not change a call's time by much: with an infinity, a NaN or a number beyond the scaled range at
    most four times what the list and row-set kernels take (they do not look at X), and 30 us for the launches.  (Walking
    the members of each such output by one lane took 10 to 35 times as long as they.)"""
    import torch
    W = si.draw_ternary(np.random.default_rng(755), K, N, 0.5)
    X = torch.randn(M, K, device="cuda")
    X[slice(None) if every_row else M // 2, K // 3] = value
    ws = torch.empty(tg.tstgemm_workspace_bytes(M, K, N)[1] + 256, dtype=torch.uint8, device="cuda")
    t = tg.tcsc_upload(tg.tcsc_build(W))
    lists = tg.tcsc_upload(tg.tcsc_build(W), forms=tg.FORM_LISTS16) if M <= 8 else t

    def us(handle, call=tg.tstgemm, **options):
        Y = torch.empty(M, N, device="cuda")
        best = float("inf")
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            call(X, handle, None, Y, workspace=ws, **options)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * e0.elapsed_time(e1))
        return best

    assert us(t) <= 4.0 * us(lists, **({} if M <= 8 else dict(cols_per_wave=4))) + 30.0
    if M <= 8 and np.isfinite(value):   # from the base-3 codes, beside the kernel on the vector ALU
        assert us(t, tg.tstgemm_packed) <= 4.0 * us(t, tg.tstgemm_packed, k_slices=1) + 30.0


@pytest.mark.parametrize("M,K,N", [(5, 300, 70), (40, 300, 70), (130, 4100, 70)])
@pytest.mark.parametrize("exponent", [-149, -140, -126, -110, 0, 60, 99, 110, 116])
def test_range_of_x(M, K, N, exponent):
    """Integers times a power of two, from the smallest float to where the sums just fit: exact, as with any order of
    additions."""
    W, X, _ = si.make_inputs(M, K, N, 0.5, "int8", seed=740 + M)
    ot = oracle.tcsc_build(W)
    Yd = oracle.tstgemm(X, ot, None)[0]
    scale = np.ldexp(1.0, exponent)
    Xs = (X.astype(np.float64) * scale).astype(np.float32)
    assert np.array_equal(Xs.astype(np.float64), X.astype(np.float64) * scale)
    Y, _ = gpu_tstgemm(W, Xs, None)
    assert np.array_equal(Y.astype(np.float64), Yd * scale)


def test_full_significands():
    """Floats whose last bits are set and whose exponents lie far apart, one entry of W per column: nothing of X is lost."""
    M, K = 70, 200
    rng = np.random.default_rng(760)
    X = (rng.integers(2**23, 2**24, (M, K)) * np.exp2(rng.integers(-120, 60, (M, K)).astype(np.float64))).astype(np.float32)
    W = np.zeros((K, K), np.int8)
    W[np.arange(K), rng.permutation(K)] = rng.choice([-1, 1], K)
    for m in (1, 8, 20, 70):
        Y, _ = gpu_tstgemm(W, X[:m], None)
        assert np.array_equal(Y.astype(np.float64), X[:m].astype(np.float64) @ W)


@pytest.mark.parametrize("M", [64, 256])
def test_without_the_row_sets_or_with_little_scratch(M):
    """What decides beside the sizes: M <= 64 without the row sets takes the lists; the least workspace is enough."""
    import torch
    K, N = 2048, 256
    W, X, b = si.make_inputs(M, K, N, 0.5, "normal", seed=770 + M)
    Yd, A, _ = oracle.tstgemm(X, oracle.tcsc_build(W), b)
    Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(b).cuda()
    least = tg.tstgemm_workspace_bytes(M, K, N)[0]
    for forms in ([tg.FORM_CUTS, tg.FORM_CUTS | tg.FORM_ROWSETS] if M <= 64 else [tg.FORM_ROWSETS]):
        t = tg.tcsc_upload(tg.tcsc_build(W), forms=forms)
        for size in (least, 64 << 20):
            ws = torch.empty(size, dtype=torch.uint8, device="cuda")
            assert_close(tg.tstgemm(Xd, t, bd, workspace=ws).cpu().numpy(), Yd, A, f"forms {forms} {size} bytes")
        with pytest.raises(tg.TstgemmError) as err:
            tg.tstgemm(Xd, t, bd, workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))
        assert err.value.code == -8


def test_y_beyond_four_gib():
    """A Y of more than 2^32 bytes whose column count is not a multiple of a tile's: every element, integer X.  (A lane whose
    column does not exist must store nowhere, also where the rest of Y would reach as far as a 32-bit offset does.)"""
    import torch
    M, K, N = 1_150_000, 20, 950
    assert M * N * 4 > (1 << 32) + (64 << 20) and N % 64
    g = torch.Generator(device="cuda").manual_seed(785)
    W = np.random.default_rng(786).integers(-1, 2, (K, N)).astype(np.int8)
    X = torch.randint(-8, 9, (M, K), generator=g, device="cuda").float()
    b = torch.randint(-8, 9, (N,), generator=g, device="cuda").float()
    t = tg.tcsc_upload(tg.tcsc_build(W), forms=tg.FORM_ROWSETS)
    ws = torch.empty(tg.tstgemm_workspace_bytes(M, K, N)[0], dtype=torch.uint8, device="cuda")
    Y = tg.tstgemm(X, t, b, torch.full((M, N), float("nan"), device="cuda"), workspace=ws)
    Wd = torch.from_numpy(W).cuda().float()
    for m in range(0, M, 1 << 17):
        Xs = X[m:m + (1 << 17)]
        assert torch.equal(Y[m:m + (1 << 17)], Xs @ Wd + b), f"rows from {m}"   # small integers: exact in any order
    rows = torch.tensor([0, 1, M // 2, M - 1], device="cuda")
    Yd = oracle.tstgemm(X[rows].cpu().numpy(), oracle.tcsc_build(W), b.cpu().numpy())[0]
    assert np.array_equal(Y[rows].cpu().numpy(), Yd.astype(np.float32))


@pytest.mark.parametrize("M", [(1 << 30) - 64, 1 << 30, (1 << 31) - 1])
def test_as_many_rows_as_an_int_holds(M):
    """Rows over a single column: as many tiles as one launch may have (its threads number less than 2^32), one more, and
    row numbers that leave no room to round up in 32 bits."""
    import torch
    X = torch.empty((M, 1), device="cuda")
    X.view(-1).copy_(torch.arange(M, device="cuda", dtype=torch.int32) % 1001)
    b = torch.full((1,), 3.0, device="cuda")
    t = tg.tcsc_upload(tg.tcsc_build(np.array([[-1]], np.int8)))
    Y = tg.tstgemm(X, t, b)
    assert torch.equal(Y, 3.0 - X)


def test_calls_follow_torchs_current_stream():
    """Without a stream argument a call goes to torch's current stream, whichever that is: behind a long piece of work on a
    side stream it reads what that work writes, and torch's own work behind it reads its result."""
    import torch
    M, K, N = 4, 512, 256
    W, X, b = si.make_inputs(M, K, N, 0.5, "int8", seed=780)
    Yd, _, _ = oracle.tstgemm(X, oracle.tcsc_build(W), b)
    t = tg.tcsc_upload(tg.tcsc_build(W))
    Xh, bd = torch.from_numpy(X).cuda(), torch.from_numpy(b).cuda()
    big = torch.randn(4096, 4096, device="cuda")
    Xd = torch.zeros_like(Xh)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(10):
            big = big @ big * 1e-3
        Xd.copy_(Xh)
        Y = tg.tstgemm(Xd, t, bd)
        twice = Y * 2
    torch.cuda.synchronize()
    assert np.array_equal(twice.cpu().numpy(), 2 * Yd.astype(np.float32))
    Y2 = tg.tstgemm(Xd, t, bd, stream=side)
    side.synchronize()
    assert torch.equal(Y2, Y)


@pytest.mark.parametrize("M,K,N", [(32, 4096, 4096), (40, 1796, 100), (100, 4099, 500), (777, 3001, 2999)])
def test_slices_whose_sums_are_near_the_largest_float(M, K, N):
    """One entry of 3e38 of either sign, or none, per slice of K and row: where the sum of all of them is a float, it is the result, in whatever
    order the slices are added."""
    rng = np.random.default_rng(795 + M)
    W = si.draw_ternary(rng, K, N, 0.25)
    t = tg.tcsc_build(W)
    slices = tg.tstgemm_query_route(t, M).k_slices
    assert slices > 1
    rows = np.arange(slices) * -(-(-(-K // 64)) // slices) * 64
    W[rows] = 1
    signs = rng.integers(-1, 2, (M, slices))
    while (wrong := np.abs(signs.sum(axis=1)) > 1).any():
        signs[wrong] = rng.integers(-1, 2, (int(wrong.sum()), slices))
    X = np.zeros((M, K), np.float32)
    X[:, rows] = signs * np.float32(3e38)
    Y, t = gpu_tstgemm(W, X, None)
    assert tg.tstgemm_query_route(t, M).k_slices == slices
    assert np.array_equal(Y, np.repeat(signs.sum(axis=1, keepdims=True) * np.float32(3e38), N, axis=1))
