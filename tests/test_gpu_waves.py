"""The matrix-core kernel whose wavefronts share nothing but their sums (32 x 64 and 32 x 128 of Y, four groups of wavefronts over K):
shapes at the edges of its tiles, blocks and copies, and X off the border that its copies need, against the oracle element by
element."""
import numpy as np
import pytest

import oracle
import paper_2510_06957_amd as tg
import synth_inputs as si
from gpu_util import gpu_tstgemm
from test_gpu_matrix import _same, tight

# rows: one, all but one, all of a tile and one more; K: four blocks of 64 and the last of them in part, one wavefront with a block more
# or with none, many blocks, an odd and an even number of them a wavefront; columns: of a fragment, of a tile, one more or less, odd.
NARROW = [(11, 256, 1), (31, 252, 63), (32, 260, 64), (33, 316, 65), (64, 320, 130), (95, 580, 257), (129, 1024, 1000), (40, 1796, 100),
          (36, 4100, 700), (256, 2048, 2048), (32, 2048, 7950), (65, 2052, 3001), (96, 2308, 4031)]
WIDE = [(33, 4096, 5000), (255, 4092, 4031), (256, 512, 4096), (64, 8196, 4100), (128, 8196, 1000),
        (300, 2048, 4100)]


def route(t, M):
    """tstgemm_query_route() with the kernel's own name: some tiles of k_matrix look like k_waves'."""
    r = tg.tstgemm_query_route(t, M)
    waves = tg.tstgemm_query_waves(t, M)
    assert not waves or r.kernel == "k_matrix"
    return "k_waves" if waves else r.kernel, r.tile_rows, r.tile_cols, r.k_groups


@pytest.mark.parametrize("M,K,N", NARROW + WIDE)
def test_routes(M, K, N):
    none, starts = np.zeros(0, np.int32), np.zeros(N + 1, np.int32)
    if M > 64:
        t = tg.tcsc_from_arrays(starts, starts, none, none, K, N)
    else:   # (with few rows an empty matrix is the lists')
        t = tg.tcsc_build(si.draw_ternary(np.random.default_rng(1), K, N, 0.5))
    assert route(t, M) == ("k_waves", 32, 64 if (M, K, N) in NARROW else 128, 4)


def test_the_kernels_name():
    """tstgemm_query_waves() tells the two kernels apart where tile and groups are alike, and refuses what tstgemm_query_route() refuses."""
    t = tg.tcsc_build(si.draw_ternary(np.random.default_rng(1), 1001, 1000, 0.5))
    assert route(t, 129) == ("k_matrix", 32, 64, 4) and not tg.tstgemm_query_waves(t, 5)
    t = tg.tcsc_build(si.draw_ternary(np.random.default_rng(1), 1000, 1000, 0.5))
    assert route(t, 129) == ("k_waves", 32, 64, 4) and not tg.tstgemm_query_waves(t, 5) and not tg.tstgemm_query_waves(t, 4096)
    with pytest.raises(tg.TstgemmError) as e:
        tg.tstgemm_query_waves(t, 0)
    assert e.value.code == -1
    tg.tcsc_select_forms(t, tg.FORM_CUTS)
    with pytest.raises(tg.TstgemmError) as e:
        tg.tstgemm_query_waves(t, 129)
    assert e.value.code == -7


@pytest.mark.parametrize("M,K,N,waves", [(192, 4096, 10880, True), (192, 4096, 11008, False), (352, 4096, 5888, True), (544, 4096, 4096, False),
                                         (352, 832, 12376, False), (480, 1472, 4480, True), (672, 1536, 6528, True)])
def test_more_tiles_than_places(M, K, N, waves):
    """Tiles that start in a second round of the chip cost more than they compute: a few of them leave the call to shared cuts of X."""
    none, starts = np.zeros(0, np.int32), np.zeros(N + 1, np.int32)
    t = tg.tcsc_from_arrays(starts, starts, none, none, K, N)
    assert tg.tstgemm_query_waves(t, M) == waves and (not waves or route(t, M)[1::2] == (32, 4))


@pytest.mark.parametrize("M,K,N,tile", [(246, 256, 6144, (32, 128, 2)), (640, 256, 1024, (32, 128, 2)), (905, 216, 1307, (32, 128, 2)),
                                        (390, 420, 2685, (64, 128, 1)), (1668, 272, 651, (64, 128, 1)), (113, 204, 4926, (32, 128, 2)),
                                        (97, 256, 7552, (32, 128, 2)), (303, 204, 522, (32, 64, 4)), (1190, 492, 906, (32, 128, 4)),
                                        (155, 436, 5861, (32, 128, 4)), (960, 320, 485, (32, 64, 4))])
def test_few_blocks_on_shared_compute_units(M, K, N, tile):
    """Up to two blocks a wavefront: the sums at the end take longer than the steps, and two workgroups of a compute unit share the way there.  Timed
    alternatives: 246 x 256 x 6144 7.1 us in k_matrix and 7.4 in k_waves, 1668 x 272 x 651 7.1 and 8.9, 303 x 204 x 522 4.7 and 4.5, 1190 x 492 x 906 10.1 and 9.3."""
    none, starts = np.zeros(0, np.int32), np.zeros(N + 1, np.int32)
    assert route(tg.tcsc_from_arrays(starts, starts, none, none, K, N), M) == ("k_waves" if tile[2] == 4 else "k_matrix",) + tile


@pytest.mark.parametrize("M,K,N,tile", [(2159, 13940, 172, ("k_matrix", 64, 256, 2, 7)), (570, 9500, 925, ("k_matrix", 64, 256, 2, 7)),
                                        (1846, 2840, 630, ("k_waves", 32, 128, 4, 1)), (2943, 2920, 348, ("k_waves", 32, 128, 4, 1)),
                                        (33, 4096, 5000, ("k_waves", 32, 128, 4, 3)), (473, 6748, 2681, ("k_waves", 32, 128, 4, 3))])
def test_slices_on_shared_compute_units(M, K, N, tile):
    """The ends of workgroups count for each of a compute unit's, in slices too.  Timed: 2159 x 13940 x 172 44.1 us in five slices of k_waves, 40.7 in seven of
    k_matrix, 1846 x 2840 x 630 29.3 in three slices, 27.2 whole."""
    t = tg.tcsc_build(si.draw_ternary(np.random.default_rng(1), K, N, 0.5))
    assert route(t, M) + (tg.tstgemm_query_route(t, M).k_slices,) == tile


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", NARROW + WIDE)
def test_tile_edges(M, K, N):
    import torch
    W, X, b = si.make_inputs(M, K, N, 0.5, "normal", seed=300 + M + K + N)
    ot = oracle.tcsc_build(W)
    Yd, A, _ = oracle.tstgemm(X, ot, b)
    Y, t = gpu_tstgemm(W, X, b)
    assert route(t, M) == ("k_waves", 32, 64 if (M, K, N) in NARROW else 128, 4)
    tight(Y, Yd, A, f"{M}x{K}x{N}")
    _, Xi, _ = si.make_inputs(M, K, N, 0.5, "int8", seed=301 + M)
    Yi = oracle.tstgemm(Xi, ot, b)[0].astype(np.float32)
    assert np.array_equal(gpu_tstgemm(W, Xi, b, handle=t)[0], Yi)
    # X four bytes off the border: through registers, the same sums
    off = torch.empty(M * K + 1, device="cuda")[1:].view(M, K)
    off.copy_(torch.from_numpy(Xi))
    Yo = torch.full((M, N), float("nan"), device="cuda")
    tg.tstgemm(off, t, torch.from_numpy(b).cuda(), Yo)
    assert np.array_equal(Yo.cpu().numpy(), Yi)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(31, 252, 63), (33, 316, 65), (36, 4100, 700), (65, 2052, 3001), (64, 8196, 1100)])
def test_infinities_beyond_the_rows(M, K, N):
    """A row's last entries and the first of the row behind it are infinite or NaN: only outputs whose lists hold them show it, also
    where the last block of K reaches into the next row."""
    W, X, b = si.make_inputs(M, K, N, 0.25, "normal", seed=320 + M)
    X[1, K - 1], X[2, 0], X[M - 1, K - 1], X[M - 1, 3] = np.inf, -np.inf, np.nan, np.inf
    with np.errstate(invalid="ignore"):
        Yd = np.stack([np.where(W != 0, X[m][:, None].astype(np.float64) * W, 0.0).sum(axis=0) for m in range(M)]) + b
    A = np.abs(np.where(np.isfinite(X), X, 0)).astype(np.float64) @ np.abs(W) + np.abs(b)
    Y, t = gpu_tstgemm(W, X, b)
    assert route(t, M)[0] == "k_waves"
    ok = np.isfinite(Yd)
    assert ok.any() and not ok.all() and _same(Y, Yd)
    assert np.all(np.abs(Y[ok] - Yd[ok]) <= 1e-6 * A[ok])


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(256, 2048, 2048), (65, 2052, 3001), (300, 832, 5824), (672, 1536, 6528), (367, 512, 2368), (33, 260, 100)])
def test_sums_are_rounded_once(M, K, N):
    """X between 1/2 and 1 in size: the top planes are multiples of 2^-8 and their sums below 2^16, what is left multiples of 2^-24 with sums below 1,
    so both are exact whatever the order, and the result is their sum rounded once, however many wavefronts share K."""
    rng = np.random.default_rng(340 + M)
    X = (rng.uniform(0.5, 1.0, (M, K)) * rng.choice([-1.0, 1.0], (M, K))).astype(np.float32)
    W = si.draw_ternary(rng, K, N, 0.5)
    Y, t = gpu_tstgemm(W, X, None)
    r = tg.tstgemm_query_route(t, M)
    assert route(t, M)[0] == "k_waves" and r.k_slices == 1
    assert np.array_equal(Y, (X.astype(np.float64) @ W).astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N", [(36, 700), (22, 2048)])
def test_a_last_block_in_part_costs_no_more_than_a_whole_one(M, N):
    """K = 204 and K = 256 are four blocks each.  What is done for the part beyond K (a few bytes of the LDS cleared) must not show: at most 6 % more (clearing
    all of the ring took 11 to 14 %), the least of many turns of a graph of 20 calls."""
    import torch
    best = {}
    for K in (204, 256):
        W, X, b = si.make_inputs(M, K, N, 0.5, "normal", seed=350)
        t = tg.tcsc_upload(tg.tcsc_build(W))
        assert route(t, M) == ("k_waves", 32, 64, 4)
        Xd, bd, Y = torch.from_numpy(X).cuda(), torch.from_numpy(b).cuda(), torch.empty(M, N, device="cuda")
        tg.tstgemm(Xd, t, bd, Y)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                tg.tstgemm(Xd, t, bd, Y)
        best[K] = float("inf")
        for _ in range(40):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                graph.replay()
            e1.record()
            torch.cuda.synchronize()
            best[K] = min(best[K], e0.elapsed_time(e1))
    assert best[204] <= 1.06 * best[256], best


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", NARROW + WIDE)
def test_results_do_not_depend_on_where_x_lies(M, K, N):
    """X four, eight and twelve bytes off a 16-byte border: the same bits.  A NaN beside X does not matter."""
    import torch
    W, X, b = si.make_inputs(M, K, N, 0.5, "normal", seed=360 + M + N)
    t = tg.tcsc_upload(tg.tcsc_build(W))
    Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(b).cuda()
    Y = tg.tstgemm(Xd, t, bd)
    assert Xd.data_ptr() % 16 == 0 and route(t, M)[0] == "k_waves"
    for by in (1, 2, 3):
        room = torch.full((M * K + 8,), float("nan"), device="cuda")
        off = room[by:by + M * K].view(M, K)
        off.copy_(Xd)
        assert off.data_ptr() % 16 == 4 * by
        assert torch.equal(tg.tstgemm(off, t, bd), Y)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(33, 4096, 5000), (255, 1532, 4031), (70, 832, 5824), (65, 8196, 1001), (95, 580, 257)])
@pytest.mark.parametrize("slopes", ["none", "one", "column"])
@pytest.mark.parametrize("off", [0, 1])
def test_epilogue_and_what_is_not_finite(M, K, N, slopes, off):
    """PReLU, and outputs that are taken again: a few infinities, NaNs and numbers beyond the scaled range in rows of both halves of a tile, the last row
    and the last entries among them, in tiles of either width, K whole and in slices, X on the border and off it."""
    import torch
    W, X, b = si.make_inputs(M, K, N, 0.25, "normal", seed=370 + M)
    rng = np.random.default_rng(371 + M)
    for m, v in ((0, np.inf), (1, np.nan), (7, 1e36), (16, -np.inf), (31, -1e36), (M - 2, np.inf), (M - 1, np.nan), (M - 1, np.inf)):
        X[m, rng.integers(0, K)] = v
    X[20, K - 1], X[21, 0], X[M - 1, K - 1] = np.inf, -np.inf, np.inf
    rest = ~np.isfinite(X)
    Xf = np.where(rest, 0, X).astype(np.float64)
    Yd, A = Xf @ W + b, np.abs(Xf) @ np.abs(W) + np.abs(b)
    with np.errstate(invalid="ignore"):
        for m, k in zip(*np.nonzero(rest)):
            Yd[m, W[k] != 0] += X[m, k] * W[k, W[k] != 0]
        alpha = None if slopes == "none" else rng.uniform(0.1, 0.4, 1 if slopes == "one" else N).astype(np.float32)
        if alpha is not None:
            Yd = np.where(Yd > 0, Yd, alpha * Yd)
    t = tg.tcsc_upload(tg.tcsc_build(W))
    assert route(t, M) == ("k_waves", 32, 128 if N > 4000 else 64, 4)
    room = torch.full((M * K + 4,), float("nan"), device="cuda")
    Xd = room[off:off + M * K].view(M, K)
    Xd.copy_(torch.from_numpy(X))
    Y = tg.tstgemm(Xd, t, torch.from_numpy(b).cuda(), alpha=None if alpha is None else torch.from_numpy(alpha).cuda()).cpu().numpy()
    ok = np.isfinite(Yd)
    assert ok.any() and not ok.all() and _same(Y, Yd)
    assert np.all(np.abs(Y[ok] - Yd[ok]) <= 1e-6 * A[ok])


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(33, 4096, 5000), (64, 8196, 4100), (82, 9024, 7424), (473, 6748, 2681)])
def test_slices_are_rounded_once_each(M, K, N):
    """X as in test_sums_are_rounded_once: each slice's sum is rounded once, and the slices are added in float, in pairs."""
    rng = np.random.default_rng(380 + M)
    X = (rng.uniform(0.5, 1.0, (M, K)) * rng.choice([-1.0, 1.0], (M, K))).astype(np.float32)
    W = si.draw_ternary(rng, K, N, 0.5)
    Y, t = gpu_tstgemm(W, X, None)
    n = tg.tstgemm_query_route(t, M).k_slices
    assert route(t, M) == ("k_waves", 32, 128, 4) and n > 1
    step = -(-(-(-K // 64)) // n) * 64
    part = [(X[:, k:k + step].astype(np.float64) @ W[k:k + step]).astype(np.float32) for k in range(0, K, step)]
    assert len(part) == n
    while n > 1:
        half = (n + 1) // 2
        for s in range(n - half):
            part[s] = part[s] + part[s + half]
        n = half
    assert np.array_equal(Y, part[0])
