"""tstgemm_query_digits(): which calls take X in digits, on the host alone."""
import ctypes

import numpy as np
import pytest

import paper_2510_06957_amd as tg


def empty_matrix(K, N):
    none, starts = np.zeros(0, np.int32), np.zeros(N + 1, np.int32)
    return tg.tcsc_from_arrays(starts, starts, none, none, K, N)


def test_large_calls_take_digits():
    t = empty_matrix(8192, 8200)
    assert not any(tg.tstgemm_query_digits(t, M) for M in (1, 8, 10, 17, 64, 256, 600))
    assert all(tg.tstgemm_query_digits(t, M) for M in (1536, 2048))
    # (k_large is faster on an empty W of this width)
    assert not tg.tstgemm_query_digits(empty_matrix(8192, 8192), 4096)
    # X large beside Y; no room for a tile in digits, or for a few only; K beyond what the kernel counts the planes of
    assert not tg.tstgemm_query_digits(empty_matrix(65536, 1000), 1024, 1 << 30)
    for size, taken in ((1 << 20, False), (16 << 20, False), (72 << 20, True)):
        assert tg.tstgemm_query_digits(t, 1536, workspace_bytes=size) == taken
    assert not tg.tstgemm_query_digits(empty_matrix(1 << 21, 8200), 1000, workspace_bytes=1 << 40)
    tg.tcsc_select_forms(t, tg.FORM_CUTS)
    with pytest.raises(tg.TstgemmError) as e:
        tg.tstgemm_query_digits(t, 1536)
    assert e.value.code == -7
    lib = tg.binding._load()
    assert lib.tstgemm_query_digits(None, 1, None) == -1 and lib.tstgemm_query_digits(t.handle, 0, None) == -1
    o = tg.binding.TstgemmOpts()
    assert lib.tstgemm_query_digits(t.handle, 1, ctypes.byref(o)) == -1      # struct_size


def test_digit_tests_take_every_tile():
    """The shapes of test_gpu_digits.py reach each tile that takes digits, with K whole and in slices."""
    from test_gpu_digits import SHAPES
    taken = set()
    for M, K, N in SHAPES:
        t = empty_matrix(K, N)
        size = tg.tstgemm_workspace_bytes(M, K, N)[1]
        assert tg.tstgemm_query_digits(t, M, size)
        r = tg.tstgemm_query_route(t, M, workspace_bytes=size)
        taken.add((r.tile_rows, r.tile_cols, r.k_groups, r.k_slices > 1))
    assert taken == {(64, 512, 1, False), (64, 512, 1, True), (64, 256, 1, False), (64, 256, 1, True)}, taken


@pytest.mark.parametrize("M", [9, 33, 64, 65, 128, 300, 777, 1500, 2048, 4096, 5000])
def test_best_workspace_is_as_good_as_any(M):
    """With the best_bytes of tstgemm_workspace_bytes() a call takes what it takes with more room than it can use, X in digits in
    one slab."""
    digits = 0
    for K, N in ((8192, 8192), (8191, 8201), (16384, 4096), (16380, 4100), (4096, 16384), (4161, 17950), (16384, 1000), (4096, 4096), (700, 9000), (65536, 600)):
        t = empty_matrix(K, N)
        best = tg.tstgemm_workspace_bytes(M, K, N)[1]

        def taken(size):
            r = tg.tstgemm_query_route(t, M, workspace_bytes=size)
            return r.kernel, r.tile_rows, r.tile_cols, r.k_groups, r.k_slices, tg.tstgemm_query_digits(t, M, size)

        assert taken(best) == taken(1 << 50), (M, K, N)
        if taken(best)[-1]:
            slices = r[4] if (r := taken(best))[4] > 1 else 0
            assert best >= -(-M // 64) * -(-K // 64) * 22529 + slices * M * (-(-N // 64) * 64) * 4
            digits += 1
    assert digits >= (2 if M >= 1500 else 0)
