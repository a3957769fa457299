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
        size = tg.tstgemm_workspace_bytes(M, K, N)[1] + (96 << 20)
        assert tg.tstgemm_query_digits(t, M, size)
        r = tg.tstgemm_query_route(t, M, workspace_bytes=size)
        taken.add((r.tile_rows, r.tile_cols, r.k_groups, r.k_slices > 1))
    assert taken == {(64, 512, 1, False), (64, 512, 1, True), (64, 256, 1, False), (64, 256, 1, True)}, taken
