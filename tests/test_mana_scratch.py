"""HM_OPT_BATCH_SHIFTS bounds the scratch of two-pass mana: a launch of two shifts holds one pair of them."""
import ctypes

import pytest

import paper_2601_07824_amd as hm


@pytest.mark.parametrize("dtype,n", [(0, 9), (0, 12), (0, 13), (1, 8), (1, 12), (0, 14), (1, 13)])
def test_small_batches_keep_to_their_scratch(dtype, n):
    ctx = hm.Context()
    pair = 3 ** n * (16 if dtype else 8)
    sums = 2048 * 3 * 8  # per-workgroup sums, one set per pass
    for shifts in (1, 2, 3, 4, 5, 6, 8, 12):
        ctx.batch_shifts(shifts)
        b = ctypes.c_size_t(0)
        assert hm.lib().hm_workspace_size(ctx.h, 4, n, dtype, 1, 0, ctypes.byref(b)) == 0
        assert b.value <= (shifts + 1) // 2 * pair + 2 * sums + 1024, (shifts, b.value)
