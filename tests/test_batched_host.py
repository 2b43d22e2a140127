"""Host side of hm_sre_batched (no GPU needed): what planning a batch costs and what its workspace covers."""
import ctypes
import time

import pytest

import paper_2601_07824_amd as hm

HM_OK = 0


def workspace(ctx, ns, dtype=0, n_q=1):
    b = ctypes.c_size_t(0)
    arr = (ctypes.c_int * len(ns))(*ns)
    assert hm.lib().hm_sre_batched_workspace(ctx.h, arr, len(ns), dtype, n_q, ctypes.byref(b)) == HM_OK
    return b.value


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_planning_grows_with_the_batch(mode):
    """8 times the states take about 8 times as long (64 times with a pass over all pairs of states)."""
    ctx = hm.Context()
    ctx.set_option(hm.OPT_BATCH_LAUNCH, mode)

    def best(count):
        ns = [10] * count
        out = []
        for _ in range(7):
            t = time.perf_counter()
            workspace(ctx, ns)
            out.append(time.perf_counter() - t)
        return min(out)
    assert best(32768) < 24 * best(4096)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("ns", [[11] * 64, [9, 10, 11, 12, 13, 14] * 200, [5, 6, 7], [17, 12, 3]])
def test_automatic_workspace_covers_both_forms(ns, dtype):
    """hm_autotune_batched may choose either form, for itself and for later calls on the workspace at hand."""
    forms = []
    for mode in (0, 1, 2):
        ctx = hm.Context()
        ctx.set_option(hm.OPT_BATCH_LAUNCH, mode)
        forms.append([workspace(ctx, ns, dtype, n_q) for n_q in (1, 3)])
    assert forms[0] == [max(a, b) for a, b in zip(forms[1], forms[2])], forms
