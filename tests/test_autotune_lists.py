"""hm_autotune times lists of shifts beside ranges (the two run different row passes): its workspace holds the list,
and what it chooses for lists gives the same sums as the untuned plan."""
import ctypes

import pytest

import paper_2601_07824_amd as hm
from synth import states as S


def a256(b):
    return (b + 255) // 256 * 256


@pytest.mark.parametrize("dtype,n,sample", [(0, 20, 16384), (0, 24, 256), (1, 18, 1024), (0, 20, 100)])
def test_workspace_holds_the_list(dtype, n, sample):
    ctx = hm.Context()
    for opt, v in ((hm.OPT_FORCE_PATH, 2), (hm.OPT_BATCH_SHIFTS, 8), (hm.OPT_ROW_BITS, 12), (hm.OPT_PIPELINE, 1),
                   (hm.OPT_LDS_SPLIT, 2), (hm.OPT_STREAMS, 1)):  # one candidate
        ctx.set_option(opt, v)
    plan, tune = ctypes.c_size_t(0), ctypes.c_size_t(0)
    assert hm.lib().hm_workspace_size(ctx.h, hm.OP_SRE_ROWS, n, dtype, 1, 0, ctypes.byref(plan)) == 0
    assert hm.lib().hm_autotune_workspace(ctx.h, n, dtype, sample, ctypes.byref(tune)) == 0
    rows = max(sample // 4, min(sample, 256))
    assert tune.value == plan.value + a256(sample * 2 * 8) + a256(rows * 8)


@pytest.mark.gpu
@pytest.mark.parametrize("c64,n", [(True, 18), (False, 17), (True, 15), (True, 21)])
def test_tuned_lists_match(c64, n):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.from_numpy(S.gaussian_state(n, seed=8700 + n)).to(torch.complex64 if c64 else torch.complex128).cuda()
    ctx = hm.Context()
    print(f"[autotune lists] n={n} c64={c64}", flush=True)
    hm.autotune(x, 512, ctx=ctx)
    rows = [0, 1, 7, 8, 2 ** (n - 1), 2 ** n - 1] + [(2654435761 * i) % 2 ** n for i in range(1, 90)]
    got, want = hm.sre_rows(x, rows, (2.0, 1.0), ctx=ctx).cpu(), hm.sre_rows(x, rows, (2.0, 1.0)).cpu()
    # a row's sum of 2^n values in another tile shape: FP32 rounding of single values, FP64 order
    assert ((got - want).abs() / want.abs()).max().item() < (2e-5 if c64 else 1e-11), (got, want)
    hm.lib().hm_tune_clear(ctx.h)
    assert torch.equal(hm.sre_rows(x, rows, (2.0, 1.0), ctx=ctx).cpu(), want)
