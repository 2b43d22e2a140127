"""hm_sre_batched's launch forms (one persistent launch, one launch per size class, the automatic choice on
both sides of its rule): the same states give the same values, state by state, as single calls.

Tolerance 1e-12 relative to max(|M_q|, 1): the forms transform a state alike (same tiles, same stage order)
and differ only in the order of FP64 sums."""
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("c64", [False, True])
@pytest.mark.parametrize("ns", [[5], [7, 11, 9, 8], [3, 6, 5, 9, 9, 1], [12, 13, 12], [8] * 65 + [9]])
def test_forms_agree(ns, c64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    dt = torch.complex64 if c64 else torch.complex128
    xs = [torch.from_numpy(S.gaussian_state(n, seed=7700 + i)).to(dt).cuda() for i, n in enumerate(ns)]
    want = torch.stack([hm.sre(x, (2.0,)) for x in xs]).cpu()
    for mode in (0, 1, 2):
        ctx = hm.Context()
        ctx.set_option(hm.OPT_BATCH_LAUNCH, mode)
        got = hm.sre_batched(xs, (2.0,), ctx=ctx).cpu()
        err = ((got - want).abs() / want.abs().clamp(min=1.0)).max().item()
        print(f"[batched forms] ns={ns[:6]} c64={c64} mode={mode} err={err:.2e}", flush=True)
        assert err < 1e-12, (mode, got, want)
