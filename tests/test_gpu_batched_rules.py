"""Which launch form hm_sre_batched takes when it is left automatic, read from the kernel families that ran."""
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("ns,q,family", [
    ([9, 10] * 12, (2.0,), "sre_rowpass_resident"), ([9, 10] * 12, (0.5,), "sre_batch_persistent"),
    ([12, 13], (0.5,), "sre_rowpass_resident"), ([7, 8, 9, 10, 11], (1.0, 2.0), "sre_batch_persistent")])
def test_form_by_size_and_index_kind(ns, q, family):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    xs = [torch.from_numpy(S.to_c64_exact(S.gaussian_state(n, seed=7800 + i))[0]).cuda() for i, n in enumerate(ns)]
    print(f"[batched rules] ns={ns[:5]} q={q}", flush=True)
    hm.sre_batched(xs, q)
    hm.profile_reset()
    hm.profile_enable(True)
    try:
        hm.sre_batched(xs, q)
        torch.cuda.synchronize()
        ran = {k for k, v in hm.profile_read().items() if v[0]}
    finally:
        hm.profile_enable(False)
    assert ran & {"sre_rowpass_resident", "sre_batch_persistent"} == {family}, ran
