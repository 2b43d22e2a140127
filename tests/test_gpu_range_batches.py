"""A range of shifts that starts inside a group of shifts is cut into no more launches than its length asks for."""
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("a0,count,launches", [(1000, 64, 1), (1003, 64, 1), (1003, 61, 1), (1003, 128, 2), (1003, 65, 2),
                                               (1003, 640, 11), (1000, 640, 10)])
def test_launches_of_a_range(a0, count, launches):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    n = 18
    ctx = hm.Context()
    ctx.batch_shifts(64)
    x = torch.from_numpy(S.gaussian_state(n, seed=8400)).cuda()
    print(f"[range batches] [{a0}, {a0 + count})", flush=True)
    hm.profile_reset()
    hm.profile_enable(True)
    try:
        got = hm.sre_partial(x, (2.0,), a0, a0 + count, ctx=ctx).cpu()
        ran = hm.profile_read()["sre_colpass"][0]
    finally:
        hm.profile_enable(False)
    assert ran == launches
    want = sum(hm.sre_partial(x, (2.0,), a, min(a + 64, a0 + count)).cpu() for a in range(a0, a0 + count, 64))
    assert ((got - want).abs() / want.abs()).max().item() < 1e-12  # FP64 sums in another order
