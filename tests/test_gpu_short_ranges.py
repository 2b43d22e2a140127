"""Short ranges of shifts keep the kernels that suit them, read from the library's own kernel timings: groups of
shifts (SRE) and families of shifts (mana) share gathers but serialise or pad, which only long ranges pay back."""
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def profiled(hm, fn, reps):
    """{kernel family: (launches, milliseconds)} of one call."""
    fn()
    hm.profile_reset()
    hm.profile_enable(True)
    try:
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        return {k: (v[0] / reps, v[2] / reps) for k, v in hm.profile_read().items() if v[0]}
    finally:
        hm.profile_enable(False)


@pytest.mark.parametrize("c64,n", [(True, 17), (True, 18), (False, 19)])
def test_few_shifts_run_beside_each_other(c64, n):
    """Eight shifts take little longer than one; as one group they took about twice as long, one after another."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    x = torch.from_numpy(S.gaussian_state(n, seed=8300 + n)).to(torch.complex64 if c64 else torch.complex128).cuda()
    count = 8 if c64 else 4
    print(f"[short ranges] n={n} c64={c64}", flush=True)
    ms = [profiled(hm, lambda: hm.sre_partial(x, (2.0,), 1000, 1000 + c), 50)["sre_rowpass_write"][1] for c in (1, count)]
    assert ms[1] < 1.6 * ms[0], ms


@pytest.mark.parametrize("c64,n", [(True, 12), (False, 12)])
def test_one_shift_of_mana_is_one_pair(c64, n):
    """One shift takes less than the six of a sextet (padded to three pairs it took the same)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    x = torch.from_numpy(S.gaussian_state(n, d=3, seed=8320)).to(torch.complex64 if c64 else torch.complex128).cuda()
    print(f"[short ranges] mana n={n} c64={c64}", flush=True)
    ms = []
    for count in (1, 6):
        t = profiled(hm, lambda: hm.mana_partial(x, 30, 30 + count), 50)
        ms.append(t["mana_rowpass_write"][1] + t["mana_colpass"][1])
    assert ms[0] < 0.85 * ms[1], ms
