"""Two-pass mana over shift ranges that start and end anywhere in a family of three shifts or a sextet (the
row pass gathers families of three and packs six shifts into three pairs), against the FP64 oracle.

Tolerance: 1e-10 relative to the sum of |chi| for complex128; 3e-6 for complex64, the FP32 noise of 3^9
values of one shift (a value of size |chi| carries about 1e-7 of the rms value; no averaging over shifts)."""
import numpy as np
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("c64", [False, True])
@pytest.mark.parametrize("n", [9, 10])
def test_range_edges(orc, n, c64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    psi = S.gaussian_state(n, d=3, seed=9300 + n)
    v, w = S.to_c64_exact(psi) if c64 else (psi, psi)
    x = torch.from_numpy(v).cuda()
    end = 3 ** n
    for a0 in (0, 1, 2, 3, 4, 5, 242, 243):
        for count in (1, 2, 5, 6, 7):
            print(f"[mana families] n={n} c64={c64} shifts [{a0}, {a0 + count})", flush=True)
            got = hm.mana_partial(x, a0, a0 + count).cpu().numpy()
            want = np.asarray(orc.mana_fft_sums(w, a0, a0 + count))[:3]
            assert np.max(np.abs(got - want)) < (3e-6 if c64 else 1e-10) * abs(want[0]), (a0, count, got, want)
    got, want = hm.mana_partial(x, end - 4, end).cpu().numpy(), np.asarray(orc.mana_fft_sums(w, end - 4, end))[:3]
    assert np.max(np.abs(got - want)) < (3e-6 if c64 else 1e-10) * abs(want[0]), (got, want)
