"""Two-pass mana over ranges long enough for families of three shifts (six shifts packed into three pairs), starting
and ending anywhere in a family or a sextet, for every row length that the family kernels are built for; and a few
shifts, which run pair by pair.  Against the FP64 oracle.

Tolerance: 1e-10 relative to the sum of |chi| for complex128; 3e-6 for complex64, the FP32 noise of the values of
one shift (a value of size |chi| carries about 1e-7 of the rms value; no averaging over shifts)."""
import numpy as np
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# least: shifts from which an aligned range goes by families (rows of 3^5, 3^5, 3^6, 3^6, 3^7; 3^4 .. 3^6)
@pytest.mark.parametrize("c64,n,least", [(True, 9, 174), (True, 10, 60), (True, 11, 24), (True, 12, 12), (True, 13, 6),
                                         (False, 8, 1026), (False, 9, 342), (False, 10, 114), (False, 11, 42),
                                         (False, 12, 18)])
def test_range_edges(orc, c64, n, least):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    psi = S.gaussian_state(n, d=3, seed=9400 + n)
    v, w = S.to_c64_exact(psi) if c64 else (psi, psi)
    x = torch.from_numpy(v).cuda()
    end = 3 ** n
    tol = 3e-6 if c64 else 1e-10
    for a0, a1 in ((0, least), (1, 6 + least), (2, 2 + least + 11), (4, 4 + least + 8), (243 + 5, 243 + 5 + least + 7),
                   (end - least - 4, end), (7, 8), (8, 11)):
        print(f"[mana family edges] n={n} c64={c64} shifts [{a0}, {a1})", flush=True)
        got, want = hm.mana_partial(x, a0, a1).cpu().numpy(), np.asarray(orc.mana_fft_sums(w, a0, a1))[:3]
        assert np.max(np.abs(got - want)) < tol * abs(want[0]), (a0, a1, got, want)
