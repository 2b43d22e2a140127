"""Renyi indices through every form of the reduction (q = 2 alone; indices among 1, 2, 3, 4; any real q) on
the resident and the two-pass kernels, against the FP64 oracle.

Tolerances as in test_gpu_sre.py: 1e-10 relative (complex128), 1e-5 (complex64).
"""
import numpy as np
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

QS = [(1.0,), (3.0,), (4.0, 3.0, 2.0, 1.0), (0.5, 2.0, 2.5), (2.0, 2.0)]


@pytest.mark.parametrize("c64", [False, True])
@pytest.mark.parametrize("n,path", [(1, 0), (4, 0), (6, 0), (9, 0), (11, 0), (12, 0), (13, 0), (13, 2)])
def test_indices_vs_oracle(orc, n, path, c64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    for name, psi in (("gauss", S.gaussian_state(n, seed=4400 + n)), ("zero", S.zero_state(n))):
        v, w = S.to_c64_exact(psi) if c64 else (psi, psi)
        x = torch.from_numpy(v).cuda()
        ctx = hm.Context()
        ctx.force_path(path)
        for q in QS:
            print(f"[q kinds] n={n} path={path} c64={c64} state={name} q={q}", flush=True)
            got, want = hm.sre(x, q, ctx=ctx).cpu().numpy(), orc.sre_fwht(w, q)
            err = np.max(np.abs(got - want) / np.maximum(np.abs(want), 1.0))
            assert err < (1e-5 if c64 else 1e-10), (q, got, want)
