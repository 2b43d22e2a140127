"""Whole evaluations of few qubits in one launch of one workgroup (up to seven qubits), and the first sizes
above, against the FP64 oracle; the sums over the shifts agree with those of two half ranges.

Tolerances as in test_gpu_sre.py: 1e-10 relative (complex128), 1e-5 (complex64).
"""
import numpy as np
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

QS = [(2.0,), (1.0, 2.0, 3.0), (0.5, 2.5)]


@pytest.mark.parametrize("c64", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_one_launch_vs_oracle(orc, n, c64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    psi = S.gaussian_state(n, seed=5100 + n)
    v, w = S.to_c64_exact(psi) if c64 else (psi, psi)
    x = torch.from_numpy(v).cuda()
    tol = 1e-5 if c64 else 1e-10
    for q in QS:
        print(f"[small] n={n} c64={c64} q={q}", flush=True)
        got, want = hm.sre(x, q).cpu().numpy(), orc.sre_fwht(w, q)
        assert np.max(np.abs(got - want) / np.maximum(np.abs(want), 1.0)) < tol, (q, got, want)
        ns = 1 << n
        whole = hm.sre_partial(x, q, 0, ns).cpu().numpy()
        halves = hm.sre_partial(x, q, 0, ns // 2) + hm.sre_partial(x, q, ns // 2, ns)
        halves = halves.cpu().numpy()
        # the same per-shift sums added in another order: FP64 rounding of at most 2^n terms
        assert np.max(np.abs(whole - halves) / np.maximum(np.abs(whole), 1.0)) < 1e-12, (q, whole, halves)
