"""The persistent launch of hm_sre_batched, asked for (HM_OPT_BATCH_LAUNCH = 1): its tiles of every workgroup size,
with the index kinds it is built for, against single calls, and the batch of 1024 states.

Tolerances: complex128 1e-12, FP64 sums in another order; complex64 2e-6, FP32 sums of a thread's values in
another tile shape."""
import numpy as np
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def persistent():
    import paper_2601_07824_amd as hm
    ctx = hm.Context()
    ctx.set_option(hm.OPT_BATCH_LAUNCH, 1)
    return hm, ctx


@pytest.mark.parametrize("q", [(2.0,), (1.0, 2.0, 3.0), (0.5, 2.0)])
@pytest.mark.parametrize("c64,ns", [(True, [13, 6, 14]), (True, [15, 8, 11]), (True, [16, 12, 7]), (False, [12, 5, 13]),
                                    (False, [14, 8, 11]), (False, [15, 12, 6])])
def test_every_tile_size(ns, c64, q):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm, ctx = persistent()
    xs = []
    for i, n in enumerate(ns):
        psi = S.gaussian_state(n, seed=7900 + i)
        xs.append(torch.from_numpy(S.to_c64_exact(psi)[0] if c64 else psi).cuda())
    print(f"[batched persistent] ns={ns} c64={c64} q={q}", flush=True)
    got = hm.sre_batched(xs, q, ctx=ctx).cpu().numpy()[:, :-1]
    want = np.stack([hm.sre(x, q).cpu().numpy() for x in xs])[:, :-1]
    np.testing.assert_allclose(got, want, rtol=2e-6 if c64 else 1e-12, atol=0)


def test_1024_states_n10_to_16():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm, ctx = persistent()
    ns = np.random.default_rng(5005).integers(10, 17, size=1024)
    xs = [torch.from_numpy(S.to_c64_exact(S.gaussian_state(int(n), seed=5000 + i))[0]).cuda() for i, n in enumerate(ns)]
    print("[batched persistent] 1024 states", flush=True)
    got = hm.sre_batched(xs, (2.0,), ctx=ctx).cpu().numpy()
    want = np.stack([hm.sre(x, (2.0,)).cpu().numpy() for x in xs])
    np.testing.assert_allclose(got[:, 0], want[:, 0], rtol=2e-6, atol=0)
