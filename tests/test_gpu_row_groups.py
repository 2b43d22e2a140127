"""The two-pass row pass by groups of consecutive shifts against the same shifts one by one (an explicit shift
list takes the per-shift row pass, which test_gpu_sre.py holds against the oracle): ranges that start and end
inside groups, on the first shifts, and where the top set bit changes; every row length the groups are built
for.

Both form every value by the same operations; only the order of the FP64 sums over shifts may differ: 1e-12."""
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("c64,n,row_bits", [(True, 14, 8), (True, 15, 9), (True, 17, 10), (True, 18, 11), (True, 19, 12),
                                            (True, 20, 13), (False, 14, 8), (False, 15, 9), (False, 16, 10), (False, 17, 11),
                                            (False, 18, 12), (False, 18, 13)])
def test_ranges_equal_single_rows(c64, n, row_bits):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    x = torch.from_numpy(S.gaussian_state(n, seed=8100 + n)).to(torch.complex64 if c64 else torch.complex128).cuda()
    ctx = hm.Context()
    ctx.force_path(2)
    ctx.set_option(hm.OPT_ROW_BITS, row_bits)
    top = 2 ** n
    for a0, a1 in ((0, 1), (0, 9), (1, 8), (3, 21), (5, 6), (8, 16), (2 ** row_bits - 5, 2 ** row_bits + 12),
                   (top // 2 - 3, top // 2 + 2), (top - 11, top)):
        print(f"[row groups] n={n} c64={c64} rows of 2^{row_bits}: shifts [{a0}, {a1})", flush=True)
        got = hm.sre_partial(x, (2.0, 1.0), a0, a1, ctx=ctx).cpu()
        want = hm.sre_rows(x, list(range(a0, a1)), (2.0, 1.0), ctx=ctx).sum(0).cpu()
        assert ((got - want).abs() / want.abs()).max().item() < 1e-12, (a0, a1, got, want)
