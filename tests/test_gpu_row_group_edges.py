"""The two-pass row pass by groups of consecutive shifts, on ranges long enough to take it, against the same shifts
one call each (a single shift takes the per-shift row pass, which test_gpu_sre.py holds against the oracle): ranges
that start and end inside groups, on the first shifts and where the top set bit changes, for every row length and
register tile that the groups are built for.

Both form every value by the same operations; only the order of the FP64 sums over shifts may differ: 1e-12."""
import pytest

from synth import states as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# (complex64, n, row bits, row register bits, shifts of the shortest range that goes by groups)
SHAPES = pytest.mark.parametrize("c64,n,row_bits,row_rb,least", [
    (True, 15, 8, 5, 384), (True, 16, 9, 5, 192), (True, 17, 10, 5, 256), (True, 18, 11, 5, 48), (True, 19, 12, 5, 24),
    (True, 20, 13, 5, 24), (True, 14, 7, 4, 768), (True, 15, 8, 4, 384), (True, 16, 9, 4, 192), (True, 17, 10, 4, 256),
    (False, 14, 7, 4, 192), (False, 15, 8, 4, 96), (False, 16, 9, 4, 48), (False, 17, 10, 4, 64), (False, 18, 11, 4, 12),
    (False, 19, 12, 4, 12), (False, 19, 13, 4, 24)])


@SHAPES
def test_ranges_equal_single_shifts(c64, n, row_bits, row_rb, least):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    x = torch.from_numpy(S.gaussian_state(n, seed=8500 + n)).to(torch.complex64 if c64 else torch.complex128).cuda()
    ctx = hm.Context()
    ctx.force_path(2)
    ctx.set_option(hm.OPT_ROW_BITS, row_bits)
    ctx.set_option(hm.OPT_ROW_RB, row_rb)
    top = 2 ** n
    for a0, a1 in ((0, least + 9), (1, least + 8), (3, least + 11), (2 ** row_bits - 5, 2 ** row_bits + least),
                   (top // 2 - 3, top // 2 + least), (top - least - 3, top)):
        print(f"[row group edges] n={n} c64={c64} rows of 2^{row_bits} by 2^{row_rb}: shifts [{a0}, {a1})", flush=True)
        got = hm.sre_partial(x, (2.0, 1.0), a0, a1, ctx=ctx).cpu()
        want = torch.stack([hm.sre_partial(x, (2.0, 1.0), a, a + 1, ctx=ctx) for a in range(a0, a1)]).sum(0).cpu()
        assert ((got - want).abs() / want.abs()).max().item() < 1e-12, (a0, a1, got, want)


@SHAPES
def test_both_stagings_agree(c64, n, row_bits, row_rb, least):
    """HM_OPT_LDS_SPLIT 1 and 2 move the same values through LDS: equal up to the order of the FP64 sums."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_07824_amd as hm
    x = torch.from_numpy(S.gaussian_state(n, seed=8600 + n)).to(torch.complex64 if c64 else torch.complex128).cuda()
    got = []
    for split in (1, 2):
        ctx = hm.Context()
        ctx.force_path(2)
        ctx.set_option(hm.OPT_ROW_BITS, row_bits)
        ctx.set_option(hm.OPT_ROW_RB, row_rb)
        ctx.set_option(hm.OPT_LDS_SPLIT, split)
        print(f"[row group staging] n={n} c64={c64} rows of 2^{row_bits} by 2^{row_rb} split={split}", flush=True)
        got.append(hm.sre_partial(x, (2.0, 1.0), 1, least + 8, ctx=ctx).cpu())
    assert ((got[0] - got[1]).abs() / got[1].abs()).max().item() < 1e-12, got
