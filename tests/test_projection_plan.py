"""The planner of the projection kernel: its rules where they are easy to get
wrong, on the host."""
import pytest

from paper_2606_07665_amd import binding as B

CUS, XCDS = 256, 8


def o_proj_plans(ks, ns, batches):
    for k in ks:
        for n in ns:
            for b in batches:
                if b <= 64 or n % 128 == 0:
                    yield b, k, n, B.o_proj_plan(b, k, n, CUS)


SIZES = ([32, 96, 1024, 2560, 4096, 8192, 65536], [16, 128, 1040, 2560, 4096, 8192, 8320, 32768],
         [1, 4, 16, 17, 32, 33, 48, 64, 65, 100, 129, 160, 200, 256])


def test_every_plan_covers_its_sizes():
    for b, k, n, p in o_proj_plans(*SIZES):
        assert p.col_groups == -(-b // (16 * p.col_tiles))
        assert p.workgroups == -(-n // (16 * p.row_tiles)) * p.col_groups * p.k_splits
        assert 1 <= p.k_splits <= (4 if n <= 8192 else 1)
        assert p.fused == 0


def test_splits_fill_one_round_of_every_xcd():
    """Column groups of a row group share an XCD: a split plan must fit the
    XCD with the most row groups, not only the device."""
    for b, k, n, p in o_proj_plans(*SIZES):
        if p.k_splits > 1 and (p.row_tiles, p.col_tiles) != (1, 1):
            rows = p.workgroups // p.col_groups // p.k_splits
            on_one = -(-rows // XCDS) if p.col_groups > 1 else rows / XCDS
            assert on_one * p.col_groups * p.k_splits <= CUS // XCDS, (b, k, n, p.row_tiles, p.col_tiles, p.k_splits)


@pytest.mark.parametrize("k,n", [(4096, 8192), (8192, 8192), (5120, 8192), (4096, 4096)])
@pytest.mark.parametrize("b", [1, 2, 4, 6, 8, 12, 16])
def test_no_line_at_one_workgroup_per_cu(b, k, n):
    """The estimate moves smoothly with the rows: where two row tiles a
    workgroup (and one or two splits) give every CU exactly one workgroup, the
    sizes next to it get the same plan."""
    near = [B.o_proj_plan(b, k, m, CUS) for m in (n - 32, n)]
    assert len({(p.row_tiles, p.col_tiles, p.k_splits) for p in near}) == 1


@pytest.mark.parametrize("k,n", [(8192, 8192), (4096, 8192), (12288, 8192), (8192, 7936)])
@pytest.mark.parametrize("b", [4, 6, 8, 10])
def test_row_tiles_128_kb_apart(b, k, n):
    """k a multiple of 4096, rows for a round of workgroups of two row tiles,
    or of four with two splits: one row tile a workgroup is faster."""
    p = B.o_proj_plan(b, k, n, CUS)
    assert (p.row_tiles, p.col_tiles, p.k_splits) == (1, 1, 1)


def test_four_row_tiles_of_one_column_tile_are_not_split():
    for b, k, n, p in o_proj_plans(*SIZES):
        assert (p.row_tiles, p.col_tiles) != (4, 1) or p.k_splits == 1, (b, k, n)


# sizes that between them reach every form and ending of the planner (k in odd
# numbers of tiles, hidden sizes and head counts up to the limits)
KS = [96, 160, 224, 288, 544, 800, 1056, 1312, 2080, 2592, 3104, 4128, 5152, 8224, 16416, 65504]
NS = [16, 48, 128, 272, 528, 640, 784, 1024, 1552, 2064, 2432, 3072, 3584, 4112, 4608, 5120, 6656, 7168, 8192, 8208, 9216,
      12288, 14336, 16400, 24576, 32768]
BS = [1, 3, 5, 9, 16, 17, 31, 33, 48, 49, 64, 65, 80, 97, 100, 112, 128, 129, 144, 160, 177, 200, 225, 255, 256]
HEADS = [(1, 1, 64), (2, 1, 64), (2, 2, 128), (5, 5, 64), (8, 2, 128), (8, 4, 128), (12, 4, 64), (12, 4, 256), (16, 4, 128),
         (24, 8, 64), (32, 8, 128), (40, 8, 128), (64, 8, 128), (56, 8, 128), (96, 8, 128), (128, 16, 128), (98, 14, 128),
         (128, 32, 256), (512, 32, 128)]


def test_the_form_tests_leave_no_plan_out():
    """Every (form, ending) the planner reaches on 256 compute units has a case
    of its own in the GPU tests of the forms, whose labels hold."""
    import test_gpu_gemv_forms as forms
    assert [forms.o_proj_name(B, *c[:3]) for c in forms.OPROJ] == [c[3] for c in forms.OPROJ]
    assert [forms.prelude_name(B, *c[:6]) for c in forms.PRELUDE] == [c[6] for c in forms.PRELUDE]
    reached = {}
    for b, k, n, p in o_proj_plans(KS, NS, BS):
        reached.setdefault(forms.name_of(p, "residual"), (b, k, n))
    missing = {f: c for f, c in reached.items() if f not in {c[3] for c in forms.OPROJ}}
    assert not missing, f"o_proj: {missing}"
    preludes = {}
    for b in BS:
        for hq, hkv, d in HEADS:
            if b > 64 and (hq + 2 * hkv) * d % 128:
                continue
            for k in KS:
                for opt in (dict(), dict(qk_norm=True)):
                    preludes.setdefault(forms.prelude_name(B, b, k, hq, hkv, d, opt), (b, k, hq, hkv, d, opt))
    missing = {f: c for f, c in preludes.items() if f not in {c[6] for c in forms.PRELUDE}}
    assert not missing, f"prelude: {missing}"
