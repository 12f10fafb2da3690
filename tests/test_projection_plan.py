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
