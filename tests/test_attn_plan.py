"""How attention calls are cut up (host code, no GPU): key ranges, rotation,
rows per work-group and the work-groups launched, as the library plans them."""
import pytest

from paper_2608_10519_amd import sparstar as S
from tests.helpers import attn_plan
from tests.test_gpu_parity import INVALID_LIST_CASES, PLAN_CASES


@pytest.fixture(scope="module")
def lib():
    return S.load()


@pytest.mark.parametrize("bh,lq,d,b,stride", [(1, 64, 128, 64, 9), (3, 200, 64, 64, 0), (7, 4420, 128, 128, 9),
                                              (5, 3800, 128, 64, 256), (24, 1000, 64, 128, 0), (35, 200, 64, 64, 0),
                                              (2, 20_001, 128, 64, 40)])
@pytest.mark.parametrize("ws", [False, True])
def test_grid_covers_every_item_once(lib, bh, lq, d, b, stride, ws):
    """The kernel's decode of its work-group id (attn_fwd.hip), over the planned
    grid, gives every (head, range) pair and query group exactly once."""
    p = attn_plan(lib, 1, bh, lq, 64 * 700 + 3, d, b, stride, ws)
    groups, pairs, bits = -(-lq // p.group_rows), bh * p.ranges, p.spread_bits
    n_u = (groups + (1 << bits) - 1) >> bits
    seen = set()
    for block in range(p.grid):
        if bits == 3:
            item = divmod(block, groups)
        else:
            ui, gi = divmod(block // 8, n_u)
            unit = ui * 8 + (block + ui) % 8
            item = unit >> bits, (gi << bits) + (unit & ((1 << bits) - 1))
        if item[0] < pairs and item[1] < groups:
            assert item not in seen
            seen.add(item)
    assert len(seen) == pairs * groups


def test_plan_without_workspace_or_with_few_blocks_is_one_range(lib):
    assert attn_plan(lib, 1, 24, 72_000, 144_512, 128, 64, 571, False).ranges == 1
    assert attn_plan(lib, 1, 24, 72_000, 64 * 15, 128, 64, 0, True).ranges == 1


def test_dense_and_full_lists_take_the_same_ranges(lib):
    for bh, lq, lk, d, b in [(24, 2880, 75_392, 128, 64), (1, 1000, 144_000, 128, 64), (3, 5000, 9000, 64, 128),
                             (2, 300, 24_616, 64, 64)]:
        dense = attn_plan(lib, 1, bh, lq, lk, d, b, 0, True)
        for stride in (-(-lk // b), -(-lk // b) + 50):
            assert attn_plan(lib, 1, bh, lq, lk, d, b, stride, True).ranges == dense.ranges


@pytest.mark.parametrize("bh", [1, 3, 8, 25, 35, 1001])
@pytest.mark.parametrize("lq", [1, 64, 65, 200, 300, 513, 4420])
@pytest.mark.parametrize("b,stride,ws", [(64, 0, False), (64, 9, False), (128, 9, True), (64, 0, True)])
def test_few_empty_work_groups(lib, bh, lq, b, stride, ws):
    """Empty work-groups (past a unit's last group) are at most a sixteenth of the items."""
    p = attn_plan(lib, 1, bh, lq, 64 * 30, 64, b, stride, ws)
    items = bh * p.ranges * -(-lq // p.group_rows)
    assert items <= p.grid <= items + items // 16


def test_many_short_heads_fit_one_launch(lib):
    """An odd number of heads beyond 4 million, one query each: 537 million
    threads in items, well inside the launch limit of 2^32 threads."""
    for stride in (0, 1):
        p = attn_plan(lib, 1, (1 << 22) + 1, 1, 1, 64, 64, stride, False)
        assert p.grid * 2 * p.group_rows < 1 << 32


@pytest.mark.parametrize("case", PLAN_CASES, ids=[c[0] for c in PLAN_CASES])
def test_plans_of_the_gpu_cases(lib, case):
    """The cases that the GPU tests run take the cuts that they are named for."""
    _, heads, lq, lk, d, b, n, ranges, rotated, shared = case
    p = attn_plan(lib, 1, heads, lq, lk, d, b, n, True)
    assert (p.ranges, p.rotation > 0, p.spread_bits > 0) == (ranges, rotated, shared)


@pytest.mark.parametrize("case", INVALID_LIST_CASES, ids=[c[0] for c in INVALID_LIST_CASES])
def test_plans_of_the_gpu_cases_with_invalid_entries(lib, case):
    name, heads, lq, lk, d, b, n, split = case
    p = attn_plan(lib, 1, heads, lq, lk, d, b, n, split)
    assert (p.ranges > 1, p.rotation > 0) == (split, name.startswith("rotated"))


@pytest.mark.parametrize("bh,lq,lk,d,b,stride", [
    (1, 1000, 144_000, 128, 64, 0), (2, 465, 55_727, 64, 64, 0), (2, 199, 57_052, 128, 128, 0),
    (1, 545, 46_955, 64, 128, 143), (2, 170, 189_379, 128, 128, 635), (1, 79, 34_864, 128, 64, 362)])
def test_few_queries_over_many_keys_take_sixteen_ranges(lib, bh, lq, lk, d, b, stride):
    """Fewer work-groups than CUs even at 8 ranges: 16 take little more than half the time."""
    assert attn_plan(lib, 1, bh, lq, lk, d, b, stride, True).ranges == 16


@pytest.mark.parametrize("bh,lq,lk,d,b,stride", [
    (4, 7686, 7226, 128, 128, 7), (5, 2375, 10_097, 128, 64, 9), (6, 2264, 8426, 128, 64, 11), (1, 6160, 3232, 128, 64, 8)])
def test_short_lists_take_one_range(lib, bh, lq, lk, d, b, stride):
    """Lists of a few blocks: the merge of even two ranges costs more than it saves."""
    assert attn_plan(lib, 1, bh, lq, lk, d, b, stride, True).ranges == 1


@pytest.mark.parametrize("bh,lq,bits", [(2, 26_971, 3), (2, 13_000, 2), (8, 6413, 0), (8, 21_332, 2), (24, 72_000, 1)])
def test_sharing_of_pairs_over_xcds(lib, bh, lq, bits):
    """One pass at D = 128, b = 64: two long heads, whose lists may differ, go to every XCD."""
    assert attn_plan(lib, 1, bh, lq, 98_334, 128, 64, 250, False).spread_bits == bits


@pytest.mark.parametrize("lq,lk,rotated", [(72_000, 144_512, True), (11_520, 84_032, True), (640, 84_032, False)])
def test_rows_of_full_width_are_rotated(lib, lq, lk, rotated):
    """Lists may be short in rows that could hold every block (one buffer for
    several budgets): the call is rotated like one with shorter rows."""
    for stride in (-(-lk // 64), -(-lk // 64) + 9):
        p = attn_plan(lib, 1, 24, lq, lk, 128, 64, stride, True)
        assert p.ranges > 1 and (p.rotation > 0) == rotated
    assert attn_plan(lib, 1, 24, lq, lk, 128, 64, 0, True).rotation == 0  # the dense call is not


@pytest.mark.parametrize("heads", [24, 8])
@pytest.mark.parametrize("stride", [1133, 1693, 1806])
def test_large_calls_with_long_lists_keep_their_ranges_in_the_l2(lib, heads, stride):
    """Half of 2,258 key blocks and more: two rotated ranges of 37 MB of K/V lose the L2."""
    p = attn_plan(lib, 1, heads, 72_000, 144_512, 128, 64, stride, True)
    assert p.ranges in (4, 8) and p.rotation > 0
