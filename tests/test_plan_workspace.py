"""The plan's short chunks never take a shape past a limit that the longest
chunks keep: what fits the library's own scratch with four leading chunks and
chunks of 9 blocks fits it, and what the work list holds with them is planned."""
import pytest

from paper_2606_00024_amd import _lib
from test_abi_host import _opts, _shape, _ws

LIMIT = _lib.STATIC_SCRATCH_BYTES


def _compact_chunks(g, groups, t_cap, block):
    """Chunks per group and the workspace bytes of the compact plan."""
    rec = (g * 128 + 2 * g) * 4
    tpb = block // 64
    buffers = 0 if g >= 8 and tpb == 1 else (3 * 4096 if g >= 8 else 3 * 32 * 288) + 16
    c_max = min(16, (78 * 1024 - buffers) // (2 * rec))
    while c_max > 1 and (c_max + 2) // 3 * tpb > 16:
        c_max -= 1
    c = min(c_max, 9)
    if c >= 3:
        c -= c % 3
    while c > 3 and groups * -(-t_cap // c) < 64:
        c -= 3
    lead, blocks = (4, 3) if c > 3 else (0, c)
    chunks = -(-t_cap // blocks) if t_cap <= lead * blocks else lead + -(-(t_cap - lead * blocks) // c)
    up = lambda x: (x + 255) // 256 * 256
    record = (g * 128 + 2 * g + 63) // 64 * 64
    size = up(8) + up(8 * 32 * 8) + up(8 * groups) + up(8 * groups * chunks) + up(groups * chunks * 2 * record * 4)
    return chunks, size


@pytest.mark.parametrize("forward", [0, 1])
@pytest.mark.parametrize("listed", [False, True])
@pytest.mark.parametrize("g", [1, 2, 4, 8, 16])
def test_scratch_limit_kept(g, listed, forward):
    seen = 0
    for groups in (1, 2, 8, 32, 96, 256, 1000):
        # the longest traversal whose compact plan fits, and lengths around it
        lo, hi = 1, 1 << 18
        while lo < hi:
            mid = (lo + hi + 1) // 2
            lo, hi = (mid, hi) if _compact_chunks(g, groups, mid, 64)[1] <= LIMIT else (lo, mid - 1)
        for t in {max(1, lo - 9), max(1, lo - 1), lo, max(1, int(lo * 0.9)), min(24, lo), min(40, lo)}:
            shape = _shape(batch=groups, num_kv_heads=1, num_q_heads=g, block_size=64, page_size=64,
                           num_pages=1 << 20, max_pages_per_seq=1 if listed else t,
                           max_blocks_per_list=t if listed else 0)
            size, status = _ws(shape, _opts(dense_order=forward))
            assert status == _lib.OK
            assert _compact_chunks(g, groups, t, 64)[1] <= LIMIT and size <= LIMIT, (groups, t, size)
            seen += 1
    assert seen >= 30


@pytest.mark.parametrize("listed", [False, True])
def test_work_list_limit_kept(listed):
    # as many chunks as the queue words hold with the compact plan
    groups = 60000
    t = next(t for t in range(4000, 100, -1)
             if groups * _compact_chunks(4, groups, t, 64)[0] + (1 << 16) < (1 << 24))
    shape = _shape(batch=groups, num_kv_heads=1, num_q_heads=4, block_size=64, page_size=64,
                   num_pages=1 << 20, max_pages_per_seq=1 if listed else t,
                   max_blocks_per_list=t if listed else 0)
    assert _ws(shape, _opts(dense_order=1))[1] == _lib.OK
