"""The plan's short chunks never take a shape past a limit that the longest
chunks keep: what fits the library's own scratch with four leading chunks and
chunks of 9 blocks fits it, and what the work list holds with them is planned.
One workspace serves every kind of walk over a shape, and the bytes that the
longest chunks take are enough for any."""
import os

import pytest

from paper_2606_00024_amd import _lib
from test_abi_host import _call, _call_static, _opts, _shape, _ws

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


WALKS = [dict(dense_order=order, no_detector=off) for order in (0, 1) for off in (0, 1)]
SHAPES = [(1, 8, 40, 64), (2, 64, 700, 128), (4, 64, 512, 64), (4, 2, 64, 64), (4, 500, 44, 64), (8, 256, 44, 64),
          (8, 256, 900, 64), (16, 32, 300, 256), (4, 3000, 300, 64), (4, 60000, 40, 64), (1, 40000, 3400, 64)]


def _shape_of(g, groups, t, block, listed=0):
    return _shape(batch=groups, num_kv_heads=1, num_q_heads=g, block_size=block, page_size=64, num_pages=1 << 20,
                  max_pages_per_seq=t * block // 64, max_blocks_per_list=listed)


@pytest.mark.parametrize("per_head", [0, 1])
@pytest.mark.parametrize("g,groups,t,block", SHAPES)
def test_one_workspace_per_shape(g, groups, t, block, per_head):
    sizes = {_ws(_shape_of(g, groups, t, block, listed), _opts(dense_order=order, per_head_stop=per_head))
             for listed in (0, 1, t) for order in (0, 1)}
    assert len(sizes) == 1 and sizes.pop()[1] == _lib.OK
    # (without the test there are no per-head stops and no room for them)
    sizes = {_ws(_shape_of(g, groups, t, block), _opts(**walk)) for walk in WALKS}
    assert len(sizes) == 1


@pytest.mark.parametrize("g,groups,t,block", SHAPES)
def test_every_walk_runs_in_the_shape_s_workspace(g, groups, t, block):
    """And in the bytes of the compact plan; under the test, in no fewer."""
    if os.path.exists("/dev/kfd"):
        pytest.skip("a GPU is visible: calls that pass the checks launch with placeholder pointers")
    need = _ws(_shape_of(g, groups, t, block), _opts())[0]
    least = _compact_chunks(g, groups, t, block)[1]
    assert least <= need
    for walk in WALKS:
        for listed in (0, t):
            shape, ptrs = _shape_of(g, groups, t, block, listed), dict(bl=16, bll=16) if listed else None
            for size in (need, least):
                assert _call(shape, _opts(**walk), ptrs, ws_bytes=size) == _lib.ERR_HIP, (walk, listed, size, need, least)
            static = _call_static(shape, _opts(**walk), ptrs)
            if need <= LIMIT:
                assert static == _lib.ERR_HIP
            if not walk["no_detector"]:
                assert _call(shape, _opts(**walk), ptrs, ws_bytes=least - 1) == _lib.ERR_WORKSPACE_TOO_SMALL
                assert static == (_lib.ERR_HIP if least <= LIMIT else _lib.ERR_WORKSPACE_TOO_SMALL)
    assert (need <= LIMIT) == (least <= LIMIT)


def test_full_attention_runs_in_its_own_bytes():
    """Without the test the chunks are longer and there are no leading ones:
    such calls take less than the shape's workspace, the static scratch too."""
    if os.path.exists("/dev/kfd"):
        pytest.skip("a GPU is visible: calls that pass the checks launch with placeholder pointers")
    g, groups, t = 4, 64, 2200
    shape, record = _shape_of(g, groups, t, 64), (g * 128 + 2 * g + 63) // 64 * 64
    chunks = -(-t // 12)
    up = lambda x: (x + 255) // 256 * 256
    own = up(8) + up(8 * 32 * 8) + up(8 * groups) + up(8 * groups * chunks) + up(groups * chunks * 2 * record * 4)
    assert own <= LIMIT < _compact_chunks(g, groups, t, 64)[1]
    off = _opts(no_detector=1)
    assert _call(shape, off, ws_bytes=own) == _lib.ERR_HIP
    assert _call(shape, off, ws_bytes=own - 1) == _lib.ERR_WORKSPACE_TOO_SMALL
    assert _call_static(shape, off) == _lib.ERR_HIP
    assert _call_static(shape, _opts()) == _lib.ERR_WORKSPACE_TOO_SMALL


def test_workspace_of_longer_sequences():
    """Sized for the longest sequences, and used for all shorter ones."""
    if os.path.exists("/dev/kfd"):
        pytest.skip("a GPU is visible: calls that pass the checks launch with placeholder pointers")
    for g, groups, most in ((4, 64, 512), (8, 256, 48), (4, 256, 1024)):
        size = _ws(_shape_of(g, groups, most, 64), _opts())[0]
        for t in range(1, most, max(1, most // 100)):
            for walk in WALKS:
                assert _call(_shape_of(g, groups, t, 64), _opts(**walk), ws_bytes=size) == _lib.ERR_HIP, (g, t, walk)
