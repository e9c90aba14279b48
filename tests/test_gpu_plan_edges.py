"""Work distribution and addressing at the edges of their rules (needs a
gfx950 GPU): numbers of groups around the number of queues, more than 64
groups in a queue, traversals that stop early in most groups (the rest of a
queue is then dropped), lists shorter than their rows and empty ones, and
rows so far apart that the kernel takes 64-bit lane addresses.  Every group
against the oracle."""
from __future__ import annotations

import pytest
import torch

from helpers import random_lists, small_workload
from parity import compare_workload, host_copy
from test_plan_workspace import _compact_chunks
from paper_2606_00024_amd import _lib, api

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _lib.load()
    yield


def _check(wl, host, name, **kw):
    api.decode_workload(wl, **kw)           # leaves the queue words of another call behind
    gpu = api.decode_workload(wl, **kw)
    torch.cuda.synchronize()
    rep = compare_workload(wl, gpu, host=host, name=name, **kw)
    assert not rep.failures, rep.failures[:3]


# (batch, KV heads, heads per group): groups 1, 3, 7, 9, 28 and 65 in each of eight queues
COUNTS = [(1, 1, 4), (3, 1, 8), (7, 1, 2), (3, 3, 4), (7, 4, 1), (65, 8, 4)]


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("lists", [False, True])
@pytest.mark.parametrize("batch,kv_heads,group", COUNTS)
def test_group_counts(batch, kv_heads, group, lists, order):
    lens = tuple((64 * (5 + 7 * b % 23) + 13 * b % 64) if b % 6 != 5 else 0 for b in range(batch))
    wl = small_workload(50 + batch, batch=batch, kv_heads=kv_heads, group=group, seq_len=lens, page_size=32,
                        dense_order=order, device=DEV)
    if lists:
        bl, bll = random_lists(wl, 3, fraction=0.6)
        bll[0] = 0
        wl.block_list, wl.block_list_len = bl.to(DEV), bll.to(DEV)
    host = host_copy(wl)
    for tau, phi, p in ((1e-3, 1e-4, 5), (0.3, 1e-1, 1), (0.0, 1e-4, 5)):
        _check(wl, host, "group_counts", tau=tau, phi=phi, patience=p)


@pytest.mark.parametrize("group", [1, 4, 8, 16])
def test_rows_far_apart(group):
    """Rows of a page 16 MiB apart ([token][page][head][dim]): the instance
    with 64-bit lane addresses gives what the packed layout gives."""
    wl = small_workload(71, batch=2, kv_heads=2, group=group, seq_len=(900, 333), page_size=16, device=DEV)
    pages, heads, slots, dim = wl.k_cache.shape
    far = (1 << 24) // 2

    def spread(t):
        buf = torch.zeros(slots * far, dtype=torch.bfloat16, device=DEV)
        v = buf.as_strided((pages, heads, slots, dim), (heads * dim, dim, far, 1))
        v.copy_(t)
        return v

    host = host_copy(wl)
    kw = dict(tau=1e-3, phi=1e-4, patience=5)
    near = api.decode_workload(wl, **kw)
    wl.k_cache, wl.v_cache = spread(wl.k_cache), spread(wl.v_cache)
    far_out = api.decode_workload(wl, **kw)
    torch.cuda.synchronize()
    rep = compare_workload(wl, far_out, host=host, name="rows_far_apart", **kw)
    assert not rep.failures, rep.failures[:3]
    for a, b in zip(near, far_out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("group", [1, 4, 8])
def test_small_workspace(group):
    """A workspace of the bytes that the longest chunks take, and not a byte
    more: every kind of walk runs in it, one after the other, and leaves what
    lies behind it alone."""
    lens = tuple(64 * 44 - 7 * b for b in range(16))
    wl = small_workload(72, batch=16, kv_heads=4, group=group, seq_len=lens, device=DEV)
    least, tail = _compact_chunks(group, 64, 44, 64)[1], 1 << 16
    buf = api.new_workspace(least + tail, DEV)
    buf[least:] = 0x5A
    lists = random_lists(wl, 5, fraction=0.9)
    host = host_copy(wl)
    ran_short = 0
    for kw in (dict(tau=1e-3, phi=1e-4, patience=5), dict(tau=0.0, phi=1e-4, patience=5)):
        for listed in (False, True):
            wl.block_list, wl.block_list_len = (x.to(DEV) for x in lists) if listed else (None, None)
            host.block_list, host.block_list_len = lists if listed else (None, None)
            for order in (0, 1):
                for off in (False, True):
                    if off and kw["tau"] > 0.0:
                        continue
                    gpu = api.decode_workload(wl, workspace=buf[:least], dense_order=order, no_detector=off, **kw)
                    again = api.decode_workload(wl, dense_order=order, no_detector=off, **kw)
                    torch.cuda.synchronize()
                    ran_short += int(not all(torch.equal(a, b) for a, b in zip(gpu, again)))
                    rep = compare_workload(wl, gpu, host=host, dense_order=order, name="small_workspace", **kw)
                    assert not rep.failures, (order, listed, off, rep.failures[:3])
    assert bool((buf[least:] == 0x5A).all())
    assert ran_short > 0     # (other chunks, other rounding: the two plans did differ)


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("group", [1, 4])
def test_thresholds_that_never_pass(group, order):
    """A launch whose thresholds cannot pass, or whose patience is out of
    reach, may have more workgroups than one whose test just never fires: the
    same bits from all of them."""
    wl = small_workload(73, batch=5, kv_heads=4, group=group, seq_len=(5000, 4099, 64, 0, 3333),
                        dense_order=order, device=DEV)
    blocks = 79
    lists = random_lists(wl, 9, fraction=0.8)
    for listed in (False, True):
        wl.block_list, wl.block_list_len = (x.to(DEV) for x in lists) if listed else (None, None)
        fired = api.decode_workload(wl, tau=1e-30, phi=1e-30, patience=5)
        for kw in (dict(tau=0.0, phi=1e-30, patience=5), dict(tau=1e-30, phi=-1.0, patience=5),
                   dict(tau=0.5, phi=0.5, patience=blocks), dict(tau=0.5, phi=0.5, patience=2 ** 31 - 1)):
            gpu = api.decode_workload(wl, **kw)
            torch.cuda.synchronize()
            for a, b in zip(fired, gpu):
                assert torch.equal(a, b), (listed, kw)
