"""Chunk lengths around the resolver's gangs of blocks (needs a gfx950 GPU).

The resolver takes a chunk's blocks several at a time and keeps one block per
lane of a row of 16 lanes, so that chunks of up to 16 blocks fit a row
exactly.  Groups of one and two heads hold chunks of 13 to 16 blocks, full and
cut short by the traversal's end, against the oracle; and a traversal whose
last block's output is infinite keeps the infinity, whatever the number of
blocks left over in the last chunk."""
from __future__ import annotations

import math

import pytest
import torch

from helpers import random_lists, small_workload
from parity import compare_per_head, compare_workload, host_copy
from paper_2606_00024_amd import _lib, api

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _lib.load()
    yield


@pytest.mark.parametrize("chunk", [13, 14, 15, 16])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("group", [1, 2])
def test_chunks_that_fill_a_row(group, block, chunk):
    lens = tuple(block * t - cut for t, cut in ((16, 0), (17, 5), (32, 0), (45, 1), (16 * 3, 63)))
    wl = small_workload(300 + chunk, batch=len(lens), kv_heads=2, group=group, seq_len=lens,
                        block_size=block, page_size=32, needles=2, device=DEV)
    lists = random_lists(wl, 300 + chunk, fraction=0.7)
    host = host_copy(wl)
    for tau, phi, p in ((0.0, 1e-4, 5), (1e-3, 1e-4, 5), (0.05, 1e-3, 2)):
        kw = dict(tau=tau, phi=phi, patience=p)
        print(f"  gpu call: g={group} block={block} chunk={chunk} {kw}", flush=True)
        rep = compare_workload(wl, api.decode_workload(wl, chunk_blocks=chunk, **kw), host=host,
                               name="chunks_of_16", **kw)
        assert rep.ok(), str(rep)
        rep = compare_per_head(wl, api.decode_workload(wl, chunk_blocks=chunk, per_head_stop=True, **kw),
                               host=host, name="chunks_of_16_per_head", **kw)
        assert rep.ok(), str(rep)
    # without the test: the whole traversal, as if no step were ever stable
    off = dict(tau=0.0, phi=1e-4, patience=5)
    rep = compare_workload(wl, api.decode_workload(wl, chunk_blocks=chunk, no_detector=True, **off), host=host,
                           name="chunks_of_16", **off)
    assert rep.ok(), str(rep)
    wl.block_list, wl.block_list_len = (x.to(DEV) for x in lists)
    host.block_list, host.block_list_len = lists
    rep = compare_workload(wl, api.decode_workload(wl, chunk_blocks=chunk, **off), host=host,
                           name="chunks_of_16", **off)
    assert rep.ok(), str(rep)


@pytest.mark.parametrize("blocks", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("group", [1, 4, 8, 16])
def test_infinite_last_block(group, blocks):
    """Equal keys, so that a block's sum of 64 values of 3e38 leaves fp32's
    range: its output is +inf, and so is the mean after it."""
    wl = small_workload(7, batch=1, kv_heads=1, group=group, seq_len=64 * blocks, dense_order=1, device=DEV)
    wl.k_cache.zero_()
    wl.v_cache.fill_(1.0)
    wl.v_cache[int(wl.page_table[0, blocks - 1])] = 3e38
    for no_detector in (False, True):
        out, lse, stop = api.decode_workload(wl, tau=0.0, phi=1e-4, patience=5, no_detector=no_detector,
                                             chunk_blocks=5)
        torch.cuda.synchronize()
        assert bool(torch.isposinf(out).all()), (no_detector, out[0, 0, :4])
        assert torch.allclose(lse, torch.full_like(lse, math.log(64 * blocks)), atol=1e-5)
        assert bool((stop == blocks).all())
