"""Merge of key-split rows and the append, at the sizes where their code
branches: rows cut into as many parts as one, two or more load rounds take, on
either side of the limits that pick another split of the heads over workgroups;
batches around the 64 requests whose lengths one load round covers.
"""
import numpy as np
import pytest

import oracle
from harness import assert_close, log, run_layer
import paper_2607_02043_amd as mla
from paper_2607_02043_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("parts", [2, 4, 5, 8, 9, 16, 17, 32, 33, 129])
def test_decode_row_of_many_parts(parts):
    """Units of one 32-key tile: a row of 32 * parts keys is cut into `parts`
    partials (and its neighbours into fewer).  The merge weighs fp32 sums in
    fp32: the bar is the parity tests' bar for decode rows, a hundredth of the
    chunk rows' (their probabilities keep 16 bits)."""
    lens = [32 * parts, 1, 33, 32 * (parts // 2 + 1) - 5, 70]
    log(f"[gpu] merge of {parts} parts: contexts {lens}")
    wl = W.custom([n - 1 for n in lens], [1] * len(lens), page_size=32, seed=parts, name=f"{parts} parts")
    li = wl.layer(0)
    mla.debug_set(mla.MLA_DEBUG_DEC_UNIT, 1)
    try:
        g = run_layer(wl.batch, li)
    finally:
        mla.debug_set(mla.MLA_DEBUG_DEC_UNIT, 0)
    _, out_ref, lse_ref = oracle.step(wl.batch, li, W.SOFTMAX_SCALE)
    assert_close(g.out_np(), out_ref, g.lse_np(), lse_ref, what=wl.name, max_abs=1e-4, mean_rel=2e-5)


@pytest.mark.parametrize("chunk", [2, 9, 65])
def test_chunk_rows_of_one_to_five_parts(chunk):
    """64-key ranges over a 200-key prefix: the rows of one block see from
    four to five ranges, some of them only through other rows of the block."""
    log(f"[gpu] chunk of {chunk} rows cut at 64 keys")
    wl = W.custom([200, 40], [chunk, 1], page_size=16, seed=chunk, name=f"chunk {chunk} in 64-key ranges")
    li = wl.layer(0)
    mla.debug_set(mla.MLA_DEBUG_CHUNK_KEYS, 64)
    try:
        g = run_layer(wl.batch, li)
    finally:
        mla.debug_set(mla.MLA_DEBUG_CHUNK_KEYS, 0)
    _, out_ref, lse_ref = oracle.step(wl.batch, li, W.SOFTMAX_SCALE)
    assert_close(g.out_np(), out_ref, g.lse_np(), lse_ref, what=wl.name)


@pytest.mark.parametrize("parts", [2, 4, 5, 9, 16, 17, 33, 70])
@pytest.mark.parametrize("last_longest", [False, True])
def test_chunk_row_of_many_parts(parts, last_longest):
    """64-key ranges: the rows of one chunk are cut into up to `parts` parts,
    beside a chunk of one range, one of two or three, and decode rows, whole or cut
    into one-tile units; the longest chunk first or last (the items of the last
    request then come first)."""
    log(f"[gpu] chunk rows of up to {parts} parts, last_longest={last_longest}")
    reqs = [(64 * parts - 11, 11), (30, 1), (10, 17), (100, 9), (700, 1)]
    if last_longest:
        reqs.reverse()
    wl = W.custom([p for p, _ in reqs], [c for _, c in reqs], page_size=16, seed=parts, name=f"chunk rows of {parts} parts")
    li = wl.layer(0)
    mla.debug_set(mla.MLA_DEBUG_CHUNK_KEYS, 64)
    mla.debug_set(mla.MLA_DEBUG_DEC_UNIT, 1 if parts % 2 else 64)
    try:
        g = run_layer(wl.batch, li, fused=True)
    finally:
        mla.debug_set(mla.MLA_DEBUG_CHUNK_KEYS, 0)
        mla.debug_set(mla.MLA_DEBUG_DEC_UNIT, 0)
    pool_ref, out_ref, lse_ref = oracle.step(wl.batch, li, W.SOFTMAX_SCALE)
    assert np.array_equal(g.pool_np(), pool_ref)
    assert_close(g.out_np(), out_ref, g.lse_np(), lse_ref, what=wl.name)


@pytest.mark.parametrize("reqs", [1, 63, 64, 65, 130])
def test_append_of_many_requests(reqs):
    rng = np.random.default_rng(reqs)
    prefix, rows = rng.integers(0, 50, reqs), rng.integers(1, 4, reqs)
    log(f"[gpu] append, {reqs} requests")
    wl = W.custom(prefix, rows, page_size=8, seed=reqs, name=f"{reqs} requests")
    li = wl.layer(0)
    g = run_layer(wl.batch, li)
    pool_ref, out_ref, lse_ref = oracle.step(wl.batch, li, W.SOFTMAX_SCALE)
    assert np.array_equal(g.pool_np(), pool_ref), "append: pool differs from the oracle"
    assert_close(g.out_np(), out_ref, g.lse_np(), lse_ref, what=wl.name)
