"""Batches of many requests, at the counts where the kernels' lookups branch: 64
requests are found in one step of one length a lane, more in steps of 256.
Decode rows and a few chunks in random order, with the plan's own work items and
with rows cut into as many parts as possible (one-tile decode units, 64-key
ranges: the merge looks its rows up too), against the oracle."""
import numpy as np
import pytest

import oracle
from harness import assert_close, log, run_layer
import paper_2607_02043_amd as mla
from paper_2607_02043_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cut", [False, True])
@pytest.mark.parametrize("reqs", [63, 64, 65, 255, 256, 257, 320, 512, 513, 1030])
def test_many_requests(reqs, cut):
    rng = np.random.default_rng(reqs)
    rows = np.ones(reqs, dtype=np.int64)
    prefix = rng.integers(0, 150, reqs)
    # chunks anywhere, one of them the last or the first request of a step
    for r in {0, reqs - 1, *rng.integers(0, reqs, 4).tolist(), min(reqs - 1, 255), min(reqs - 1, 256)}:
        rows[r] = rng.integers(2, 20)
        prefix[r] = rng.integers(0, 400)
    prefix[rng.integers(0, reqs, 3)] = rng.integers(900, 2000, 3)
    log(f"[gpu] {reqs} requests, {int((rows > 1).sum())} chunks, cut={cut}")
    wl = W.custom(prefix, rows, page_size=16, seed=reqs, name=f"{reqs} requests")
    li = wl.layer(0)
    if cut:
        mla.debug_set(mla.MLA_DEBUG_DEC_UNIT, 1)
        mla.debug_set(mla.MLA_DEBUG_CHUNK_KEYS, 64)
    try:
        g = run_layer(wl.batch, li, fused=True)
    finally:
        mla.debug_set(mla.MLA_DEBUG_DEC_UNIT, 0)
        mla.debug_set(mla.MLA_DEBUG_CHUNK_KEYS, 0)
    pool_ref, out_ref, lse_ref = oracle.step(wl.batch, li, W.SOFTMAX_SCALE)
    assert np.array_equal(g.pool_np(), pool_ref), "append: pool differs from the oracle"
    assert_close(g.out_np(), out_ref, g.lse_np(), lse_ref, what=wl.name)
