"""The attention kernels as the compiler lays them out (host code, no GPU): the
library's own source and flags, compiled to assembly.

* No kernel uses scratch memory: a spilled register costs the chunk tiles a
  round trip behind every DMA in flight.
* In the prologue of a chunk item nothing waits between the DMAs of its second
  tile and the first scores, so that they stay in flight across the barrier.
  (The DMAs are inline assembly, which the compiler does not count: a wait that
  it places for an earlier load covers them too.)
* The wait for the item's page ids leaves the query loads in flight."""
import os
import re
import subprocess

import pytest

from paper_2607_02043_amd import build

QUERY_LOADS = 18  # operands of 32 dims


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("asm") / "mla_kernels.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, *flags, "-fPIC", "--offload-device-only", "-S", os.path.join(build.CSRC, "mla_kernels.hip"), "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_no_scratch(asm):
    sizes = dict(re.findall(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", asm))
    assert len(sizes) >= 4 and any("attention_kernel" in k for k in sizes), sorted(sizes)
    assert not [k for k, v in sizes.items() if int(v) != 0], sizes


def _prologue(asm):
    """(kind, text) of the loads, waits and barriers from a chunk item's query
    loads to its first matrix instruction."""
    body = asm[re.search(r"^_ZN\S*attention_kernel\S*:", asm, re.M).start():]
    body = body[:body.index(".Lfunc_end")]
    events = []
    for line in body.splitlines():
        op = line.split(";")[0].split()
        if not op:
            continue
        if op[0] == "global_load_dwordx4":
            events.append(("query", line))
        elif op[0] == "global_load_lds_dwordx4":
            events.append(("dma", line))
        elif op[0] == "s_waitcnt" and "vmcnt" in line:
            events.append(("wait", re.search(r"vmcnt\((\d+)\)", line).group(1)))
        elif op[0] == "s_barrier":
            events.append(("barrier", ""))
        elif op[0] == "ds_write_b32":
            events.append(("page ids", ""))
        elif op[0].startswith("v_mfma"):
            events.append(("mfma", ""))
    kinds = [k for k, _ in events]
    first = next(i for i in range(len(kinds)) if kinds[i:i + QUERY_LOADS] == ["query"] * QUERY_LOADS)
    return events[first + QUERY_LOADS:first + kinds[first:].index("mfma")]


def test_page_ids_do_not_wait_for_the_queries(asm):
    events = _prologue(asm)
    waits = [v for k, v in events[:events.index(("barrier", ""))] if k == "wait"]
    assert waits and all(int(v) >= QUERY_LOADS for v in waits), waits


def test_second_tile_stays_in_flight(asm):
    kinds = [k for k, _ in _prologue(asm)]
    # page window barrier, tile 0 (two forms of nine rounds), the waits, tile 1, barrier
    assert kinds.count("dma") == 36 and kinds.count("barrier") == 2
    last_dma = len(kinds) - 1 - kinds[::-1].index("dma")
    assert "wait" not in kinds[last_dma:], kinds[last_dma:]
    waits = [i for i, k in enumerate(kinds) if k == "wait"]
    assert kinds[:waits[-1]].count("dma") == 18, "tile 1 is issued before the last wait"
