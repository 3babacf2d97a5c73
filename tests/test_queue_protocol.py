"""The attention launch's work protocol, modelled on the host over the library's
own index functions (compiled from the header): G persistent workgroups, each
with a first item fixed by its index, then two atomic counters (chunk items,
decode items) that deal out what is left from the end of the fixed ones, and a
count of finished workgroups.  A launch with no more items than workgroups makes
no atomic operation: every workgroup leaves after its first item.  Otherwise a
workgroup goes on with the queue its first item came from, tries the other one
once when its own is empty, and leaves when both are; the last one to leave zeroes
the counters.  Under random interleavings of the atomic operations every item is
taken exactly once, every workgroup leaves, and the counters end at zero (the
loop of attention_kernel)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "mla_kernels.h"
extern "C" int first_chunk_items(int nc, int nd, int D, int G) { return mla::first_chunk_items(nc, nd, D, G); }
extern "C" int first_item(int nc, int nd, int D, int G, int b) { return mla::first_item(nc, nd, D, G, b); }
"""


@pytest.fixture(scope="module")
def index(tmp_path_factory):
    cxx = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(cxx):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("queue")
    (d / "index.cpp").write_text(SOURCE)
    subprocess.run([cxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "paper_2607_02043_amd", "csrc"),
                    str(d / "index.cpp"), "-o", str(d / "index.so")], check=True, capture_output=True)
    return ctypes.CDLL(str(d / "index.so"))


def run_protocol(index, G, n_chunk, n_dec, first, rng):
    work = [0, 0, 0]  # next chunk item, workgroups done, next decode item
    taken, atomics = [], [0]

    # each workgroup is a generator yielding before each atomic operation
    def wg(b):
        it = index.first_item(n_chunk, n_dec, first, G, b)
        on_dec = it >= n_chunk
        while True:
            taken.append((b, it))
            if n_chunk + n_dec <= G:
                return
            fixed_chunk = index.first_chunk_items(n_chunk, n_dec, first, G)
            it = -1
            for _ in range(2):
                yield
                atomics[0] += 1
                if on_dec:
                    d = G - fixed_chunk + work[2]; work[2] += 1
                    if d < n_dec:
                        it = n_chunk + d
                else:
                    c = fixed_chunk + work[0]; work[0] += 1
                    if c < n_chunk:
                        it = c
                if it >= 0:
                    break
                on_dec = not on_dec
            if it < 0:
                break
        yield
        atomics[0] += 1
        done = work[1]; work[1] += 1
        if done == G - 1:
            assert len(live) == 1, "a workgroup still runs when the counters are zeroed"
            work[0] = work[1] = work[2] = 0

    live = {b: wg(b) for b in range(G)}
    steps = 0
    while live:
        b = list(live)[rng.integers(len(live))]
        try:
            next(live[b])
        except StopIteration:
            del live[b]
        steps += 1
        assert steps < 100 * (G + n_chunk + n_dec) + 1000, "a workgroup never leaves"
    return taken, work, atomics[0]


@pytest.mark.parametrize("seed", range(40))
def test_every_item_once_and_counters_zeroed(index, seed):
    rng = np.random.default_rng(seed)
    n_chunk, n_dec = int(rng.integers(0, 30)), int(rng.integers(0, 30))
    n_dec = max(n_dec, 1 - n_chunk)
    G = int(rng.integers(1, min(12, n_chunk + n_dec) + 1))  # never more workgroups than items
    first = int(rng.integers(0, G + 1))
    taken, work, _ = run_protocol(index, G, n_chunk, n_dec, first, rng)
    assert sorted(it for _, it in taken) == list(range(n_chunk + n_dec))
    assert work == [0, 0, 0]


@pytest.mark.parametrize("n_chunk,n_dec,first", [(7, 0, 0), (0, 7, 0), (0, 1, 1), (4, 3, 2), (1, 6, 7), (5, 2, 6)])
def test_no_more_items_than_workgroups_takes_no_atomic(index, n_chunk, n_dec, first):
    rng = np.random.default_rng(n_chunk)
    G = n_chunk + n_dec
    taken, work, atomics = run_protocol(index, G, n_chunk, n_dec, min(first, G), rng)
    assert sorted(taken) == [(b, index.first_item(n_chunk, n_dec, min(first, G), G, b)) for b in range(G)]
    assert sorted(it for _, it in taken) == list(range(G)) and work == [0, 0, 0] and atomics == 0


def test_decode_first_workgroups_start_on_decode(index):
    # with items to spare, each decode-first workgroup's first item is a decode item
    rng = np.random.default_rng(5)
    taken, _, _ = run_protocol(index, 6, 40, 40, 3, rng)
    first_item = {}
    for b, it in taken:
        first_item.setdefault(b, it)
    assert all((first_item[b] >= 40) == (b < 3) for b in first_item)
