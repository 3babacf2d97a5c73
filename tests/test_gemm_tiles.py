"""The projections' choice of GEMM tiles (host code, no GPU): the real choice is
built into a small harness and asked for every GEMM of a layer over its range
of rows.

Every choice is a shape that is instantiated for its epilogue.  Where a caller
forces one of tile rows, columns and LDS stages, the other two keep the plain
choice (the largest LDS-ring tile that covers the CUs; 256 x 128
register-staged for the batched value up-projection from 1024 rows), whose
neighbours are instantiated; the shapes chosen for speed alone have none."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "planner", "gemm_harness.cpp")

BF16, F32, SPLIT, F16 = range(4)  # epilogues
# name: N, K, batch, epilogue, fp32 activations, gathered rows
GEMMS = {
    "query / latent": (3072 + 576, 2048, 1, SPLIT, 0, 0),
    "absorption": (512, 128, 16, BF16, 0, 0),
    "values, fp32": (128, 512, 16, BF16, 1, 0),
    "values, bf16": (128, 512, 16, BF16, 0, 0),
    "output, fp32": (2048, 2048, 1, F32, 0, 0),
    "output, bf16": (2048, 2048, 1, BF16, 0, 0),
    "keys and values": (4096, 512, 1, F16, 0, 1),
}
ROWS = sorted({*range(1, 130), *range(131, 1200, 13), 511, 512, 513, 1023, 1024, *range(1200, 12000, 97), 6912, 6913, 1 << 17})
NCU = 256
RING = [(128, 128, 2), (64, 128, 3), (64, 64, 4), (32, 64, 6)]


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(cxx):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("tiles") / "gemm_harness")
    inc = [f"-I{os.path.join(ROOT, 'include')}", f"-I{os.path.join(ROOT, 'paper_2607_02043_amd', 'csrc')}"]
    subprocess.run([cxx, "-O1", "-std=c++17", *inc, SRC, "-o", exe], check=True, capture_output=True)
    return exe


def picks(exe, calls):
    """calls: (M, gemm name, bm, bn, depth); returns (bm, bn, depth, kg) of each."""
    text = "".join(" ".join(map(str, (m, *GEMMS[g], bm, bn, d))) + "\n" for m, g, bm, bn, d in calls)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(calls)
    return [tuple(map(int, line.split())) for line in out]


def plain(M, gemm):
    """The plain choice, before anything forced."""
    N, K, batch, epi, f32, _ = GEMMS[gemm]
    if not f32 and N <= 128 and M >= 1024:
        return 256, 128, 0
    for bm, bn, d in RING:
        if -(-M // bm) * -(-N // bn) * batch >= NCU * 85 // 100:
            break
    return (min(bm, 128), 64, d) if f32 else (bm, bn, d)


@pytest.mark.parametrize("knob,values", [(0, (32, 64, 128, 256)), (1, (64, 128, 256)), (2, (0, 2, 3, 4, 6))])
def test_one_forced_value_keeps_the_plain_choice_of_the_others(harness, knob, values):
    calls, want = [], []
    for g, (N, K, batch, epi, f32, _) in GEMMS.items():
        for m in ROWS:
            for v in values:
                forced = [-1, -1, -1]
                forced[knob] = v
                calls.append((m, g, *forced))
                shape = list(plain(m, g))
                if not (knob == 1 and f32):  # fp32 activations: 64 columns always
                    shape[knob] = v
                want.append((*shape, 1))
    for c, got, w in zip(calls, picks(harness, calls), want):
        assert got == w, c


def test_all_three_forced(harness):
    calls = [(m, g, 128, 128, 3) for g in GEMMS for m in (1, 48, 300, 4160, 8000)]
    for c, got in zip(calls, picks(harness, calls)):
        assert got == (128, 64 if GEMMS[c[1]][4] else 128, 3, 1), c


def kernel_of(gemm, shape):
    """The kernel that computes `gemm` in `shape`, as the library's symbols name it."""
    _, K, _, epi, f32, _ = GEMMS[gemm]
    bm, bn, d, kg = shape
    if d == -1:
        steps, ks = {2048: (8, 8), 512: (2, 8), 128: (4, 1)}[K]
        return f"gemm_skinny_kernel<{bm // 16}, {steps}, {ks}, {'true' if f32 else 'false'}, {epi}>"
    if f32:
        return f"gemm_f32a_kernel<{bm}, {epi}>"
    if d == 0:
        return f"gemm_reg_kernel<{bm}, {bn}, {4 if bm == 256 else 2}, {4 if bn == 256 else 2}, {epi}>"
    return f"gemm_ring_kernel<{bm}, {bn}, {d}, {kg}, {epi}, 2, {4 if bn == 256 else 2}>"


# every shape the tuning values may ask for (rows, columns, stages)
FORCED = [(32, 64, 6), (64, 64, 4), (128, 64, 3), (32, 128, 4), (64, 128, 3), (128, 128, 2), (128, 128, 3),
          (32, 128, 0), (64, 128, 0), (128, 128, 0), (128, 256, 0), (256, 128, 0)]


def test_the_library_holds_the_kernels_that_are_chosen_and_no_others(harness):
    """Kernel names from the symbol table of the library built here."""
    lib = os.path.join(ROOT, "paper_2607_02043_amd", "libmlastep.so")
    if not os.path.exists(lib) or shutil.which("nm") is None:
        pytest.skip("library not built, or no nm")
    symbols = subprocess.run(["nm", "-C", lib], capture_output=True, text=True, check=True).stdout
    built = {line.split("__device_stub__")[1].split("(")[0] for line in symbols.splitlines() if "__device_stub__gemm_" in line}
    calls = [(m, g, -1, -1, -1) for g in GEMMS for m in ROWS]
    chosen = {kernel_of(c[1], p) for c, p in zip(calls, picks(harness, calls))}
    forced = {kernel_of(g, (bm, bn, d, 1)) for g in GEMMS for bm, bn, d in FORCED
              if not (GEMMS[g][3] == F16 and d == 0) and not (GEMMS[g][4] and bm > 128)}
    assert chosen <= built, sorted(chosen - built)
    assert built == chosen | forced, (sorted(built - chosen - forced), sorted(forced - built))
