"""Host arithmetic of launches (no GPU): what a workgroup of the one-launch kernel writes into LDS stays inside what its
launch asks for; workgroups of a pass that goes downwards take every tile once."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2602_13140_amd import binding as qb

HIP_ERROR_INVALID_VALUE = 1
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "qsv_kernels.h"
using namespace qsv;

// Bytes a workgroup of k_forward_small touches: sums of 64 doubles, the matrices, and behind them first the staged
// angles and features, later (several wavefronts) two exchange buffers.
static size_t touched(const CircDev& c, const SmallShape& s, int regs) {
    const size_t mats = 512 + (size_t)s.mat_floats * 4;
    size_t end = mats;
    if (small_has_unitaries(c)) {
        const int rows = c.reupload ? s.rows : 1;
        if ((size_t)rows * c.n_layers * c.n * 32 > (size_t)s.mat_floats * 4) return ~(size_t)0;
        end = mats + (size_t)(small_staged_angles(c) + small_staged_features(c, rows)) * 4;
    }
    if (s.threads > 64 && mats + (size_t)2 * (2 << regs) * s.threads * 4 > end)
        end = mats + (size_t)2 * (2 << regs) * s.threads * 4;
    return end;
}

int main() {
    int checked = 0, bad = 0;
    const long long batches[] = {1, 3, 64, 2048, 2049, 5000, 100000};
    for (int n = 1; n <= kSmallMaxQubits; ++n)
        for (int regs = 2; regs <= 4; ++regs)
            for (int layers = 0; layers <= 512; layers = layers < 4 ? layers + 1 : layers * 2)
                for (int slots = 0; slots <= 4; ++slots)
                    for (int reup = 0; reup <= 1 && reup <= slots && slots - reup <= 3; ++reup)
                        for (long long batch : batches) {
                            const CircDev c{n, layers, reup, slots - reup, {1, 2, 3}};
                            if (n - regs > 8 || small_mats_per_group(c, regs) > kSmallMats) continue;
                            const SmallShape s = small_shape(c, regs, batch);
                            ++checked;
                            // nothing is staged or built for a circuit without unitaries
                            const bool has = layers > 0 && slots > 0;
                            if (small_has_unitaries(c) != has || touched(c, s, regs) > s.lds || s.lds > 65536 || s.rows < 1) {
                                ++bad;
                                std::printf("n %d regs %d layers %d slots %d reupload %d batch %lld: touched %zu of %zu\n", n, regs,
                                            layers, slots, reup, batch, touched(c, s, regs), s.lds);
                            }
                        }
    std::printf("checked %d bad %d\n", checked, bad);
    return bad || checked < 1000;
}
"""


ORDER = r"""
#include <cstdio>
#include <vector>
#include "qsv_kernels.h"
using namespace qsv;
int main() {
    for (int rev = 1; rev <= 2; ++rev)
        for (unsigned tiles = 1; tiles <= 300; ++tiles) {
            std::vector<int> seen(tiles, 0);
            for (unsigned b = 0; b < tiles; ++b) {
                const unsigned t = reversed_tile(b, tiles, rev);
                const bool on_its_xcd = rev == 1 || tiles % 8 != 0 || t % 8 == b % 8;
                if (t >= tiles || seen[t]++ || !on_its_xcd) { std::printf("rev %d tiles %u b %u -> %u\n", rev, tiles, b, t); return 1; }
            }
        }
    return 0;
}
"""


def run(tmp_path, program):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "program.cpp", str(tmp_path / "program")
    src.write_text(program)
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "paper_2602_13140_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                           str(src), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:]


def test_lds_of_the_one_launch_kernel_holds_all_it_writes(tmp_path):
    run(tmp_path, PROGRAM)


def test_a_pass_that_goes_downwards_takes_every_tile_once(tmp_path):
    run(tmp_path, ORDER)


def test_launches_that_would_read_beyond_a_table_are_refused():
    """A table of scalars is read through the execution order, and a sample has at most as many entries as its state.  The
    arguments are looked at before anything is launched, so no device is needed to be refused."""
    lib = qb.load()
    circ = (ctypes.c_int * 7)(3, 1, 0, 1, 2, 0, 0)                # CircDev: 3 qubits, 1 layer, 1 rotation
    some = ctypes.c_void_p(256)
    shifted = lib["_ZN3qsv20launch_build_shiftedERKNS_7CircDevEPKfS4_lPKiPKdiPfP12ihipStream_t"]
    assert shifted(circ, some, None, ctypes.c_long(1), None, some, 3, some, None) == HIP_ERROR_INVALID_VALUE
    encode = lib["_ZN3qsv13launch_encodeEPKflliPdiS2_PfP15HIP_vector_typeIfLj2EEP12ihipStream_t"]
    for n in (3, 8, 13, 16):
        for dim in (0, (1 << n) + 1):
            assert encode(some, ctypes.c_long(1), ctypes.c_long(dim), n, some, 1, some, None, some, None) == HIP_ERROR_INVALID_VALUE
