"""Bounds that the kernels take from csrc/ef_kernels.h, worked out on the host.  No GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2510_26730_amd import build as b

SLICES = r"""
#include <cstdio>
#include "ef_kernels.h"
// every stage whose fragments a wave of the LDS-shared kernels loads: the ring of `depth` stages, then one refill per stage
int main() {
    for (int F = 128; F <= 640; F += 128)
        for (int slices = 1; slices <= 8; ++slices)
            for (int depth = 2; depth <= 3; ++depth) {
                const int n = F / 64;
                int covered = 0;
                for (int s = 0; s < slices; ++s) {
                    const int q0 = ef::shared_slice_begin(n, slices, s), q1 = ef::shared_slice_begin(n, slices, s + 1);
                    const int last = ef::shared_last_stage(q1);
                    if (q0 != covered || q1 < q0) { printf("gap F=%d slices=%d\n", F, slices); return 1; }
                    covered = q1;
                    for (int st = q0; st < q1 + depth; ++st)
                        if (ef::shared_stage_offset(st, last) > 4096u * (n - 1)) {
                            printf("F=%d slices=%d slice %d: offset %u of %d stages\n", F, slices, s, ef::shared_stage_offset(st, last), n);
                            return 1;
                        }
                    for (int st = q0; st < q1; ++st)
                        if (ef::shared_stage_offset(st, last) != 4096u * st) { printf("F=%d stage %d\n", F, st); return 1; }
                }
                if (covered != n) { printf("F=%d slices=%d: %d stages\n", F, slices, covered); return 1; }
                const int kept = ef::ffn_down_shared_slices(F, slices);
                if (kept < 1 || kept > slices || kept > n || (kept < slices && kept != n)) { printf("F=%d kept %d\n", F, kept); return 1; }
            }
    return 0;
}
"""


def test_k_slices_of_the_lds_shared_kernels_stay_inside_their_stages(tmp_path):
    """More K slices than stages included: an empty slice still fills its register ring."""
    if not shutil.which("g++") or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no host compiler or no HIP headers here")
    src, exe = tmp_path / "slices.cpp", tmp_path / "slices"
    src.write_text(SLICES)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", b.CSRC, "-w", "-o", str(exe), str(src)],
                   check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
