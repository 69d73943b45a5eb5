"""The grid-wide barrier of the persistent launches, as the compiler emits it: a
wavefront's stores and atomics have been performed before the workgroup counts
as arrived.  s_barrier does not wait for them, and thread 0's release covers only
what it finds in the L2."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "pf_grid.h"
__global__ void phases(uint32_t *ws, float *stored, unsigned long long *added) {
    const pfk::grid::Barrier bar = pfk::grid::barrier_at(ws, 1000);
    stored[blockIdx.x * blockDim.x + threadIdx.x] = 1.0f;
    __hip_atomic_fetch_add(added + (threadIdx.x & 3), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!pfk::grid::grid_barrier(bar, 1)) return;
    stored[0] = (float)added[threadIdx.x & 3];
}
"""


def test_every_wavefront_waits_before_it_arrives(tmp_path):
    src = tmp_path / "phases.hip"
    src.write_text(SOURCE)
    asm = tmp_path / "phases.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O3", "-std=c++17", "--offload-arch=gfx950",
                    "--cuda-device-only", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1902_05942_amd", "csrc"),
                    "-S", str(src), "-o", str(asm)], check=True, capture_output=True)
    lines = [x.split(";")[0].strip() for x in asm.read_text().splitlines()]
    arrival = lines.index("s_barrier")
    writes = [i for i in range(arrival) if re.match(r"(global|flat)_(store|atomic)", lines[i])]
    assert writes, "the phase's writes come before its barrier"
    waits = [i for i in range(writes[-1], arrival) if re.match(r"s_waitcnt .*vmcnt\(0\)", lines[i])]
    assert waits, lines[writes[-1]:arrival + 1]
