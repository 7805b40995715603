"""The index of a deposit log's entry, on the host: the device header's functions, compiled by
hipcc into a host program (no GPU).  A job alone has 32 bits for the staging word, so a run on a
volume of more than 2^26 staging words finds its own job and word again; a launch of several jobs
splits the index into 6 bits and 26, and the rule that lets it log refuses a larger tally."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_13929_amd", "csrc")

PROGRAM = r"""
#include "stage.hpp"
#include <cstdio>
using namespace pmc;

static int check(int nx, int ny, int nz, bool several)
{
    Job J = {};
    J.nx = nx; J.ny = ny; J.nz = nz;
    J.lnx = (nx + 1) / 2; J.lny = (ny + 1) / 2;
    for (int planes = 0; planes < 2; ++planes) {
        const PlaneDims P = plane_dims(nx, ny, nz);
        if (planes && P.words > (1ull << 32)) continue;
        J.stage_planes = planes;
        J.stage_off1 = P.off1; J.stage_off2 = P.off2;
        const uint64_t words = stage_words(J);
        if (!planes && (words > log_words(64)) != !several) { printf("%d x %d x %d: several jobs\n", nx, ny, nz); return 1; }
        if (words > log_words(1)) { printf("%d x %d x %d: one job refused\n", nx, ny, nz); return 1; }
        const int corner[][3] = {{0, 0, 0}, {nx - 1, 0, 0}, {nx - 1, ny - 1, 0}, {nx / 2, ny / 2, nz / 2}, {nx - 1, ny - 1, nz - 1}};
        for (const auto &c : corner)
            for (uint32_t t = 0; t < 3; ++t) {
                const uint32_t w = planes ? plane_index(P, nx, ny, t, c[0], c[1], c[2]) : stage_index(J.lnx, J.lny, c[0], c[1], c[2]);
                const uint64_t v = ((uint64_t)c[2] * ny + c[1]) * nx + c[0];
                if (w >= words || stage_voxel(J, w) != v) { printf("word %u outside the tally\n", w); return 1; }
                const uint32_t e = w | log_tag<false>(0);
                if (log_job<false>(e) != 0u || log_word<false>(e) != w) { printf("one job: word %u lost\n", w); return 1; }
                if (words > log_words(64)) continue;
                for (int32_t job = 0; job < 64; ++job) {
                    const uint32_t m = w | log_tag<true>(job);
                    if (log_job<true>(m) != (uint32_t)job || log_word<true>(m) != w) { printf("job %d: word %u lost\n", job, w); return 1; }
                }
            }
    }
    return 0;
}

int main()
{
    // up to 2^26 words several jobs may log, above only one; the last has 2^32 words in the line layout
    if (check(5, 7, 9, true) || check(256, 256, 256, true) || check(512, 512, 256, true)) return 1;
    if (check(512, 512, 257, false) || check(1024, 1024, 384, false) || check(2048, 2048, 1024, false)) return 1;
    printf("log index: ok\n");
    return 0;
}
"""


def test_log_entries_find_their_job_and_word(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not available")
    src = tmp_path / "index.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "index"
    build = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", f"-I{CSRC}",
                            f"-I{os.path.join(ROOT, 'include')}", str(src), "-o", str(exe)],
                           capture_output=True, text=True, timeout=600)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "log index: ok" in run.stdout
