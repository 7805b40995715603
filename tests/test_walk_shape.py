"""What the walk makes of a launch shape, on the host: the internal header's function, compiled by
hipcc into a host program (no GPU).  Wavefronts that are full wait for as many lanes as the caller
says, over the whole range of `defer`; only those with fewer photons than lanes wait less."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_13929_amd", "csrc")

PROGRAM = r"""
#include "internal.hpp"
#include <cstdio>
using namespace pmc::host;

int main()
{
    const uint64_t waves = 4096;
    for (int defer = 1; defer <= 64; ++defer) {
        const mc_tune t = {256, 16, 256, 32, defer};
        for (const uint64_t n : {waves * 64, waves * 1000, (uint64_t)1 << 32}) {
            const WalkShape s = walk_shape(t, waves, n);
            if (s.cap != 64 || s.refill != 32 || s.defer != defer || s.chunk > 256 || (uint64_t)s.chunk > n / waves) {
                printf("full wavefronts: defer %d became %d\n", defer, s.defer);
                return 1;
            }
        }
        for (const uint64_t n : {(uint64_t)1, waves, waves * 16, waves * 63}) {
            const WalkShape s = walk_shape(t, waves, n);
            const int share = (int)((n + waves - 1) / waves), most = share / 8 > 1 ? share / 8 : 1;
            if (s.cap != share || s.chunk != share || s.refill > share || s.defer != (defer < most ? defer : most)) {
                printf("%d lanes: defer %d became %d\n", share, defer, s.defer);
                return 1;
            }
        }
    }
    printf("walk shape: ok\n");
    return 0;
}
"""


def test_full_wavefronts_keep_the_callers_defer(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not available")
    src = tmp_path / "shape.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "shape"
    build = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", f"-I{CSRC}",
                            f"-I{os.path.join(ROOT, 'include')}", str(src), "-o", str(exe)],
                           capture_output=True, text=True, timeout=600)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "walk shape: ok" in run.stdout
