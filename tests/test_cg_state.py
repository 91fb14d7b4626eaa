"""Scalar steps of a CG slot on the CPU.  alpha is formed beside the blocks of a
Dslash that read the slot's status, so forming it leaves the status alone; a
curvature that breaks down ends the slot at the end of the iteration, without
a step."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_6749_amd", "csrc")

# lane 0 of the wave that forms alpha, on one partial sum
PROG = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "tm_types.h"
using namespace tmk;
#define __device__
#define __forceinline__ inline
static struct { unsigned x; } threadIdx;
static double wave_sum(double v) { return v; }
%s
int main(int, char **argv)
{
    SlotState S{};
    S.status = ST_RUNNING;
    S.max_iter = 9;
    S.rr = S.rr0 = S.rr_new = 2.0;
    const double pap = std::atof(argv[1]);
    cg_alpha_wave(S, &pap, 1);
    std::printf("%%d %%g %%d", S.status, S.alpha, S.xpend);
#ifdef TM_HD
    std::printf(" %%d", (int)cg_steps(S));
    cg_beta(S, 0.5);
    std::printf(" %%d %%d %%g", S.status, S.iter, S.rr);
#endif
    std::printf("\n");
}
"""


def _run(tmp_path, pap):
    dev = open(os.path.join(CSRC, "tm_dev.h")).read()
    parts = re.findall(r"^__device__ __forceinline__ bool finite_pos.*$", dev, re.M)
    parts += re.findall(r"^__device__ __forceinline__ void cg_alpha_wave.*?^}$", dev, re.M | re.S)
    src, exe = tmp_path / "cg.cpp", str(tmp_path / "cg")
    src.write_text(PROG % "\n".join(parts))
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wno-unknown-pragmas", "-I", CSRC, str(src), "-o", exe], check=True,
                   capture_output=True, text=True)
    return [float(v) for v in subprocess.run([exe, pap], check=True, capture_output=True, text=True).stdout.split()]


RUNNING, NUMERIC = 1, 5


@pytest.mark.parametrize("pap", ["0", "-3", "nan", "inf", "2e300"])
def test_breakdown_ends_the_slot_after_the_iteration(tmp_path, pap):
    status, alpha, xpend, *rest = _run(tmp_path, pap)
    assert (status, alpha, xpend) == (RUNNING, 0.0, 0)
    assert rest == [0, NUMERIC, 0, 2.0]


def test_step_goes_on(tmp_path):
    assert _run(tmp_path, "4") == [RUNNING, 0.5, 1, 1, RUNNING, 1, 0.5]
