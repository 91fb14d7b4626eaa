"""Rules of the timeslice walk on the CPU: chunk shapes, the lattices left to
the register kernel, and walk lengths against measured times."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_6749_amd", "csrc")

PROG = r"""
#include <cstdio>
#include <cstdlib>
#include "tm_launch.h"
using namespace tmk;
int main(int, char **a)
{
    const int dims[4] = {std::atoi(a[1]), std::atoi(a[2]), std::atoi(a[3]), std::atoi(a[4])};
    const int sp = std::atoi(a[5]), n = std::atoi(a[6]), waves = std::atoi(a[7]), beside = std::atoi(a[8]);
    const Geom g = make_geom(dims, -1);
    const WalkPlan p = walk_plan(g, sp);
    std::printf("%d %d %d %d %d %d\n", p.cy, p.cz, p.tiles, p.tiles ? walk_length(g, p, n, sp, waves, beside != 0) : 0,
                (int)register_lattice(p, sp), ntile_of(g, sp));
}
"""
PREC = {"f64": (0, 2), "f32": (1, 3), "f16": (2, 4), "bf16": (3, 4)}  # index, waves per SIMD


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(PROG)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    str(d / "r.cpp"), "-o", str(d / "r")], check=True, capture_output=True, text=True)

    def run(dims, prec, n, beside=0):
        args = [str(v) for v in (*dims, PREC[prec][0], n, PREC[prec][1], beside)]
        return [int(v) for v in subprocess.run([str(d / "r"), *args], check=True, capture_output=True,
                                               text=True).stdout.split()]
    return run


@pytest.mark.parametrize("dims,shape", [((26, 26, 26, 26), (13, 1)), ((14, 14, 14, 28), (14, 2)), ((18, 18, 18, 36), (9, 3)),
                                        ((32, 32, 32, 64), (4, 4)), ((24, 24, 24, 48), (4, 4)), ((16, 16, 16, 32), (8, 4)),
                                        ((10, 30, 26, 14), (15, 2)), ((6, 14, 10, 40), (14, 5))])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_chunk_shapes(rules, dims, shape, prec):
    """Sites that lie close together, and blocks that fill a CU."""
    assert tuple(rules(dims, prec, 1)[:2]) == shape


@pytest.mark.parametrize("dims,register", [((34, 34, 34, 8), ("f64", "f16", "bf16")), ((46, 46, 46, 8), ("f16", "bf16")),
                                           ((102, 22, 22, 8), ()), ((32, 32, 32, 64), ()),
                                           ((34, 34, 2, 2), ()), ((514, 2, 2, 2), ("f64", "f32", "f16", "bf16"))])
def test_register_kernel_lattices(rules, dims, register):
    """Few busy lanes leave a lattice of some size to the register kernel, whose
    sums are per 64 sites."""
    vh = dims[0] * dims[1] * dims[2] * dims[3] // 2
    for prec in PREC:
        _, _, tiles, _, reg, ntile = rules(dims, prec, 1)
        assert bool(reg) == (prec in register), prec
        assert ntile == ((vh + 63) // 64 if reg else tiles)


# (lattice, precision, right-hand sides x parities): microseconds per walk length
MEASURED = [
    ((34, 34, 34, 8), "f32", 24, {1: 754, 2: 695, 4: 690, 8: 745}),
    ((14, 14, 14, 28), "f64", 6, {1: 43.7, 2: 50.5, 4: 54.6, 7: 64.2}),
    ((24, 24, 24, 48), "f64", 12, {1: 1647, 2: 1426, 3: 1374, 4: 1368, 6: 1352, 8: 1418}),
    ((32, 32, 32, 32), "f64", 24, {1: 2213, 2: 1866, 4: 1692, 8: 1625}),
    ((16, 16, 16, 32), "f64", 2, {1: 24.5, 2: 25.7, 4: 36.8, 8: 66.7}),
    ((46, 46, 46, 8), "f64", 3, {1: 569, 2: 558, 4: 585, 8: 676}),
    ((24, 24, 24, 48), "f32", 1, {1: 72.5, 2: 79.1, 3: 73.8, 4: 72.0, 6: 89.0, 8: 98.7}),
    ((32, 32, 32, 32), "f32", 12, {1: 1184, 2: 1003, 4: 897, 8: 927}),
    ((16, 16, 16, 32), "f32", 12, {1: 120, 2: 104, 4: 95.8, 8: 122}),
    ((28, 28, 28, 28), "f16", 3, {1: 117, 2: 114, 4: 135, 7: 140}),
    ((32, 32, 32, 32), "f16", 24, {1: 688, 2: 625, 4: 592, 8: 578}),
    ((24, 24, 24, 48), "f16", 12, {1: 462, 2: 447, 3: 435, 4: 436, 6: 439, 8: 469}),
    ((18, 18, 18, 36), "f16", 12, {1: 148, 2: 145, 3: 142, 4: 156, 6: 155}),
]


@pytest.mark.parametrize("dims,prec,n,times", MEASURED)
def test_walk_length_near_the_fastest(rules, dims, prec, n, times):
    tw = rules(dims, prec, n)[3]
    assert times[tw] <= 1.1 * min(times.values()), (tw, times)


def test_walk_length_beside_another_batch(rules):
    """FP64 at 16^3 x 32: the bulk batch of 12 walks long beside another batch (52.6
    against 53.7 ms for the estimate), four right-hand sides and the other
    precisions as they do alone."""
    dims = (16, 16, 16, 32)
    assert (rules(dims, "f64", 12)[3], rules(dims, "f64", 12, 1)[3]) == (2, 8)
    assert rules(dims, "f64", 4, 1)[3] == rules(dims, "f64", 4)[3] == 2
    for prec in ("f32", "f16"):
        assert rules(dims, prec, 12, 1)[3] == rules(dims, prec, 12)[3]
