"""Times of a request that is submitted between the worker's clock reading and
its look at the queue: admission and completion are not before submission."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "serve_sim.cpp")
CSRC = os.path.join(ROOT, "paper_1401_6749_amd", "csrc")
INC = os.path.join(ROOT, "include")

PROG = r"""
#define main sim_main
#include "%s"
#undef main
int main(int argc, char **argv)
{
    tm_gauge G{{4, 4, 4, 8}};
    SimDev dev;
    dev.p_create = argc > 1 ? 1.0 : 0.0;
    tm_tsm_params P{};
    P.n_hp = 1;
    P.n_lp = 2;
    P.hp.mode = P.lp.mode = TM_SOLVE_F64;
    P.hp.max_iter = P.lp.max_iter = 100;
    P.batch = 12;
    S_ Q(dev, (char *)(uintptr_t)0x100000000ull, (size_t)1 << 40);
    dev.mem.alloc = [](void *self, size_t n) -> void * { return ((Arena *)self)->alloc(n); };
    dev.mem.free = [](void *self, void *p) { ((Arena *)self)->release(p); };
    dev.mem.self = &Q.arena;
    Req *R = new Req();
    R->G = &G;
    R->P = P;
    Q.submit(R, 2.0);
    Q.step(1.0);  // the worker's clock, read before the submission
    const bool failed = !Q.finished.empty();
    std::printf("%%d %%g %%g %%g\n", (int)failed, R->t_submit, R->t_admit, R->t_done);
    std::fflush(stdout);
    std::_Exit(0);
}
"""


@pytest.mark.parametrize("create_fails", [False, True])
def test_admission_and_completion_not_before_submission(tmp_path, create_fails):
    src, exe = tmp_path / "times.cpp", str(tmp_path / "times")
    src.write_text(PROG % SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, "-I", INC, str(src), "-o", exe, "-lpthread"],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([exe] + ["x"] * create_fails, check=True, capture_output=True, text=True, timeout=60).stdout
    failed, t_submit, t_admit, t_done = (float(v) for v in out.split())
    assert bool(failed) == create_fails
    if create_fails:
        assert t_submit <= t_done
    else:
        assert t_submit <= t_admit
