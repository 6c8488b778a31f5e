"""CG's scalars where a vector pass finishes the reductions before it: every block of such a launch forms the
scalars from the sums, the first stores them while others are still to enter. What a later block decides has
to be the same before and after that store, in a breakdown too, whose flag the next finalize launch raises.
Host build of the formulas that the kernels use (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1306_3159_amd", "csrc")

PROGRAM = r"""
#include "cg_scalars.hpp"
#include <cstdio>
#include <cstring>
using namespace brd;

static int bad = 0;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s (case %d)\n", __LINE__, #x, id); ++bad; } } while (0)

static Scalars state(int iters, int project) {
    Scalars s{};
    s.alpha = 0.7; s.rsum = 1.5; s.qsum = -0.25; s.inv_ncell = 1.0 / 512; s.eBe_inv = 0.125;
    s.rz[iters & 1] = 2.0; s.rz[(iters & 1) ^ 1] = 3.0; s.iters = iters; s.project = project;
    s.step[0] = 0.1; s.step[1] = 0.2;
    return s;
}
template <typename C> static bool same(const C& a, const C& b) {  // NaN results compare by their bits
    return a.bad == b.bad && !std::memcmp(&a, &b, offsetof(C, bad));
}

int main() {
    const double inf = HUGE_VAL, nan = NAN;
    int id = 0;
    for (int iters = 0; iters < 4; ++iters)
        for (int project = 0; project < 2; ++project) {
            // sum z, z.r, z.q; the last with the previous z.r lost, which makes beta non-finite
            const double beta_sums[5][3] = {{1, 2, 3}, {1, nan, 3}, {1, inf, 3}, {1, 2, nan}, {1, 2, 3}};
            for (int k = 0; k < 5; ++k, ++id) {
                const double* t = beta_sums[k];
                Scalars s = state(iters, project);
                if (k == 4) s.rz[(iters & 1) ^ 1] = 0.0;
                const CgBeta first = cg_beta(t[0], t[1], t[2], &s);
                CHECK(cg_dir_runs(&s));
                CHECK(first.bad == (k == 1 || k == 2 || (k > 2 && iters > 0)));
                cg_beta_store(first, &s, true);
                CHECK(cg_dir_runs(&s));  // a block that enters late
                CHECK(same(cg_beta(t[0], t[1], t[2], &s), first));
                CHECK(s.step[0] == 0.1 && s.step[1] == 0.2 && s.iters == iters);
                CHECK(cg_update_runs(&s) == !first.bad);
                CHECK(cg_halted(&s) == first.bad);
                Scalars u = state(iters, project);  // stored by the finalize kernel
                if (k == 4) u.rz[(iters & 1) ^ 1] = 0.0;
                cg_beta_store(first, &u, false);
                CHECK((u.done && u.status) == first.bad && !cg_halted(&u));
                if (first.bad) cg_stop(&s);
                CHECK(s.done == u.done && s.status == u.status && !std::memcmp(&s.beta, &u.beta, 8));
            }
            const double alpha_sums[6][2] = {{4, 1}, {0, 1}, {-1, 1}, {nan, 1}, {inf, 1}, {4, 1}};
            for (int k = 0; k < 6; ++k, ++id) {
                const double* t = alpha_sums[k];
                Scalars s = state(iters, project);
                if (k == 5) s.rz[iters & 1] = nan;
                const CgAlpha first = cg_alpha(t[0], t[1], &s);
                CHECK(cg_update_runs(&s));
                CHECK(first.bad == (k > 0));
                cg_alpha_store(first, t[0], t[1], &s, true);
                CHECK(cg_update_runs(&s));
                CHECK(same(cg_alpha(t[0], t[1], &s), first));
                CHECK(cg_halted(&s) == first.bad);
                CHECK(s.xsteps == (iters & ~1));
                CHECK(s.step[iters & 1] == (first.bad ? (iters & 1 ? 0.2 : 0.1) : first.alpha));
                Scalars u = state(iters, project);
                if (k == 5) u.rz[iters & 1] = nan;
                cg_alpha_store(first, t[0], t[1], &u, false);
                CHECK((u.done && u.status) == first.bad && !cg_halted(&u));
                if (first.bad) cg_stop(&s);
                CHECK(s.done == u.done && s.status == u.status && s.alpha == u.alpha);
            }
        }
    std::printf("%d cases, %d faults\n", id, bad);
    return bad != 0;
}
"""


def test_late_blocks_decide_as_the_first(tmp_path):
    src = tmp_path / "cg_scalars.cpp"
    src.write_text("#include <cstddef>\n" + PROGRAM)
    exe = str(tmp_path / "cg_scalars")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wno-unknown-pragmas", "-I", CSRC,
                        str(src), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
