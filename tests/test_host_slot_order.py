"""The order of a phase's segments by slot index (csrc/tuna_plan.h, moving_below): the positions of the moving blocks are 0, 1, 2 .. in
ascending slot indices, and the table entries name the same blocks, slots and phases as in message order."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "tuna_plan.h"
using namespace tuna;
int main(int, char** v) {
    const int P = atoi(v[1]), Q = atoi(v[2]), rl = atoi(v[3]), rg = atoi(v[4]);
    for (int fused = 0; fused < 2; ++fused) {
        const PlanHost m = make_plan(P, Q, rl, rg, fused), e = make_plan(P, Q, rl, rg, fused, true, true);
        for (size_t i = 0; i < m.phases.size(); ++i) {
            const PhaseHost &a = m.phases[i], &b = e.phases[i];
            const PhaseScalars ps = phase_scalars(b);
            if (a.nseg != b.nseg || a.zt != b.zt || moving_below(e.sc, ps, P) != b.nseg) return 1;
            std::vector<int> at(P, -1);
            for (int s = 0; s < a.nseg; ++s) at[a.seg[s].e] = s;
            for (int s = 0; s < b.nseg; ++s) {
                const SegInfo& y = b.seg[s];
                if ((s && b.seg[s - 1].e >= y.e) || at[y.e] < 0) return 2;
                const SegInfo& x = a.seg[at[y.e]];
                if (x.z != y.z || x.src_slot != y.src_slot || x.dst_slot != y.dst_slot || x.src_phase != y.src_phase || x.nxt_phase != y.nxt_phase) return 3;
                if (y.src_phase >= 0 && e.phases[y.src_phase].seg[y.src_seg].e != y.e) return 4;
            }
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    folder = tmp_path_factory.mktemp("slot_order")
    (folder / "order.cpp").write_text(PROGRAM)
    out = str(folder / "order")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_02581_amd", "csrc"), "-o", out, str(folder / "order.cpp")],
                   check=True)
    return out


@pytest.mark.parametrize("P,Q", [(2, 2), (7, 7), (64, 64), (100, 100), (343, 343), (96, 16), (120, 8), (60, 2), (60, 30), (1024, 32)])
def test_segments_by_slot_index(program, P, Q):
    for rl in {2, 3, 7, 8, Q}:
        for rg in {2, 5, P // Q} if P > Q else {2}:
            done = subprocess.run([program, str(P), str(Q), str(rl), str(max(rg, 2))])
            assert done.returncode == 0, (rl, rg, done.returncode)
