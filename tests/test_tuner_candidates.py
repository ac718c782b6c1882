"""The plans that the tuner weighs against the planner's own where that one launches steps with a slice per lane."""
import os
import subprocess

import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LANE = -8


def test_whole_row_candidates_are_one_launch_without_workspace(tmp_path):
    """Random problems planned without compiled instances, so that many launch steps with a slice per lane: a whole-row candidate
    launches itself and nothing else, reads X, writes Y and needs no workspace; the planner's own plan has room for what it
    launches, and no launch reads the buffer that it writes."""
    src = tmp_path / "candidates.cpp"
    src.write_text("""
#include "paper_2401_10187_amd/csrc/plan.hpp"
#include <cstdio>
#include <random>
using namespace km;
int main()
{
    const GenericKernel gen{256, 128, 32, 24576, 256, 1024, 512, 96 * 1024, 8, 256, 128, 256};
    std::mt19937 rng(5);
    int lanes = 0, fma_rows = 0, mfma_rows = 0;
    for (int k = 0; k < 20000; ++k) {
        const int n = 2 + rng() % 3;
        int P[4], Q[4];
        for (int i = 0; i < n; ++i) P[i] = 1 + rng() % 48, Q[i] = 1 + rng() % 48;
        Problem pr;
        if (make_problem(300 + rng() % 725, n, P, Q, KM_F32, pr) != KM_OK || pr.k_in > 16384) continue;
        Options opt;
        Plan deflt, spare, fma, mfma;
        opt.kernels = 0x27;                              // (tiled launches, as where the whole-row kernels do not win)
        if (make_plan(pr, opt, nullptr, 0, gen, deflt, spare) != KM_OK) return printf("unplanned\\n"), 1;
        bool lane = false;
        for (const km_plan_step& l : deflt.steps) {
            lane = lane || l.variant == LANE_VARIANT;
            const size_t out = (size_t)(pr.M * l.k_out) * pr.esize;
            if (l.src == l.dst) return printf("buffers\\n"), 1;
            if ((l.dst == KM_BUF_WS0 && deflt.ws0_bytes < out) || (l.dst == KM_BUF_WS1 && deflt.ws1_bytes < out)) return printf("no room\\n"), 1;
        }
        if (!lane) continue;
        ++lanes;
        opt.kernels = 0x37;
        whole_row_candidates(pr, opt, nullptr, 0, gen, deflt, fma, mfma);
        const Plan* rows[2] = {&fma, &mfma};
        for (int which = 0; which < 2; ++which) {
            const Plan& p = *rows[which];
            if (p.steps.empty()) continue;
            ++(which ? mfma_rows : fma_rows);
            const km_plan_step& l = p.steps[0];
            if (p.steps.size() != 1 || l.kernel != KM_KERNEL_ROWS || l.variant != (which ? ROWM_VARIANT : -1) || l.num_factors != n) return printf("other launches\\n"), 1;
            if (l.src != KM_BUF_X || l.dst != KM_BUF_Y || p.ws0_bytes + p.ws1_bytes != 0) return printf("workspace\\n"), 1;
        }
    }
    printf("ok %d %d %d\\n", lanes > 500, fma_rows > 300, mfma_rows > 300);
}
""")
    exe = tmp_path / "candidates"
    subprocess.run(["g++", "-std=c++17", "-I", ROOT, "-o", str(exe), str(src)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True).stdout.strip() == "ok 1 1 1"


def test_a_slice_per_lane_is_timed_for_every_factor_it_can_run(tmp_path):
    """Among the tuner's choices for a single factor, as the step that the planner would make of it; not in fp64, with wishes or without its family."""
    src = tmp_path / "choices.cpp"
    src.write_text("""
#include "paper_2401_10187_amd/csrc/plan.hpp"
#include <cstdio>
#include <cstring>
#include <random>
using namespace km;
int main()
{
    const GenericKernel gen{256, 128, 32, 24576, 256, 1024, 512, 96 * 1024, 8, 256, 128, 256};
    std::mt19937 rng(7);
    int same = 0, more = 0;
    for (int k = 0; k < 20000; ++k) {
        const int n = 1 + rng() % 3;
        int P[3], Q[3];
        for (int i = 0; i < n; ++i) P[i] = 1 + rng() % 90, Q[i] = 1 + rng() % 90;
        Problem pr;
        const bool f32 = rng() % 4 != 0;
        if (make_problem(1 + (int)(rng() >> rng() % 28 >> 4), n, P, Q, f32 ? KM_F32 : KM_F64, pr) != KM_OK) continue;
        Options opt;
        opt.kernels = rng() % 5 ? 0x27 : 0x07;
        opt.tiles_per_wg = rng() % 5 ? 0 : 4;
        Plan plan, spare;
        if (make_plan(pr, opt, nullptr, 0, gen, plan, spare) != KM_OK) return printf("unplanned\\n"), 1;
        std::vector<int64_t> width;
        row_widths(pr, width);
        for (const km_plan_step& st : plan.steps) {
            const int f = st.first_factor;
            std::vector<Choice> cands;
            uncompiled_choices(pr, opt, f, width[f + 1], cands);
            bool timed = false;
            for (const Choice& ch : cands) {
                km_plan_step t = build_step(pr, opt, nullptr, f + 1, 1, ch, width, gen);
                if (t.grid <= 0 || t.block <= 0 || t.lds_bytes < 0 || t.lds_bytes > 160 * 1024) return printf("launch\\n"), 1;
                if (t.variant != LANE_VARIANT) continue;
                timed = true;
                t.src = st.src, t.dst = st.dst;
                if (st.variant == LANE_VARIANT && memcmp(&t, &st, sizeof t) != 0) return printf("another step\\n"), 1;
            }
            if (timed && !(f32 && opt.kernels == 0x27 && opt.tiles_per_wg == 0 && lane_takes(P[f], Q[f]))) return printf("not allowed\\n"), 1;
            if (!timed && st.variant == LANE_VARIANT) return printf("not timed\\n"), 1;
            if (timed) ++(st.variant == LANE_VARIANT ? same : more);
        }
    }
    printf("ok %d %d\\n", same > 1000, more > 1000);
}
""")
    exe = tmp_path / "choices"
    subprocess.run(["g++", "-std=c++17", "-I", ROOT, "-o", str(exe), str(src)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True).stdout.strip() == "ok 1 1"


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes", [(942, [(60, 50), (18, 8)]), (719, [(2, 1), (13, 3), (90, 76), (2, 1)]), (1024, [(24, 1), (60, 23), (5, 9)])], ids=str)
def test_tuned_plans_launch_what_they_have_room_for(M, shapes):
    """Whatever the tuner keeps: every workspace that the planned steps use has a size, and the
    calls with and without a workspace of the caller's agree with the reference (bit for bit on small integers)."""
    import oracle
    P, Q = [p for p, _ in shapes], [q for _, q in shapes]
    X, Fs = kron_inputs.make_problem(M, shapes, "float32", seed=83, x="int2", f="int1")
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    ref = oracle.kron_matmul(X, Fs)
    old = km.get_option(km.KM_OPT_KERNELS)
    try:
        km.set_option(km.KM_OPT_KERNELS, 39)             # the planner's own plan in tiled launches
        assert LANE in [s["variant"] for s in km.plan(M, P, Q, "float32")]
        for kernels in (39, 55):
            km.set_option(km.KM_OPT_KERNELS, kernels)
            before = km.workspace_size(M, P, Q, "float32")
            print("tune M=%d %s kernels %d" % (M, shapes, kernels), flush=True)
            km.tune(M, P, Q, "float32")
            steps = km.plan(M, P, Q, "float32")
            need = km.workspace_size(M, P, Q, "float32")
            assert need <= before
            assert (need > 0) == any(s["dst"] in (km.KM_BUF_WS0, km.KM_BUF_WS1) for s in steps)
            assert all(s["src"] != s["dst"] for s in steps)
            assert np.array_equal(km.kronmatmul(Xd, Fd).cpu().numpy(), ref)
            ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
            Y = torch.empty(ref.shape, device="cuda")
            assert np.array_equal(km.kronmatmul(Xd, Fd, Y=Y, workspace=ws).cpu().numpy(), ref)
    finally:
        km.release()
        km.set_option(km.KM_OPT_KERNELS, old)
