"""The run-time-shape MFMA kernel with a slice per lane (variant -8 of kronmatmul_plan)."""
import os
import subprocess

import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LANE, PAD = -8, -3


@pytest.fixture(autouse=True)
def no_whole_row_kernels():
    """Many of the rows here are short enough for one launch; these tests are about the tiled ones."""
    old = km.get_option(km.KM_OPT_KERNELS)
    km.set_option(km.KM_OPT_KERNELS, 39)
    yield
    km.set_option(km.KM_OPT_KERNELS, old)


def _shapes(S, P, Q):
    """Rows of S slices of P elements: the last factor, P x Q, is applied first, the one before it then sums up the slices."""
    return [(S, 1), (P, Q)]


def _first(M, shapes, dtype="float32"):
    return km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)[0]


# (rows, slices of a row, P, Q): every pair of chunk length (2 to 7, 9 and 13 vectors) and groups of four columns (1 to 32) that a launch
# can have, at the smallest size that takes the kernel, with 0 to 3 elements left over of slices and columns, rows of 16 slices (several to a tile), of no
# multiple of 64 and of whole tiles, a ragged last tile
CASES = [
    (1001, 131, 5, 1), (993, 132, 7, 6), (986, 133, 5, 9), (957, 137, 5, 16), (247, 133, 8, 17), (99, 331, 7, 22), (97, 338, 5, 27), (97, 338, 5, 30),
    (125, 263, 7, 33), (125, 263, 6, 40), (99, 331, 6, 41), (96, 342, 5, 46), (125, 263, 6, 49), (125, 263, 5, 56), (125, 263, 5, 59),
    (125, 263, 5, 62), (125, 263, 5, 65), (125, 264, 5, 69), (128, 258, 5, 75), (128, 258, 5, 78), (126, 262, 6, 81), (126, 261, 5, 87),
    (126, 262, 5, 91), (126, 262, 5, 94), (127, 259, 6, 99), (126, 261, 6, 104), (126, 261, 6, 107), (126, 261, 6, 110), (99, 333, 5, 114),
    (126, 261, 5, 120), (126, 261, 5, 123), (126, 261, 5, 126), (1725, 19, 9, 1), (964, 17, 10, 8), (17166, 67, 10, 11), (15248, 66, 9, 15),
    (911, 18, 9, 17), (10608, 69, 9, 24), (9347, 68, 11, 27), (8664, 68, 12, 29), (8073, 68, 11, 33), (6933, 67, 12, 40), (1639, 20, 14, 3),
    (820, 20, 13, 5), (603751, 1, 31, 9), (13762, 65, 13, 14), (9720, 71, 16, 19), (6636, 70, 30, 22), (9347, 68, 13, 25), (7802, 72, 14, 29),
    (4939, 73, 32, 35), (6933, 67, 14, 38), (1561, 21, 20, 1), (911, 18, 17, 8), (205, 80, 17, 9), (1928, 17, 37, 14), (911, 18, 17, 17),
    (8446, 65, 20, 24), (8133, 66, 18, 27), (7469, 66, 18, 31), (7176, 66, 18, 33), (6299, 65, 19, 40), (1561, 21, 21, 3), (863, 19, 24, 7),
    (1725, 19, 42, 11), (1725, 19, 45, 14), (99, 331, 116, 19), (1725, 19, 118, 22), (1928, 17, 120, 25), (1561, 21, 85, 32), (129, 256, 117, 35),
    (96, 342, 119, 38), (129, 256, 96, 41), (99, 332, 113, 48), (464, 337, 88, 67), (236, 625, 96, 69), (452, 331, 88, 74), (997, 263, 96, 80),
    (1928, 17, 25, 3), (964, 17, 25, 6), (1725, 19, 55, 11), (1725, 19, 74, 14), (1928, 17, 112, 19), (437, 75, 74, 22), (1725, 19, 76, 25),
    (1821, 18, 77, 32), (97, 338, 111, 35), (126, 261, 109, 38), (98, 335, 111, 41), (126, 261, 112, 48), (2415, 69, 78, 67), (486, 332, 80, 70),
    (483, 332, 76, 75), (462, 336, 76, 80), (863, 19, 101, 3), (1725, 19, 62, 6), (1639, 20, 36, 9), (1821, 18, 70, 13), (1639, 20, 123, 17),
    (1928, 17, 106, 22), (99, 331, 103, 27), (1639, 20, 102, 30), (127, 259, 127, 35), (127, 259, 97, 38), (97, 338, 99, 41), (127, 259, 100, 48),
    (2632, 67, 70, 67), (168, 1024, 72, 70), (359, 334, 128, 74), (352, 333, 128, 79), (1725, 19, 50, 7), (1928, 17, 51, 10), (1821, 18, 50, 13),
    # from the form with the factor in registers: rows of one slice, of a few, of part of a tile, of many; one tile to a wavefront and two
    (712000, 1, 27, 7), (206400, 3, 31, 8), (64000, 11, 30, 7), (41200, 17, 31, 8), (70500, 30, 27, 20), (3600, 330, 9, 13), (1150, 330, 33, 33), (1200, 625, 17, 17), (1100, 530, 21, 21),
    (900, 400, 30, 40), (300, 629, 65, 66), (330, 512, 71, 76), (136, 1333, 68, 68),
]


@pytest.mark.parametrize("M,S,P,Q", CASES)
def test_the_list_takes_the_kernel_and_its_launches_fit(M, S, P, Q):
    st = _first(M, _shapes(S, P, Q))
    assert st["variant"] == LANE and st["kernel"] == km.KM_KERNEL_MFMA_ANY
    assert st["block"] == 256 and st["grid"] % 8 == 0 and st["lds_bytes"] <= 160 * 1024
    assert 256 * (st["grid"] - 8) < M * S <= 2 * 256 * st["grid"]           # four tiles of 64 slices, once or twice


def _run(tmp_path, body):
    src, exe = tmp_path / "prog.cpp", tmp_path / "prog"
    src.write_text('#include "paper_2401_10187_amd/csrc/plan.hpp"\n#include <cstdio>\n#include <random>\nusing namespace km;\n' + body)
    subprocess.run(["g++", "-std=c++17", "-I", ROOT, "-o", str(exe), str(src)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True).stdout.strip()


def test_the_list_covers_every_compiled_kernel(tmp_path):
    """The pairs of chunk length and column groups that launch_lane.hpp instantiates are those of CASES."""
    out = _run(tmp_path, """
int main()
{
    for (int U : {2, 3, 4, 5, 6, 7, 9, 13})
        for (int G = 1; G <= 32; ++G)
            if (lane_compiled(G, U)) printf("%d,%d ", U, G);
    printf("|");
    for (int P = LANE_MINP; P <= LANE_MAXP; ++P) printf(" %d", lane_units(P));
}
""")
    compiled, units = [half.split() for half in out.split("|")]
    assert {"%s,%d" % (units[P - 5], (Q + 3) // 4) for _, _, P, Q in CASES} == set(compiled) and len(compiled) > 100


def test_what_the_rule_takes_is_compiled(tmp_path):
    """Random problems, any families of kernels: a step that the rule would give to this kernel is of a shape that it is compiled for, so the limits
    of shapes stand in one place only."""
    assert _run(tmp_path, """
int main()
{
    const GenericKernel gen{256, 128, 32, 24576, 256, 1024, 512, 96 * 1024, 8, 256, 128, 256};
    std::mt19937 rng(17);
    int wins = 0;
    for (int k = 0; k < 60000; ++k) {
        const int n = 1 + rng() % 4;
        int P[4], Q[4];
        for (int i = 0; i < n; ++i) P[i] = 1 + rng() % (rng() % 2 ? 40 : 130), Q[i] = 1 + rng() % (rng() % 2 ? 40 : 130);
        Problem pr;
        if (make_problem(1 + (int)(rng() >> rng() % 30 >> 2), n, P, Q, KM_F32, pr) != KM_OK || (double)pr.M * (double)pr.k_in > 1e9) continue;
        Options opt;
        opt.kernels = rng() % 2 ? 0x27 : 0x21;
        opt.prefer_threads = 1;                          // (a wish: the plan without this kernel)
        Plan plan, spare;
        if (make_plan(pr, opt, nullptr, 0, gen, plan, spare) != KM_OK) return printf("unplanned"), 1;
        for (size_t i = 0; i < plan.steps.size(); ++i) {
            const int p = pr.P[plan.steps[i].first_factor], q = pr.Q[plan.steps[i].first_factor];
            if (p < LANE_MINP || p > LANE_MAXP || q > LANE_MAXP || (plan.steps[i].kernel != KM_KERNEL_GENERIC && plan.steps[i].kernel != KM_KERNEL_MFMA_ANY)) continue;
            if (!lane_wins(pr, plan, i)) continue;
            ++wins;
            if (!lane_takes(p, q)) return printf("%dx%d variant %d", p, q, plan.steps[i].variant), 1;
        }
    }
    printf("ok %d", wins > 5000);
}
""") == "ok 1"


def test_where_the_line_lies():
    """64 workgroups of 256 slices for the generic kernel's steps, more for slices of up to 8 elements; 128 for the
    chunked form's, whose whole vectors stay with it unless columns are many; rows of 16 slices; 92 MiB for the form in registers, with
    rows of less than 64 slices only where they gain; never in fp64, nor when an option asks for kernels or tiles."""
    def flips(M, S, P, Q, other=-1):
        return _first(M, _shapes(S, P, Q))["variant"] == other and _first(M + 1, _shapes(S, P, Q))["variant"] == LANE
    assert flips(1008, 16, 13, 6) and flips(1008, 16, 10, 3) and flips(8176, 16, 7, 3) and flips(510, 128, 7, 3) and flips(131056, 16, 7, 20)
    assert flips(127, 256, 40, 8) and flips(127, 256, 42, 15) and flips(127, 256, 36, 12) and flips(127, 256, 72, 20)
    assert _first(4000, _shapes(256, 48, 12))["variant"] == -1
    assert _first(4000, _shapes(15, 13, 6))["variant"] == -1
    assert flips(1141, 320, 33, 33, PAD) and flips(709330, 1, 27, 7, PAD)
    for S, P, Q in ((1, 20, 15), (1, 16, 16), (16, 27, 20), (63, 36, 36), (330, 32, 6), (330, 34, 32), (330, 60, 60), (330, 100, 100), (330, 52, 68)):
        assert _first(-(-25000000 // (S * P)), _shapes(S, P, Q))["variant"] == PAD
    assert _first(4000, _shapes(320, 10, 3), "float64")["variant"] == -1
    old = km.get_option(km.KM_OPT_PREFER_THREADS)
    try:
        km.set_option(km.KM_OPT_PREFER_THREADS, 256)
        assert _first(4000, _shapes(320, 10, 3))["variant"] == -1
    finally:
        km.set_option(km.KM_OPT_PREFER_THREADS, old)


def test_rows_of_slices_are_found_exactly_up_to_the_most_slices(tmp_path):
    """The kernel's division by the slices of a row, for the first and the last slices of rows and of all: exact for as many slices as a
    launch may have, and problems of more are left to the generic kernel.  (The last slice of 1 x (5x1)^15, 2^32.5 slices, is one that it
    would put into a second row.)"""
    assert _run(tmp_path, """
static int64_t found(int64_t g, int64_t S) { return S == 1 ? g : (int64_t)(((unsigned __int128)(uint64_t)g * lane_row_magic(S)) >> 64); }
int main()
{
    std::mt19937_64 rng(9);
    for (int k = 0; k < 200000; ++k) {
        const int64_t S = k < 64 ? LANE_MAX_SLICES - k : 1 + ((int64_t)(rng() % (uint64_t)LANE_MAX_SLICES) >> rng() % 32);
        const int64_t rows = LANE_MAX_SLICES / S, r = rng() % (uint64_t)rows;
        for (int64_t g : {r * S, r * S + S - 1, (rows - 1) * S, rows * S - 1, r * S + (int64_t)(rng() % (uint64_t)S)})
            if (found(g, S) != g / S) return printf("slice %lld of %lld a row\\n", (long long)g, (long long)S), 1;
        if (lane_shape(5, 1, rows * S).lds_bytes == 0) return printf("refused\\n"), 1;
    }
    const int64_t S = 6103515625;                        // 5^14
    printf("%d %d %d\\n", found(S - 1, S) == 0, lane_shape(5, 1, S).lds_bytes, lane_shape(5, 1, LANE_MAX_SLICES + 1).lds_bytes);
}
""") == "0 0 0"
    assert [st["variant"] for st in km.plan(1, [5] * 15, [1] * 15, "float32")][:3] == [-1, LANE, LANE]


def test_launches_are_not_mixed_around_the_last_level_cache():
    """Intermediates of 160 to 320 MiB (256 where their runs are not aligned) that the form in registers leaves in the last-level cache."""
    forms = lambda M, P, Q: [s["variant"] for s in km.plan(M, [P] * 3, [Q] * 3, "float32")]
    assert forms(2250, 31, 31) == forms(1790, 31, 32) == forms(8388, 20, 20) == [PAD] * 3
    assert forms(1500, 30, 30) == forms(2700, 30, 30) == forms(682, 36, 36) == forms(1367, 33, 33) == [LANE] * 3


def test_the_plan_names_what_runs_and_other_steps_stay_as_they_are():
    """Beside the plan without this kernel (an option that asks for a workgroup size no kernel has): its steps replace generic ones and
    ones of its family, factors, rows and buffers stay.  kronmatmul_launches gives the same list."""
    rng, lane = np.random.default_rng(3), 0
    old = km.get_option(km.KM_OPT_PREFER_THREADS)
    for _ in range(3000):
        dtype = "float32" if rng.random() < 0.7 else "float64"
        n = int(rng.integers(1, 5))
        P, Q = [[int(2 ** rng.uniform(1, 7.2)) for _ in range(n)] for _ in range(2)]
        M = int(10 ** rng.uniform(0, 7))
        steps = km.plan(M, P, Q, dtype)
        assert km.launches(M, P, Q, dtype) == steps
        if LANE not in [st["variant"] for st in steps]:
            continue
        try:
            km.set_option(km.KM_OPT_PREFER_THREADS, 1)
            without = km.plan(M, P, Q, dtype)
        finally:
            km.set_option(km.KM_OPT_PREFER_THREADS, old)
        assert len(without) == len(steps) and dtype == "float32"
        for st, had in zip(steps, without):
            if st["variant"] != LANE:
                assert st == had
                continue
            lane += 1
            assert had["variant"] in (-1, PAD) and had["kernel"] in (km.KM_KERNEL_GENERIC, km.KM_KERNEL_MFMA_ANY)
            assert all(st[k] == had[k] for k in ("first_factor", "num_factors", "k_in", "k_out", "src", "dst", "tile_rows"))
            assert 0 < st["grid"] * st["block"] < 2 ** 32
    assert lane > 300


@pytest.mark.gpu
@pytest.mark.parametrize("M,S,P,Q", CASES)
def test_matches_the_reference(M, S, P, Q):
    """Relative to the largest value 1e-5 (a chain of dot products of lengths P_i is off by at most (sum P_i + N) u of the product
    of absolute values); bit for bit on small integers, whose sums stay below 2^24 (2 * 1333 * 128 at most)."""
    import oracle
    shapes = _shapes(S, P, Q)
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, shapes, "float32", seed=71, **kinds)
        print("lane M=%d S=%d %dx%d" % (M, S, P, Q), flush=True)
        got = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]).cpu().numpy()
        ref = oracle.kron_matmul(X, Fs)
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("M,S,P,Q", [(296, 443, 6, 14), (100, 164, 21, 5), (514, 64, 23, 4), (66, 500, 42, 15)])
def test_nothing_leaks_between_rows(M, S, P, Q):
    """Slices are read in unaligned vectors, the last of which overlaps the one before: infinities in the first and the last element
    of a row must not reach the rows beside it, nor one in the last element of X any other row."""
    shapes = _shapes(S, P, Q)
    assert _first(M, shapes)["variant"] == LANE
    X, Fs = kron_inputs.make_problem(M, shapes, "float32", seed=72)
    F = [torch.from_numpy(f).cuda() for f in Fs]
    clean = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    X[3, 0] = X[3, -1] = X[M - 1, -1] = np.inf
    got = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    rest = [r for r in range(M) if r not in (3, M - 1)]
    assert torch.equal(got[rest], clean[rest])
    assert not torch.isfinite(got[3]).any() and not torch.isfinite(got[M - 1]).any()


@pytest.mark.gpu
def test_replays_from_a_graph_and_both_store_forms():
    """24x24^3, 1300 rows: an intermediate of 69 MiB, stored so that it stays in the last-level cache, and the last one not; every
    replay is compared, with eager work between them."""
    M, shapes = 1300, [(24, 24)] * 3
    assert [s["variant"] for s in km.plan(M, [24] * 3, [24] * 3, "float32")] == [LANE] * 3
    X = torch.randn(M, 24 ** 3, device="cuda")
    F = [torch.randn(24, 24, device="cuda") / 24 ** 0.5 for _ in range(3)]
    want = km.kronmatmul(X, F)
    call = km.Prepared(X, F)
    out = call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(km.kronmatmul(X, F), want)
