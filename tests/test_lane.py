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


# (rows, slices of a row, P, Q): every compiled chunk length (2 to 7, 9 and 13 vectors), one chunk, several and overlapping ones, 0 to 3
# elements left over, 1 to 32 groups of columns with and without a remainder, 64 workgroups and more; rows of 16 slices (several to a
# tile), of no multiple of 64 and of whole tiles, with aligned and misaligned results; a ragged last tile
CASES = [
    (1025, 16, 5, 1), (700, 24, 5, 9), (37, 443, 6, 14), (130, 128, 7, 23), (64, 257, 8, 5), (9, 1856, 9, 4), (50, 330, 11, 3),
    (600, 30, 13, 6), (20, 820, 16, 3), (70, 235, 18, 2), (100, 164, 21, 5), (257, 64, 23, 4), (64, 256, 26, 5), (12, 1366, 29, 5),
    (130, 253, 34, 11), (80, 410, 37, 8), (66, 500, 42, 15), (36, 911, 50, 8), (42, 781, 51, 15), (32, 1040, 60, 14), (62, 529, 69, 14), (16, 2049, 84, 22),
    (38, 863, 97, 17), (52, 640, 110, 20), (34, 964, 127, 3), (60, 547, 128, 26), (16, 1025, 5, 126), (70, 255, 5, 32),
    # from the form with the factor in registers
    (1150, 330, 33, 33), (1200, 625, 17, 17), (800, 500, 36, 29), (900, 400, 30, 40), (300, 629, 65, 66), (330, 512, 68, 76), (160, 1333, 45, 71),
]


@pytest.mark.parametrize("M,S,P,Q", CASES)
def test_the_list_takes_the_kernel_and_its_launches_fit(M, S, P, Q):
    st = _first(M, _shapes(S, P, Q))
    assert st["variant"] == LANE and st["kernel"] == km.KM_KERNEL_MFMA_ANY
    assert st["block"] == 256 and st["grid"] % 8 == 0 and st["lds_bytes"] <= 160 * 1024
    assert 256 * (st["grid"] - 8) < M * S <= 2 * 256 * st["grid"]           # four tiles of 64 slices, once or twice


def test_where_the_line_lies():
    """64 workgroups of 256 slices for the generic kernel's steps, 128 for the chunked form's, rows of 16 slices; 96 MB for the form in
    registers; never in fp64, nor when an option asks for kernels or tiles."""
    assert _first(1008, _shapes(16, 10, 3))["variant"] == -1 and _first(1009, _shapes(16, 10, 3))["variant"] == LANE
    assert _first(127, _shapes(256, 42, 15))["variant"] == -1 and _first(128, _shapes(256, 42, 15))["variant"] == LANE
    assert _first(1200, _shapes(15, 10, 3))["variant"] == -1
    assert _first(1136, _shapes(320, 33, 33))["variant"] == PAD and _first(1137, _shapes(320, 33, 33))["variant"] == LANE
    assert _first(4000, _shapes(320, 10, 3), "float64")["variant"] == -1
    assert _first(4000, _shapes(320, 60, 60))["variant"] == PAD and _first(640, _shapes(320, 100, 100))["variant"] == PAD
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
    src = tmp_path / "rows.cpp"
    src.write_text("""
#include "paper_2401_10187_amd/csrc/plan.hpp"
#include <cstdio>
#include <random>
using namespace km;
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
""")
    exe = tmp_path / "rows"
    subprocess.run(["g++", "-std=c++17", "-I", ROOT, "-o", str(exe), str(src)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True).stdout.strip() == "0 0 0"
    assert [st["variant"] for st in km.plan(1, [5] * 15, [1] * 15, "float32")][:3] == [-1, LANE, LANE]


def test_launches_are_not_mixed_around_the_last_level_cache():
    """Results of 160 to 320 MiB: with a step of aligned ones in the problem, which stays, the others of that size stay too."""
    forms = lambda M, P, Q: [s["variant"] for s in km.plan(M, [P] * 3, [Q] * 3, "float32")]
    assert forms(1790, 31, 32) == forms(2000, 30, 32) == [PAD] * 3
    assert forms(5488, 22, 22) == [LANE] * 3                   # none is aligned
    assert forms(682, 36, 36) == [LANE] * 3                    # 121 MiB


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
    of absolute values); bit for bit on small integers, whose sums stay below 2^24 (2 * 1856 * 128 at most)."""
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
@pytest.mark.parametrize("M,S,P,Q", [(37, 443, 6, 14), (100, 164, 21, 5), (257, 64, 23, 4), (66, 500, 42, 15)])
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
