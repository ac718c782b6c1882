"""The fp32 MFMA launches that leave their digits in place (variants -4: the last two factors, -5: one before them)."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

CHAIN, DIGIT = -4, -5

# (rows, factors): as many matrices as wavefronts and one more; columns (Q) of every compiled count of blocks, contractions
# of 16 to 128; fewer runs of columns than wavefronts and more, runs whose next one lies in another block; two leading digits.  (54 rows of
# (64x128, 48x48^2): 33 take 45.3 us with digits in place and 44.5 as rotating launches, which they are.)
CASES = [(2048, [(48, 48)] * 2), (2051, [(48, 48)] * 2), (32, [(64, 64)] * 3), (43, [(48, 48)] * 3),
         (128, [(16, 16)] + [(48, 48)] * 2), (131, [(16, 32)] + [(64, 64)] * 2), (16, [(128, 16)] + [(64, 64)] * 2),
         (22, [(96, 96)] + [(48, 48)] * 2), (32, [(64, 112)] + [(64, 64)] * 2), (19, [(112, 80)] + [(48, 48)] * 2),
         (54, [(64, 128)] + [(48, 48)] * 2), (8, [(16, 16), (16, 48)] + [(48, 48)] * 2), (5, [(32, 16), (16, 64)] + [(64, 64)] * 2)]


def _plan(M, shapes, dtype="float32"):
    return km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)


def test_plans_leave_every_digit_in_place_or_none():
    for M, shapes in CASES:
        steps = _plan(M, shapes)
        assert [s["variant"] for s in steps] == [CHAIN] + [DIGIT] * (len(shapes) - 2), (M, shapes)
        k = int(np.prod([p for p, _ in shapes]))
        for s in steps:
            assert s["kernel"] == km.KM_KERNEL_MFMA and s["k_in"] == k and 0 < s["grid"] <= 512 and s["tile_order"] == 4
            for p, q in shapes[s["first_factor"]:s["first_factor"] + s["num_factors"]]:
                k = k // p * q
            assert s["k_out"] == k
        rotating = max(M * s["k_out"] for s in steps[:-1]) * 4 if len(steps) > 1 else 0
        assert km.workspace_size(M, [p for p, _ in shapes], [q for _, q in shapes], "float32") <= 2 * (rotating + 255)
    for M, shapes, dtype in ((2047, [(48, 48)] * 2, "float32"), (31, [(64, 64)] * 3, "float32"), (5000, [(64, 64)] * 2, "float32"),
                             (64, [(48, 48)] * 3, "float64"), (64, [(64, 64)] * 2 + [(48, 48)], "float32"),
                             (64, [(24, 32)] + [(64, 64)] * 2, "float32"), (64, [(144, 16)] + [(48, 48)] * 2, "float32")):
        assert all(s["variant"] not in (CHAIN, DIGIT) for s in _plan(M, shapes, dtype)), (M, shapes, dtype)


@pytest.mark.parametrize("M,shapes", [(128, [(16, 16)] * 2 + [(64, 64)] * 2), (8, [(16, 16)] * 3 + [(64, 64)] * 2), (1, [(16, 16)] * 4 + [(48, 48)] * 2),
                                      (16, [(32, 32)] * 2 + [(64, 64)] * 2), (20, [(128, 128)] + [(48, 48)] * 2), (30, [(128, 128)] + [(48, 48)] * 2),
                                      (19, [(128, 128)] + [(64, 64)] * 2), (1, [(32, 32), (128, 128)] + [(48, 48)] * 2),
                                      (33, [(64, 128)] + [(48, 48)] * 2)], ids=str)
def test_rotating_launches_stay_where_they_are_the_faster_ones(M, shapes):
    """Leading factors that rotating launches take two at a time, and wide ones with few columns."""
    assert all(s["variant"] not in (CHAIN, DIGIT) for s in _plan(M, shapes))


def test_a_digit_with_few_columns_has_a_workgroup_for_each_stretch_of_them():
    for M, P, grid in ((24, 112, 216), (28, 96, 252), (57, 80, 256), (40, 96, 180)):
        (_, st) = _plan(M, [(P, P)] + [(48, 48)] * 2)
        assert st["variant"] == DIGIT and st["tile_slices"] == 512 and st["grid"] == grid
        assert st["tiles_per_wg"] == -(-(-(-M * 2304 // 512)) // grid)


@pytest.mark.parametrize("option,value", [("MAX_FUSE", 1), ("KERNELS", 51), ("TILE_ORDER", 2), ("TILES_PER_WG", 8), ("PREFER_TILE", 32)])
def test_options_that_ask_for_other_kernels_get_them(option, value):
    key = getattr(km, "KM_OPT_" + option)
    old = km.get_option(key)
    km.set_option(key, value)
    try:
        assert all(s["variant"] not in (CHAIN, DIGIT) for s in _plan(64, [(64, 64)] * 3))
    finally:
        km.set_option(key, old)


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_matches_the_reference(M, shapes):
    """1e-5 of the largest value (sums of P terms per factor: at most (P + 1) N u of the product of absolute values), and bit
    for bit on small integers; factors given transposed: the same bits."""
    import oracle
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        if exact and 2.0 * np.prod([p for p, _ in shapes], dtype=np.float64) >= 2 ** 24:
            continue
        X, Fs = kron_inputs.make_problem(M, shapes, "float32", seed=81, **kinds)
        print("in place M=%d %s" % (M, shapes), flush=True)
        Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
        Y = km.kronmatmul(Xd, Fd)
        ref, got = oracle.kron_matmul(X, Fs), Y.cpu().numpy()
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
            assert torch.equal(km.kronmatmul(Xd, [F.t().contiguous() for F in Fd], transposed=True), Y)


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes", [(2051, [(48, 48)] * 2), (33, [(64, 64)] * 3), (128, [(16, 16)] + [(48, 48)] * 2)], ids=str)
def test_what_is_not_finite_stays_in_its_row_and_stores_keep_to_y(M, shapes):
    """Wavefronts read their last piece again once they have run out; nothing of it may reach a result, and nothing is
    written before or behind Y."""
    X, Fs = kron_inputs.make_problem(M, shapes, "float32", "uniform", "normal", seed=82)
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    clean = km.kronmatmul(torch.from_numpy(X).cuda(), Fd)
    X[7, 0] = X[M - 1, -1] = np.inf
    X[3, 5] = np.nan
    n = clean.numel()
    frame = torch.full((n + 2048,), -7.0, device="cuda")
    Y = frame[1024:1024 + n].view(clean.shape)
    print("in place, not finite, M=%d %s" % (M, shapes), flush=True)
    got = km.kronmatmul(torch.from_numpy(X).cuda(), Fd, Y=Y)
    rest = [r for r in range(M) if r not in (3, 7, M - 1)]
    assert torch.equal(got[rest], clean[rest])
    assert not torch.isfinite(got[[3, 7, M - 1]]).any()
    assert (frame[:1024] == -7).all() and (frame[1024 + n:] == -7).all()


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes", [(2048, [(48, 48)] * 2), (32, [(64, 64)] * 3), (8, [(16, 16), (16, 48)] + [(48, 48)] * 2)], ids=str)
def test_factors_are_applied_last_to_first(M, shapes):
    """Scaling by powers of two changes no rounding as long as nothing overflows: of two neighbours the later one makes values small
    and the earlier one large again, so any other order of the two is infinite."""
    X, Fs = kron_inputs.make_problem(M, shapes, "float32", "uniform", "normal", seed=93)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    want = km.kronmatmul(Xd, Fd) * 2.0 ** 60
    for i in range(len(Fd) - 1):
        scaled = list(Fd)
        scaled[i], scaled[i + 1] = Fd[i] * 2.0 ** 80, Fd[i + 1] * 2.0 ** -80
        assert torch.equal(km.kronmatmul(Xd * 2.0 ** 60, scaled), want), i


# both forms of the first kernel, and the second one for every count of blocks of columns: a launch before the last one
# writes 48 MiB and more
KEPT = [(128, [(48, 48)] * 3), (64, [(64, 64)] * 3), (8, [(48, 48)] * 4), (11, [(32, 16), (16, 16)] + [(48, 48)] * 2),
        (11, [(16, 16), (16, 32)] + [(48, 48)] * 2), (8, [(16, 16), (16, 48)] + [(48, 48)] * 2), (6, [(16, 16), (32, 64)] + [(48, 48)] * 2),
        (5, [(16, 16), (32, 80)] + [(48, 48)] * 2), (4, [(16, 16), (32, 96)] + [(48, 48)] * 2),
        (2, [(16, 16), (64, 112)] + [(64, 64)] * 2), (3, [(16, 16), (48, 128)] + [(48, 48)] * 2)]


def _kept(M, shapes):
    """Which launches write an intermediate that stays in the last-level cache."""
    return [(s["variant"], s["k_out"] // s["k_in"] if s["variant"] == CHAIN else shapes[s["first_factor"]][1] // 16)
            for s in _plan(M, shapes)[:-1] if 48 << 20 <= M * s["k_out"] * 4 <= 320 << 20]


def test_the_cases_reach_every_form_that_keeps_its_results():
    for M, shapes in KEPT:
        assert [s["variant"] for s in _plan(M, shapes)] == [CHAIN] + [DIGIT] * (len(shapes) - 2), (M, shapes)
    assert {mb for c in KEPT for v, mb in _kept(*c) if v == DIGIT} == set(range(1, 9))
    assert {c[1][-1][0] for c in KEPT if any(v == CHAIN for v, _ in _kept(*c))} == {48, 64}


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes", KEPT, ids=lambda v: str(v).replace(" ", ""))
def test_kept_intermediates_change_no_bit_and_stores_keep_to_the_workspace(M, shapes):
    """With ordinary and with non-temporal stores the same bits; sampled rows match the reference (1e-5 of the largest value, as
    above); nothing is written behind the workspace or around Y."""
    import oracle
    X, Fs = kron_inputs.make_problem(M, shapes, "float32", "uniform", "normal", seed=94)
    print("in place, kept, M=%d %s" % (M, shapes), flush=True)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    P, Q = [p for p, _ in shapes], [q for _, q in shapes]
    need, n = km.workspace_size(M, P, Q, "float32"), M * int(np.prod(Q))
    ws = torch.full((need + 4096,), 7, dtype=torch.uint8, device="cuda")
    frame = torch.full((n + 2048,), -7.0, device="cuda")
    Y = frame[1024:1024 + n].view(M, -1)
    got, old = [], km.get_option(km.KM_OPT_KEEP_MIB)
    try:
        for keep in (old, 0, 1 << 20):
            km.set_option(km.KM_OPT_KEEP_MIB, keep)
            km.kronmatmul(Xd, Fd, Y=Y, workspace=ws[:need])
            got.append(Y.clone())
    finally:
        km.set_option(km.KM_OPT_KEEP_MIB, old)
    assert (ws[need:] == 7).all() and (frame[:1024] == -7).all() and (frame[1024 + n:] == -7).all()
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    rows = sorted({0, M // 2, M - 1})
    ref = oracle.kron_matmul(X[rows], Fs)
    assert np.abs(got[0][rows].cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
