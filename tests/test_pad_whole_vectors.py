"""The register form of the run-time-shape MFMA kernel on slices that are whole 16-byte vectors: it loads without a
branch per lane and lets the end of the buffer answer, so what lies behind X and behind the factor must not be seen."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

PAD = -3
# (dtype, P, Q): every class of the contraction, its ends and P % 4 != 0, one to eight column blocks and ragged ones
SHAPES = [("float32", 20, 18), ("float32", 28, 33), ("float32", 44, 30), ("float32", 60, 63), ("float32", 84, 81),
          ("float32", 100, 100), ("float32", 128, 113), ("float64", 20, 20), ("float64", 30, 31), ("float64", 50, 47),
          ("float64", 70, 66), ("float64", 98, 100), ("float64", 128, 127)]


def _tile(dtype, P, Q):
    step = km.plan(3000, [P], [Q], dtype)[0]
    return step["tile_slices"] if step["variant"] == PAD else 0


def test_the_shapes_take_the_kernel():
    for dtype, P, Q in SHAPES:
        assert _tile(dtype, P, Q) > 0 and P * np.dtype(dtype).itemsize % 16 == 0, (dtype, P, Q)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P,Q", SHAPES, ids=str)
def test_ends_of_the_last_tile(dtype, P, Q):
    """Slices one past a tile, one short of one and whole tiles; NaN right behind X and behind the factor.  A dot
    product of P terms is off by at most P u of the sum of absolute values; equal to the bit on small integers."""
    import oracle
    tile, u = _tile(dtype, P, Q), np.finfo(dtype).eps / 2
    for slices in (3 * tile + 1, 17 * tile - 1, 16 * tile):
        for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
            X, Fs = kron_inputs.make_problem(slices, [(P, Q)], dtype, seed=71, **kinds)
            hold = [torch.full((a.size + 64,), float("nan"), dtype=getattr(torch, dtype), device="cuda") for a in (X, Fs[0])]
            for h, a in zip(hold, (X, Fs[0])):
                h[:a.size] = torch.from_numpy(a.reshape(-1)).cuda()
            print("pad %s %dx%d, %d slices" % (dtype, P, Q, slices), flush=True)
            got = km.kronmatmul(hold[0][:X.size].view(X.shape), [hold[1][:Fs[0].size].view(P, Q)]).cpu().numpy()
            if exact:
                assert np.array_equal(got, oracle.kron_matmul(X, Fs))
            else:
                ref = X.astype(np.longdouble) @ Fs[0].astype(np.longdouble)
                assert (np.abs(got - ref) <= P * u * (np.abs(X).astype(np.float64) @ np.abs(Fs[0]).astype(np.float64))).all()
