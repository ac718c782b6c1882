"""The copies that the transposed entry points make of their factors, at the ends of a workgroup's share (1024
elements) and with rows below and above the 256 elements that its threads lie apart."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")
import paper_2401_10187_amd as km  # noqa: E402

CASES = [[(31, 33), (1, 9)], [(32, 32), (2, 2)], [(25, 41), (5, 1)], [(7, 500)], [(300, 11), (3, 4)], [(3, 256), (2, 257)],
         [(129, 255)], [(700, 701)], [(1, 1)] * 5 + [(2, 3)]]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("shapes", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_same_bits_as_factors_transposed_by_the_caller(dtype, shapes):
    """The plan and the kernels of the product are the same, so the copies have to be the same numbers."""
    X, Fs = kron_inputs.make_problem(3, shapes, dtype, seed=68)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    print("transposed copy %s %s" % (dtype, shapes), flush=True)
    got = km.kronmatmul(Xd, [F.t().contiguous() for F in Fd], transposed=True)
    assert np.array_equal(got.cpu().numpy(), km.kronmatmul(Xd, Fd).cpu().numpy())
