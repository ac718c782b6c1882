"""What the binding returns, whatever kind of tensor it is given."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")
import paper_2401_10187_amd as km  # noqa: E402


class Tagged(torch.Tensor):
    """A subclass that keeps its type through torch's own operations."""


@pytest.mark.gpu
@pytest.mark.parametrize("wrap", [lambda t: t, lambda t: t.as_subclass(Tagged), torch.nn.Parameter], ids=["tensor", "subclass", "parameter"])
def test_a_new_result_is_a_plain_tensor_without_gradient(wrap):
    X, Fs = kron_inputs.make_problem(5, [(4, 3), (6, 7)], "float32", seed=70)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    want = km.kronmatmul(Xd, Fd)
    for got in (km.kronmatmul(wrap(Xd), Fd), km.Prepared(wrap(Xd), Fd)()):
        assert type(got) is torch.Tensor and not got.requires_grad
        assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
