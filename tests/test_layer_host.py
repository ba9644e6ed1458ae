"""The PyTorch layer's state, without a GPU."""
import copy
import pickle

import pytest

torch = pytest.importorskip("torch")


def test_layers_are_copied_and_pickled_without_what_evaluation_keeps():
    from paper_2106_00003_amd import layer
    net = layer.OrthogonalLinear(6, device="cpu")
    net._captured.append("a matrix")
    old = {k: v for k, v in net.__dict__.items() if not k.startswith(("_eval", "_captured"))}
    old["_eval_tables"] = None                              # what earlier versions kept
    from_old = layer.OrthogonalLinear.__new__(layer.OrthogonalLinear)
    from_old.__setstate__(old)
    for other in (copy.deepcopy(net), pickle.loads(pickle.dumps(net)), from_old):
        assert other._eval_matrix is None and other._eval_run is None and other._captured == []
        assert not hasattr(other, "_eval_tables")
        assert torch.equal(other.theta, net.theta) and (other.n, other.m) == (6, None)
    assert net._captured == ["a matrix"]
