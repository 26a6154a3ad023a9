"""What a runner refuses before it hands addresses to the library (no GPU: a host-only partition, buffers on the CPU)."""
import numpy as np
import pytest
import torch

from paper_2308_03209_amd import binding as B
from paper_2308_03209_amd import model as M


def runner(kind):
    P = B.build_partition(6, np.array([0, 1, 2, 3, 4]), np.array([1, 2, 3, 4, 5]), 1, 0, 1, flags=B.HOST_ONLY)
    model = M.Model(kind, [(5, 7, 9), (9, 7, 3)], device="cpu")
    return model, M.PartitionRunner(P, model, device="cpu")


@pytest.mark.parametrize("kind", ["gcn", "sage", "sage_conv"])
def test_buffers_put_in_place_of_the_runners_own(kind, monkeypatch):
    calls = []
    for name in ("layers_fwd", "layers_bwd", "loss_weighted"):
        monkeypatch.setattr(B, name, lambda *a, name=name: calls.append(name))
    X, y = torch.zeros(6, 5), torch.zeros(6, dtype=torch.int32)
    model, run = runner(kind)
    run.forward(X)
    run.loss_backward(y)
    assert calls == ["layers_fwd", "loss_weighted", "layers_bwd"]
    need = max(o + n for sl in model.slices for o, n, _ in sl.values())   # the padding behind the last tensor is not read
    short, strided = torch.zeros(need - 1), torch.zeros(2 * need)[::2]
    for bad in (short, strided):
        model, run = runner(kind)
        model.theta = bad
        with pytest.raises(ValueError):
            run.forward(X)
        model, run = runner(kind)
        run.forward(X)
        model.grad = bad
        with pytest.raises(ValueError):
            run.loss_backward(y)
    model.theta = model.grad = torch.zeros(need)
    run.forward(X)
    run.loss_backward(y)
    model, run = runner(kind)
    run.H[1] = torch.zeros(9, 6).T
    with pytest.raises(ValueError):
        run.forward(X)
