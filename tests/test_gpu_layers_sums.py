"""Gradients of all layers of a small graph are summed by one launch: the same numbers as with a launch per layer, which a
workspace without room for all partials gets, also with more sums than one launch takes and with a shared gradient."""
import numpy as np
import pytest

from paper_2308_03209_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2308_03209_amd import binding as B
    from paper_2308_03209_amd import model as M
    wl = inputs.WORKLOADS[0]
    src, dst = inputs.workload_graph(wl)
    return dict(B=B, M=M, torch=torch, P=B.build_partition(wl.n_nodes, src, dst, 4, 0, inputs.SEED_CUT))


def gradients(env, kind, dims, dtype, roomy, tied=False):
    B, M, torch, P = env["B"], env["M"], env["torch"], env["P"]
    model = M.Model(kind, dims)
    model.load(inputs.model_params(kind, dims, seed=3, random_bias=True))
    if tied:
        model.offsets[2] = model.offsets[1]
    run = M.PartitionRunner(P, model, None, 0.2, 9, dtype=dtype)
    descs = [run.desc(l, 0) for l in range(len(dims))]
    least = max(B.layer_workspace_bytes(d, P.num_nodes, b) for d in descs for b in (False, True))
    assert run.workspace.numel() > least
    if not roomy:
        run.workspace = torch.empty(least, dtype=torch.uint8, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(P.num_nodes, dims[0][0], generator=gen, device="cuda").to(run.torch_dtype)
    y = torch.randint(0, dims[-1][2], (P.num_nodes,), generator=gen, device="cuda", dtype=torch.int32)
    model.grad.fill_(0.5)
    for accumulate in (False, True):
        run.iteration(X, y, 1, accumulate=accumulate)
    return model.grad.clone()


@pytest.mark.parametrize("kind", ["gcn", "sage", "sage_conv"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layers", [2, 7])
def test_one_launch_or_many(env, kind, dtype, layers):
    print(f"[case] sums of {layers} layers {kind} {dtype}", flush=True)
    dims = [(40, 24, 24)] + [(24, 24, 24)] * (layers - 2) + [(24, 24, 7)]
    assert env["torch"].equal(gradients(env, kind, dims, dtype, True), gradients(env, kind, dims, dtype, False))


@pytest.mark.parametrize("kind", ["gcn", "sage", "sage_conv"])
def test_layers_that_share_a_gradient(env, kind):
    print(f"[case] sums of tied layers {kind}", flush=True)
    dims = [(40, 24, 24), (24, 24, 24), (24, 24, 24), (24, 24, 7)]
    a, b = gradients(env, kind, dims, "f32", True, tied=True), gradients(env, kind, dims, "f32", False, tied=True)
    assert env["torch"].equal(a, b) and bool(env["torch"].isfinite(a).all())
