"""Room for parameters split beforehand only saves time in float32: calls without it are accepted and give the same results, and
small graphs do not ask for it.  What a layer cannot do without is still refused."""
import pytest

pytestmark = pytest.mark.gpu

SMALL, LARGE = 2_000, 200_000  # nodes; 256 x 512 over LARGE is more than 2e10 operand pairs


@pytest.fixture(scope="module")
def env():
    import numpy as np
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2308_03209_amd import binding as B

    def ring(n):
        src = np.arange(n, dtype=np.int64)
        return B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    return dict(B=B, torch=torch, part={n: ring(n) for n in (SMALL, LARGE)})


def layer(env, kind, n, dtype):
    B, torch = env["B"], env["torch"]
    d_in, d_msg, d_out = 256, 288, 512  # the mean first, in all kinds
    code = {"gcn": B.GCN, "sage": B.SAGE_MEAN, "sage_conv": B.SAGE_CONV}[kind]
    desc = B.layer_desc(code, d_in, d_msg, d_out, dtype=B.F32 if dtype is torch.float32 else B.BF16)
    gen = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda") * 0.1
    p = {"W": rand(d_msg, d_in), "bW": rand(d_msg), "U": rand(d_out, d_msg + d_in), "bU": rand(d_out)} if kind == "sage" else \
        {"W": rand(d_out, 2 * d_in if kind == "sage_conv" else d_in), "bW": rand(d_out)}
    H, dY = rand(n, d_in).to(dtype), rand(n, d_out).to(dtype)
    saved = {"Z": torch.empty(n, d_msg, device="cuda", dtype=dtype), "A": torch.empty(n, d_msg, device="cuda", dtype=dtype)}
    return desc, p, H, dY, saved


@pytest.mark.parametrize("kind", ["gcn", "sage", "sage_conv"])
@pytest.mark.parametrize("n", [SMALL, LARGE])
def test_float32_layers_do_without(env, kind, n):
    B, torch, P = env["B"], env["torch"], env["part"][n]
    print(f"[case] workspace of a float32 {kind} layer, {n} nodes", flush=True)
    desc, p, H, dY, saved = layer(env, kind, n, torch.float32)
    size = [B.layer_workspace_bytes(desc, n, x) for x in (False, True)]
    assert (size[0] > 256) == (n == LARGE)
    room = [torch.empty(x, dtype=torch.uint8, device="cuda") for x in size]
    out = []
    for fwd, bwd in ((room[0], room[1]), (None, room[1] if n == SMALL else room[1][:-256])):
        Y, dX = torch.empty(n, dY.shape[1], device="cuda"), torch.empty_like(H)
        g = {k: torch.empty_like(v) for k, v in p.items()}
        B.layer_fwd(P, None, 0, desc, H, p, Y, saved, fwd)
        B.layer_bwd(P, None, 0, desc, H, Y, p, saved, dY, dX, g, False, bwd)
        out.append([Y, dX, *g.values()])
    assert all(bool(torch.isfinite(a).all()) and torch.equal(a, b) for a, b in zip(*out))
    with pytest.raises(B.CofreeError, match="workspace"):
        B.layer_bwd(P, None, 0, desc, H, Y, p, saved, dY, dX, g, False, room[1][:n * 256 * 4])


@pytest.mark.parametrize("kind", ["gcn", "sage", "sage_conv"])
def test_bfloat16_layers_do_not(env, kind):
    B, torch, P = env["B"], env["torch"], env["part"][SMALL]
    print(f"[case] workspace of a bfloat16 {kind} layer", flush=True)
    desc, p, H, dY, saved = layer(env, kind, SMALL, torch.bfloat16)
    Y = torch.empty(SMALL, dY.shape[1], device="cuda", dtype=torch.bfloat16)
    for ws in (None, torch.empty(256, dtype=torch.uint8, device="cuda")):
        with pytest.raises(B.CofreeError, match="workspace"):
            B.layer_fwd(P, None, 0, desc, H, p, Y, saved, ws)
