"""Weight and bias gradients of bfloat16 layers against float64, at the edges of their tiles (64, 128 and 256 rows, 128 and
256 columns), pieces of eight columns, steps of 32 and 64 nodes and chunks."""
import numpy as np
import pytest

from paper_2308_03209_amd import inputs  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2308_03209_amd import binding as B
    return dict(B=B, torch=torch, rings={})


def ring(env, n):
    if n not in env["rings"]:
        src = np.arange(n, dtype=np.int64)
        env["rings"][n] = env["B"].build_partition(n, src, (src + 1) % n, 1, 0, 3)
    return env["rings"][n]


def assert_rounding(got, ref, mag, n, what):
    """Products of bfloat16 are exact in float32, so only the float32 sum of n of them rounds: n 2^-24 of the sum of
    magnitudes."""
    err, bound = (got.double() - ref).abs(), (n + 4.0) * 2.0 ** -24 * mag
    assert bool((err <= bound).all()), f"{what}: error {float((err / bound.clamp_min(1e-300)).max()):.2f} of its bound"


@pytest.mark.parametrize("n", [33, 1_983, 40_003])
@pytest.mark.parametrize("kind,d_in,d_out", [("gcn", 8, 8), ("gcn", 9, 47), ("gcn", 63, 65), ("gcn", 100, 129), ("gcn", 128, 256),
                                             ("gcn", 172, 257), ("gcn", 300, 300), ("gcn", 257, 512), ("sage_conv", 12, 64),
                                             ("sage_conv", 100, 128), ("sage_conv", 128, 128), ("sage_conv", 129, 130),
                                             ("sage_conv", 256, 256), ("sage_conv", 7, 40)])
def test_saved_aggregates(env, n, kind, d_in, d_out):
    """Aggregate-first layers without activation: dW = dH^T A (GCN), dH^T [H | A] (conventional GraphSAGE), db = column
    sums of dH, for any saved A."""
    B, torch = env["B"], env["torch"]
    print(f"[case] bfloat16 weight gradient {kind} n={n} {d_in} -> {d_out}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    H, A = (torch.randn(n, d_in, generator=gen, device="cuda").bfloat16() for _ in range(2))
    dH = torch.randn(n, d_out, generator=gen, device="cuda").bfloat16()
    conv = kind == "sage_conv"
    W = torch.randn(d_out, 2 * d_in if conv else d_in, generator=gen, device="cuda")
    d = B.layer_desc(B.SAGE_CONV if conv else B.GCN, d_in, 0, d_out, dtype=B.BF16)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    g = {"W": torch.full_like(W, float("nan")), "bW": torch.full((d_out,), float("nan"), device="cuda")}
    B.layer_bwd(ring(env, n), None, 0, d, H, dH, {"W": W, "bW": torch.zeros(d_out, device="cuda")}, {"A": A}, dH, None, g,
                False, ws)
    x, h = (torch.cat([H, A], 1) if conv else A).double(), dH.double()
    assert_rounding(g["W"], h.T @ x, h.abs().T @ x.abs(), n, "dW")
    assert_rounding(g["bW"], h.sum(0), h.abs().sum(0), n, "db")


@pytest.mark.parametrize("n,d_in,d_out", [(33, 16, 8), (1_983, 300, 41), (40_003, 256, 172)])
def test_sums_of_another_matrix(env, n, d_in, d_out):
    """Transform-first GCN: the column sums of dPre come from further workgroups of the launch."""
    B, torch = env["B"], env["torch"]
    print(f"[case] bfloat16 column sums n={n} {d_in} -> {d_out}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    H, dH = (torch.randn(n, c, generator=gen, device="cuda").bfloat16() for c in (d_in, d_out))
    W = torch.randn(d_out, d_in, generator=gen, device="cuda")
    d = B.layer_desc(B.GCN, d_in, 0, d_out, dtype=B.BF16)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    g = {"W": torch.full_like(W, float("nan")), "bW": torch.full((d_out,), float("nan"), device="cuda")}
    B.layer_bwd(ring(env, n), None, 0, d, H, dH, {"W": W, "bW": torch.zeros(d_out, device="cuda")}, {}, dH, None, g, False, ws)
    h = dH.double()
    assert_rounding(g["bW"], h.sum(0), h.abs().sum(0), n, "db")
    t = (h + h.roll(1, 0) + h.roll(-1, 0)) / 3.0  # rounded to bfloat16 before the product: 2^-9 of every element
    ref, mag = t.T @ H.double(), t.abs().T @ H.double().abs()
    assert bool(((g["W"].double() - ref).abs() <= (2.0 ** -8 + n * 2.0 ** -24) * mag).all())
