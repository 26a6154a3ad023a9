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


# nodes and widths that reach each tile of the kernel with more steps than its ring of loads holds twice, ragged at the end
@pytest.mark.parametrize("n,d_in,d_out,tile", [(100_002, 200, 200, "128x128"), (300_002, 100, 40, "64x128"), (300_002, 256, 256, "128x256"),
                                               (300_002, 256, 40, "64x256"), (140_002, 100, 600, "256x128"),
                                               (140_002, 300, 512, "256x256"), (1_100_002, 256, 256, "256x256"),
                                               (20_002, 602, 256, "128x128"), (140_002, 602, 256, "256x256")])
def test_exact_sums(env, n, d_in, d_out, tile):
    """Small whole numbers, whose sums are exact in float32: a row left out or taken twice shows.  Nodes in pairs, so that
    the aggregated gradient of a transform-first layer, the mean of two even numbers, is whole too."""
    B, torch = env["B"], env["torch"]
    print(f"[case] bfloat16 weight gradient, exact sums n={n} {d_in} -> {d_out} ({tile})", flush=True)
    assert 12 * n < 2 ** 24 and n % 2 == 0
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    A = torch.randint(-3, 4, (n, d_in), generator=gen, device="cuda").bfloat16()
    dH = (2 * torch.randint(-2, 3, (n, d_out), generator=gen, device="cuda")).bfloat16()
    src = np.arange(0, n, 2, dtype=np.int64)
    P = B.build_partition(n, src, src + 1, 1, 0, 3)
    W = torch.zeros(d_out, d_in, device="cuda")
    d = B.layer_desc(B.GCN, d_in, 0, d_out, dtype=B.BF16)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    g = {"W": torch.full_like(W, float("nan")), "bW": torch.full((d_out,), float("nan"), device="cuda")}
    B.layer_bwd(P, None, 0, d, A, dH, {"W": W, "bW": torch.zeros(d_out, device="cuda")}, {"A": A}, dH, None, g, False, ws)
    h = dH.double()
    t = h if d_in <= d_out else (h + h.view(-1, 2, d_out).flip(1).reshape(n, d_out)) / 2
    assert torch.equal(g["W"].double(), t.T @ A.double())
    assert torch.equal(g["bW"].double(), h.sum(0))
