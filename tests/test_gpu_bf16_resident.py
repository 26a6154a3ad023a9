"""bfloat16 products with the parameters resident in LDS: layers whose widths sit at the edges of its column blocks (32),
pieces (64 k) and limits, and matrices of more rows than one pass of the chip takes, ragged at the end."""
import numpy as np
import pytest

from test_gpu_bf16 import G, check_single_layer_bf16  # noqa: F401  (G is the fixture)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def resident(monkeypatch):
    """Also for as few rows as these, where the tiled kernel would be taken."""
    monkeypatch.setenv("COFREE_BF16_TILE", "0")


# forward N = d_out (or d_msg), K = d_in; backward N = d_in; sums of two segments K = d_out + d_msg (sage), 2 d_out
@pytest.mark.parametrize("kind,dims", [("gcn", (8, 8, 32)), ("gcn", (33, 8, 65)), ("gcn", (64, 8, 96)), ("gcn", (128, 8, 129)),
                                       ("gcn", (172, 8, 256)), ("gcn", (256, 8, 224)), ("gcn", (500, 8, 64)),
                                       ("gcn", (513, 8, 47)), ("sage_conv", (65, 8, 63)), ("sage_conv", (256, 8, 100)),
                                       ("sage_conv", (192, 8, 255)), ("sage", (64, 72, 33)), ("sage", (100, 128, 128)),
                                       ("sage", (47, 200, 41)), ("sage", (31, 32, 34))])
def test_layer_widths(G, kind, dims):  # noqa: F811
    check_single_layer_bf16(G, kind, dims)


@pytest.mark.parametrize("n", [33, 70_017, 131_073])
@pytest.mark.parametrize("d_in,d_out", [(72, 40), (256, 33), (200, 130)])
def test_many_rows(G, n, d_in, d_out):  # noqa: F811
    """A conventional GraphSAGE layer on a ring: plain, accumulating and gated products over all rows."""
    B, torch = G["B"], G["torch"]
    print(f"[case] resident product n={n} {d_in} -> {d_out}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(n)
    H = torch.randn(n, d_in, generator=gen, device="cuda").bfloat16()
    dO = torch.randn(n, d_out, generator=gen, device="cuda").bfloat16()
    W = torch.randn(d_out, 2 * d_in, generator=gen, device="cuda") / d_in ** 0.5
    b = torch.randn(d_out, generator=gen, device="cuda")
    d = B.layer_desc(B.SAGE_CONV, d_in, 0, d_out, act=1, dtype=B.BF16, grad_flags=B.GRAD_IN_GATED | B.GRAD_OUT_GATED)
    ws = torch.empty(max(B.layer_workspace_bytes(d, n, False), B.layer_workspace_bytes(d, n, True)), dtype=torch.uint8, device="cuda")
    out, dH = torch.full_like(dO, float("nan")), torch.full_like(H, float("nan"))
    prm = {"W": W, "bW": b}
    g = {"W": torch.empty_like(W), "bW": torch.empty_like(b)}
    B.layer_fwd(P, None, 0, d, H, prm, out, {}, ws)
    B.layer_bwd(P, None, 0, d, H, out, prm, {}, dO, dH, g, False, ws)

    def mean(x):
        return 0.5 * (x.roll(1, 0) + x.roll(-1, 0))
    h, w, z = H.double(), W.double(), dO.double()
    ref = torch.relu(h @ w[:, :d_in].T + mean(h @ w[:, d_in:].T) + b.double())
    ref_dH = (z @ w[:, :d_in] + mean(z) @ w[:, d_in:]) * (h > 0)
    # stored intermediates and parameters are rounded to 2^-9 each: three roundings of rows of about unit size
    for got, want, what in ((out, ref, "H_out"), (dH, ref_dH, "dH_in")):
        err = (got.double() - want).abs().max() / want.abs().max()
        fro = (got.double() - want).norm() / want.norm()
        assert float(err) <= 2e-2 and float(fro) <= 1e-2, (what, float(err), float(fro))


@pytest.mark.parametrize("kind,dims", [("gcn", (1, 8, 3)), ("gcn", (7, 8, 64)), ("gcn", (8, 8, 31)), ("gcn", (63, 8, 17)), ("gcn", (64, 8, 9)),
                                       ("gcn", (65, 8, 40)), ("gcn", (130, 8, 63)), ("sage", (5, 9, 64)), ("sage", (66, 33, 20)),
                                       ("sage", (64, 70, 48)), ("sage_conv", (130, 8, 24)), ("sage_conv", (20, 8, 50))])
def test_narrow_products_of_few_rows(G, kind, dims, monkeypatch):  # noqa: F811
    """Tiles of 64 columns, which read few rows' parameters as they are: edges of columns, steps of 64 k and of eight, both segments.
    (Not a single column: its one bias gradient is a sum that cancels, 2.7 % off with the converted copy and without, whose bits agree.)"""
    monkeypatch.setenv("COFREE_BF16_TILE", "128")
    check_single_layer_bf16(G, kind, dims)


@pytest.mark.parametrize("n", [1, 130, 2_003])
@pytest.mark.parametrize("d_in", [9, 64, 130])
def test_a_single_column(n, d_in, monkeypatch):
    """Every column of the tile but one is the last one again.  Its bias gradient may cancel: judged by the size of its terms."""
    import torch
    from paper_2308_03209_amd import binding as B
    monkeypatch.delenv("COFREE_BF16_TILE")
    print(f"[case] a single column n={n} d_in={d_in}", flush=True)
    src = np.arange(max(n, 3), dtype=np.int64)
    n = len(src)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(d_in + n)
    H, dO = torch.randn(n, d_in, generator=gen, device="cuda").bfloat16(), torch.randn(n, 1, generator=gen, device="cuda").bfloat16()
    p = {"W": torch.randn(1, d_in, generator=gen, device="cuda"), "bW": torch.randn(1, generator=gen, device="cuda")}
    d = B.layer_desc(B.GCN, d_in, 0, 1, dtype=B.BF16)
    ws = torch.empty(max(B.layer_workspace_bytes(d, n, x) for x in (False, True)), dtype=torch.uint8, device="cuda")
    Y, dH = torch.full_like(dO, float("nan")), torch.full_like(H, float("nan"))
    g = {k: torch.full_like(v, float("nan")) for k, v in p.items()}
    B.profile_enable(True)
    B.layer_fwd(P, None, 0, d, H, p, Y, {}, ws)
    B.layer_bwd(P, None, 0, d, H, Y, p, {}, dO, dH, g, False, ws)
    names = list(B.profile_read())
    B.profile_enable(False)
    assert any(x.startswith("gemm_bf16_kernel<false,false,true,2,2,1> N=1 ") for x in names), names

    def ahat(x):  # every node has degree two
        return (x.roll(1, 0) + x.roll(-1, 0) + x) / 3
    h, w, z = H.double(), p["W"].double(), dO.double()
    t = ahat(z)
    # parameters, the stored intermediate and the result are rounded, each by at most 2^-8 of its value (eight significant bits)
    for got, ref, mag, what in ((Y, ahat(h @ w.T) + p["bW"].double(), ahat(h.abs() @ w.abs().T) + p["bW"].double().abs(), "H_out"),
                                (dH, t @ w, ahat(z.abs()) @ w.abs(), "dH_in"),
                                (g["W"], t.T @ h, ahat(z.abs()).T @ h.abs(), "dW"),
                                (g["bW"], z.sum(0), z.abs().sum(0), "dbW")):
        assert bool(((got.double() - ref).abs() <= 3.05 * 2.0 ** -8 * mag).all()), what
