"""bfloat16 products with the parameters resident in registers: layers whose widths sit at the edges of its column blocks (32, 64 a
wavefront, 256 a workgroup), pieces (64 k) and segments, and matrices of more rows than one pass of the chip takes, ragged at the end."""
import numpy as np
import pytest

from test_gpu_bf16 import G, check_single_layer_bf16  # noqa: F401  (G is the fixture)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def pinned(monkeypatch):
    """Also for as few rows as these."""
    monkeypatch.setenv("COFREE_BF16_TILE", "1")


# forward N = d_out (or d_msg), K = d_in; backward N = d_in, K = d_out; sums of two segments K = d_out + d_msg (sage), 2 d_out
@pytest.mark.parametrize("kind,dims", [("gcn", (257, 8, 129)), ("gcn", (320, 8, 160)), ("gcn", (256, 8, 200)), ("gcn", (250, 8, 172)), ("gcn", (129, 8, 384)), ("gcn", (385, 8, 191)),
                                       ("gcn", (449, 8, 257)), ("gcn", (512, 8, 256)), ("gcn", (256, 8, 512)), ("gcn", (300, 8, 500)),
                                       ("sage_conv", (170, 8, 150)), ("sage_conv", (256, 8, 256)), ("sage_conv", (300, 8, 130)),
                                       ("sage", (47, 256, 256)), ("sage", (100, 256, 256)), ("sage", (256, 256, 192)),
                                       ("sage", (200, 263, 140))])
def test_layer_widths(G, kind, dims):  # noqa: F811
    check_single_layer_bf16(G, kind, dims)


@pytest.mark.parametrize("n", [33, 8_193, 131_073])
@pytest.mark.parametrize("d_in,d_out", [(256, 250), (288, 160), (500, 224)])
def test_many_rows(n, d_in, d_out):
    """A conventional GraphSAGE layer on a ring: two-segment, accumulating and gated products over all rows."""
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] pinned product n={n} {d_in} -> {d_out}", flush=True)
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
