"""bfloat16 products with the parameters resident in registers: layers whose widths sit at the edges of its column blocks (32, 64 a
wavefront, 256 a workgroup), pieces (64 k) and segments, and matrices of more rows than one pass of the chip takes, ragged at the end."""
import numpy as np
import pytest

from oracle.layers import dropout_keep
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


# a workgroup takes three to ten tiles of 32 rows: their dropout runs beside the next tile's matrix instructions, the last one's behind them
@pytest.mark.parametrize("kind,n,d_in,d_out,nch", [("gcn", 20_001, 256, 512, 4), ("gcn", 20_001, 320, 324, 5), ("sage_conv", 40_001, 256, 256, 8),
                                                   ("sage_conv", 40_001, 160, 172, 6), ("sage_conv", 20_001, 193, 260, 8)])
def test_dropout_over_many_rows(kind, n, d_in, d_out, nch):
    """Against the same layer without dropout times the oracle's keep decisions."""
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] dropout of a pinned product {kind} n={n} {d_in} -> {d_out}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(n)
    H = torch.randn(n, d_in, generator=gen, device="cuda").bfloat16()
    p = {"W": torch.randn(d_out, d_in * (2 if kind == "sage_conv" else 1), generator=gen, device="cuda") / d_in ** 0.5,
         "bW": torch.randn(d_out, generator=gen, device="cuda")}
    saved = {"A": torch.empty(n, d_in, dtype=torch.bfloat16, device="cuda")}
    out, q = [], 0.3
    for rate in (0.0, q):
        d = B.layer_desc(B.SAGE_CONV if kind == "sage_conv" else B.GCN, d_in, 0, d_out, act=1, dropout_q=rate, layer_id=3, seed=2 ** 40 + 9,
                         epoch=6, dtype=B.BF16)
        Y = torch.full((n, d_out), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.profile_enable(True)
        B.layer_fwd(P, None, 0, d, H, p, Y, saved, torch.empty(B.layer_workspace_bytes(d, n, False), dtype=torch.uint8, device="cuda"))
        names = list(B.profile_read())
        B.profile_enable(False)
        assert any(x.startswith(f"gemm_bf16_pinned_kernel<{nch},{2 if rate else 0}>") for x in names), names
        assert not any(x.startswith("mask_grad") for x in names), names
        out.append(Y.float())
    keep = torch.from_numpy(dropout_keep(n, d_out, q, 2 ** 40 + 9, 6, 3)).cuda()
    want = out[0] * float(np.float32(1.0 / (1.0 - np.float32(q))))
    assert bool(torch.isfinite(out[0]).all()) and bool((out[1][~keep] == 0).all())
    # both runs round once, by at most 2^-8
    assert bool(((out[1] - want)[keep].abs() <= 2.0 ** -7 * want[keep].abs()).all())
