"""Dropout applied by the launch that finishes a layer's output: every kernel that does so, at widths around its limits,
against the same layer without dropout times the oracle's keep decisions."""
import numpy as np
import pytest

from oracle.layers import dropout_keep
from test_gpu_bf16 import G  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

# widths and the kernel that ends the layer (f32 / bf16)
SHAPES = [("sage_conv", 72, 132),   # aggregate first: split / resident product, ragged column block
          ("sage_conv", 256, 128),  # transform first: the aggregation, which adds the self part / a launch of its own
          ("sage_conv", 40, 94),    # no multiple of four columns: a launch of its own
          ("gcn", 256, 512),        # widest split tiles / column parts of the resident product
          ("gcn", 72, 300),         # column parts that are no multiple of four columns where there are three
          ("gcn", 128, 36),         # transform first: the aggregation
          ("gcn", 700, 640),        # aggregation in two panels / with two pieces per lane
          ("gcn", 1100, 1028),      # last panel of a bfloat16 row narrower than one access
          ("gcn", 80, 12),          # rows of few lanes, one window moved left
          ("gcn", 128, 37), ("gcn", 128, 39), ("gcn", 700, 641), ("sage_conv", 200, 33), ("sage_conv", 90, 9), ("gcn", 1100, 1037),  # lanes that begin inside draws
          ("sage", 100, 260), ("sage", 64, 36)]


@pytest.mark.parametrize("dtype,products", [("f32", None), ("bf16", "0"), ("bf16", None)])
@pytest.mark.parametrize("kind,d_in,d_out", SHAPES)
def test_against_keep_decisions(G, kind, d_in, d_out, dtype, products, monkeypatch):  # noqa: F811
    """products: resident ones wherever they fit ("0"), or as many rows as here take (mostly tiled ones)."""
    B, torch = G["B"], G["torch"]
    if products is not None:
        monkeypatch.setenv("COFREE_BF16_TILE", products)
    print(f"[case] fused dropout {kind} {d_in} -> {d_out} {dtype}", flush=True)
    n, q = 5003, 0.3
    rng = np.random.default_rng(1)
    hub = np.arange(1, 4401, dtype=np.int64)  # node 0: a hub row; nodes 1 .. 200: rows of a wavefront or a workgroup
    src = np.concatenate([np.zeros_like(hub), rng.integers(1, 200, 20_000), np.arange(n, dtype=np.int64)])
    dst = np.concatenate([hub, rng.integers(200, n, 20_000), (np.arange(n, dtype=np.int64) + 1) % n])
    lo, hi = np.minimum(src, dst), np.maximum(src, dst)
    pair = np.unique(lo * n + hi)
    P = B.build_partition(n, pair // n, pair % n, 1, 0, 3)
    assert P.num_nodes == n
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    code = {"gcn": B.GCN, "sage": B.SAGE_MEAN, "sage_conv": B.SAGE_CONV}[kind]
    d_msg = 72 if kind == "sage" else 0
    gen = torch.Generator(device="cuda").manual_seed(5)

    def rand(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")
    H = rand(n, d_in).to(td)
    prm = {"W": rand(d_msg or d_out, d_in * (2 if kind == "sage_conv" else 1)) / d_in ** 0.5, "bW": rand(d_msg or d_out)}
    if kind == "sage":
        prm.update(U=rand(d_out, d_msg + d_in) / d_in ** 0.5, bU=rand(d_out))
    saved = {"Z": torch.empty(n, max(d_msg, 1), dtype=td, device="cuda"),
             "A": torch.empty(n, max(d_msg, d_in, d_out), dtype=td, device="cuda")}
    out = []
    for rate in (0.0, q):
        d = B.layer_desc(code, d_in, d_msg, d_out, act=0 if kind == "sage" else 1, dropout_q=rate, layer_id=3, seed=2 ** 40 + 9,
                         epoch=6, dtype=B.F32 if dtype == "f32" else B.BF16)
        y = torch.full((n, d_out), float("nan"), device="cuda", dtype=td)
        B.layer_fwd(P, None, 0, d, H, prm, y, saved, torch.empty(B.layer_workspace_bytes(d, n, False), dtype=torch.uint8, device="cuda"))
        out.append(y.float().cpu().numpy())
    keep = dropout_keep(n, d_out, q, 2 ** 40 + 9, 6, 3)
    want = np.where(keep, out[0] * np.float32(1.0 / (1.0 - np.float32(q))), np.float32(0.0))
    assert np.all(out[1][~keep] == 0.0)
    if dtype == "f32":  # the same sums and one more product
        np.testing.assert_allclose(out[1], want, rtol=2e-7, atol=0)
    else:  # the plain run rounds once more, by 2^-9 of its value
        np.testing.assert_allclose(out[1], want, rtol=2.0 ** -7, atol=0)


@pytest.mark.parametrize("dtype,width", [("f32", 5), ("f32", 7), ("bf16", 9), ("bf16", 22)])
@pytest.mark.parametrize("n", [65_535, 65_536])
def test_narrow_rows_over_many_nodes(dtype, width, n):
    """A launch of its own from 65,536 nodes on, the aggregation's before."""
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] dropout of narrow rows {dtype} {n} x {width}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    td, code = (torch.float32, B.F32) if dtype == "f32" else (torch.bfloat16, B.BF16)
    gen = torch.Generator(device="cuda").manual_seed(width)
    H = torch.randn(n, width + 7, generator=gen, device="cuda").to(td)
    p = {"W": torch.randn(width, width + 7, generator=gen, device="cuda"), "bW": torch.randn(width, generator=gen, device="cuda")}
    q, out = 0.3, []
    for rate in (0.0, q):
        d = B.layer_desc(B.GCN, width + 7, 0, width, act=1, dropout_q=rate, layer_id=3, seed=2 ** 40 + 9, epoch=6, dtype=code)
        Y = torch.full((n, width), float("nan"), dtype=td, device="cuda")
        B.profile_enable(True)
        B.layer_fwd(P, None, 0, d, H, p, Y, {}, torch.empty(B.layer_workspace_bytes(d, n, False), dtype=torch.uint8, device="cuda"))
        names = list(B.profile_read())
        B.profile_enable(False)
        assert any(x.startswith("mask_grad") for x in names) == (rate > 0 and n >= 65_536), names
        out.append(Y.float().cpu().numpy())
    keep = dropout_keep(n, width, q, 2 ** 40 + 9, 6, 3)
    want = np.where(keep, out[0] * np.float32(1.0 / (1.0 - np.float32(q))), np.float32(0.0))
    assert np.all(out[1][~keep] == 0.0)
    # float32: one more product; bfloat16: both runs round once, by at most 2^-8
    np.testing.assert_allclose(out[1], want, rtol=2e-7 if dtype == "f32" else 2.0 ** -7, atol=0)
