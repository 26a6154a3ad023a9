"""Float32 products of at most 64 columns and weight gradients of at most 64 rows or columns against float64: edges of
blocks and windows, ranges of less than one step, two segments, everything the epilogue can do, parameters beyond LDS."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2308_03209_amd import binding as B
    return dict(B=B, torch=torch)


def ring(B, n):
    src = np.arange(n, dtype=np.int64)
    return B.build_partition(n, src, (src + 1) % n, 1, 0, 3)


def within_rounding(got, ref, mag, terms, what):
    """A float32 sum of `terms` products: terms 2^-24 of the sum of magnitudes, and the result's own rounding."""
    err, bound = (got.double() - ref).abs(), (terms + 4.0) * 2.0 ** -24 * mag
    assert bool((err <= bound).all()), f"{what}: error {float((err / bound.clamp_min(1e-300)).max()):.2f} of its bound"


# rows: less than a tile, ragged, several rounds of all workgroups; columns: windows of 1 .. 3, moved, whole; k: short,
# one window, moved windows, whole steps, more steps than LDS holds
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (15, 2, 3), (17, 3, 15), (33, 4, 16), (1000, 5, 17), (2049, 16, 31), (300, 17, 602),
                                   (19_717, 33, 500), (40_001, 47, 128), (5_000, 49, 129), (70_003, 64, 40), (66_000, 63, 7),
                                   (3_000, 64, 1433), (2_100, 48, 900), (515, 9, 2600), (35_000, 20, 70), (50_000, 7, 33),
                                   # the last four k of a segment, element by element below four, rings of one, two and four steps
                                   (5_000, 33, 5), (50, 60, 2), (140_000, 20, 3), (100_003, 64, 6), (300_001, 16, 9), (65_537, 30, 64),
                                   # two wavefronts of 32 columns a row tile, with parameters beyond LDS in the first
                                   (20_003, 50, 1433), (24_001, 64, 77), (17_003, 49, 602),
                                   # parameters beyond LDS in two parts, read again by two (66,003 and 70,003 rows) and three rounds
                                   (66_003, 9, 2600), (70_003, 17, 1300), (140_001, 41, 900),
                                   # tiles of 128 x 64
                                   (90_001, 41, 900), (70_003, 64, 1433), (60_001, 50, 130), (60_001, 64, 256)])
@pytest.mark.parametrize("relu", [False, True])
def test_products(env, M, N, K, relu):
    B, torch = env["B"], env["torch"]
    print(f"[case] narrow product M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, W, b = (torch.randn(*s, generator=gen, device="cuda") for s in ((M, K), (N, K), (N,)))
    C = torch.full((M + 1, N), float("nan"), device="cuda")
    B.dense_nt_f32(A, W, b, C[:M], relu)
    ref = A.double() @ W.double().T + b.double()
    within_rounding(C[:M], ref.clamp_min(0.0) if relu else ref, A.double().abs() @ W.double().abs().T + b.double().abs(), K + 1, "product")
    assert bool(torch.isnan(C[M]).all())  # nothing behind the result


@pytest.mark.parametrize("M,N,K,tiled", [(65_536, 64, 1433, False), (65_537, 64, 1433, True), (131_072, 33, 900, True), (131_073, 33, 900, False),
                                         (70_000, 32, 1300, False), (65_537, 64, 600, False), (53_249, 49, 113, True), (53_248, 49, 113, False),
                                         (98_304, 64, 320, True), (98_305, 64, 320, False), (60_000, 64, 112, False), (60_000, 64, 321, False),
                                         (60_000, 48, 128, False)])
def test_which_kernel(env, M, N, K, tiled):
    """Parameters beyond LDS read again every round, and a round and a bit of 49 to 64 columns, go to the tiles."""
    B, torch = env["B"], env["torch"]
    print(f"[case] kernel of the product M={M} N={N} K={K}", flush=True)
    A, W = torch.ones(M, K, device="cuda"), torch.ones(N, K, device="cuda")
    C = torch.empty(M, N, device="cuda")
    B.profile_enable(True)
    B.dense_nt_f32(A, W, torch.zeros(N, device="cuda"), C, False)
    names = list(B.profile_read())
    B.profile_enable(False)
    assert len(names) == 1 and names[0].startswith("gemm_kernel<false,false,1>" if tiled else "narrow_gemm_kernel<"), names
    assert bool((C == K).all())


def test_non_finite_operands_stay_in_their_rows_and_columns(env):
    B, torch = env["B"], env["torch"]
    print("[case] narrow product of non-finite operands", flush=True)
    A, W = torch.rand(100, 37, device="cuda") + 0.1, torch.rand(43, 37, device="cuda") + 0.1
    A[3, 20], A[5, 36], A[6, 0] = float("inf"), float("nan"), -float("inf")
    W[42, 36] = float("inf")
    C = torch.empty(100, 43, device="cuda")
    B.dense_nt_f32(A, W, torch.zeros(43, device="cuda"), C, False)
    ref = A.double() @ W.double().T
    bad = ~torch.isfinite(ref)
    assert bool((torch.isnan(C) == torch.isnan(ref)).all()) and bool((C.double() == ref)[bad & ~torch.isnan(ref)].all())
    assert bool(torch.isfinite(C[~bad]).all())


# Both directions of a layer on a ring, whose aggregation is a mean over neighbours: products of either order with every
# epilogue (conventional GraphSAGE accumulates where it transforms first) and weight gradients of either narrow side.
# The printed layer's inner ReLU cannot be switched off, so it runs where no pre-activation is within rounding of zero.
@pytest.mark.parametrize("kind,n,d_in,d_msg,d_out",
                         [(k, n, *d) for k in ("gcn", "sage", "sage_conv")
                          for n, *d in [(129, 3, 2, 2), (2_000, 64, 16, 16), (5_003, 41, 33, 7), (33_000, 100, 64, 47),
                                        (20_011, 130, 48, 63), (9_001, 12, 5, 200), (40_000, 256, 40, 1)]
                          if k != "sage" or n <= 10_000] + [("sage", 4_001, 128, 256, 50)] +
                         # weight gradients of 50 and 64 rows or columns whose chunks are cut in two and in three
                         [("gcn", 45_001, 601, 2, 50), ("gcn", 90_001, 50, 2, 320), ("sage_conv", 130_003, 512, 2, 64)] +
                         # k-major parameters in two segments beyond LDS, in one round and in two; a short segment before a long one;
                         # tiles in both orders and accumulating
                         [("sage_conv", 5_003, 48, 2, 600), ("sage_conv", 70_003, 20, 2, 700), ("sage", 3_001, 40, 100, 2),
                          ("sage_conv", 60_001, 50, 2, 130), ("sage_conv", 60_001, 150, 2, 50)] +
                         # wide input gradients from 8 to 15 k, wide weight gradients over 5 to 13 nodes (gemm_split.hip)
                         [("gcn", 3_001, 100, 2, 8), ("sage_conv", 3_001, 130, 2, 13), ("gcn", 257, 70, 2, 15), ("gcn", 300, 80, 2, 16),
                          ("gcn", 5, 65, 2, 66), ("gcn", 9, 65, 2, 66), ("gcn", 13, 65, 2, 130)])
def test_layers(env, kind, n, d_in, d_msg, d_out):
    from oracle import dropedge as o_dropedge
    from oracle import layers as o_layers
    from oracle import partition as o_partition
    from paper_2308_03209_amd import inputs
    from util import assert_close
    B, torch = env["B"], env["torch"]
    print(f"[case] narrow {kind} n={n} {d_in} -> {d_msg} -> {d_out}", flush=True)
    code = {"gcn": B.GCN, "sage": B.SAGE_MEAN, "sage_conv": B.SAGE_CONV}[kind]
    prm = inputs.model_params(kind, [(d_in, d_msg, d_out)], random_bias=True)[0]
    src = np.arange(n, dtype=np.int64)
    O = o_dropedge.full_graph(o_partition.build_partition(n, src, (src + 1) % n, 1, 0, 3))
    rng = np.random.default_rng(n + d_in)
    H, dY = rng.standard_normal((n, d_in)).astype(np.float32), rng.standard_normal((n, d_out)).astype(np.float32)
    desc = B.layer_desc(code, d_in, d_msg, d_out)
    ws = torch.empty(max(B.layer_workspace_bytes(desc, n, x) for x in (False, True)), dtype=torch.uint8, device="cuda")
    p = {k: torch.from_numpy(v).cuda() for k, v in prm.items()}
    h, dy = torch.from_numpy(H).cuda(), torch.from_numpy(dY).cuda()
    Y, dX = torch.full((n, d_out), float("nan"), device="cuda"), torch.full((n, d_in), float("nan"), device="cuda")
    saved = {"Z": torch.empty((n, d_msg), device="cuda"), "A": torch.empty((n, max(d_msg, d_in)), device="cuda")}
    g = {k: torch.full_like(v, float("nan")) for k, v in p.items()}
    P = ring(B, n)
    B.layer_fwd(P, None, 0, desc, h, p, Y, saved, ws)
    B.layer_bwd(P, None, 0, desc, h, Y, p, saved, dy, dX, g, False, ws)
    p64 = {k: v.astype(np.float64) for k, v in prm.items()}
    if kind == "sage":
        ref, sv = o_layers.sage_fwd(O, H, p64)
        ref_dX, ref_g = o_layers.sage_bwd(O, p64, sv, dY)
    elif kind == "sage_conv":
        ref, sv = o_layers.sage_conv_fwd(O, H, p64, False)
        ref_dX, ref_g = o_layers.sage_conv_bwd(O, p64, sv, dY)
    else:
        ref, sv = o_layers.gcn_fwd(O, H, p64, False)
        ref_dX, ref_g = o_layers.gcn_bwd(O, p64, sv, dY)
    assert_close(Y.cpu().numpy(), ref, what="H_out")
    assert_close(dX.cpu().numpy(), ref_dX, what="dH_in")
    for k in ref_g:
        assert_close(g[k].cpu().numpy(), ref_g[k], what=f"d{k}")


@pytest.mark.parametrize("kind,d_in,d_msg,d_out", [("sage_conv", 100, 0, 33), ("sage_conv", 40, 0, 64), ("sage", 48, 70, 20), ("sage", 30, 24, 40),
                                                   ("sage", 8, 100, 40)])
def test_two_weight_gradients_in_one_launch(env, kind, d_in, d_msg, d_out, monkeypatch):
    """The two weight gradients of a layer from one launch, or (as the second stream wants them) from two: the same bits."""
    B, torch = env["B"], env["torch"]
    n = 3_001
    print(f"[case] paired weight gradients {kind} {d_in} -> {d_msg} -> {d_out}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d_in)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    desc = B.layer_desc({"sage": B.SAGE_MEAN, "sage_conv": B.SAGE_CONV}[kind], d_in, d_msg, d_out)
    p = {"W": rand(d_msg, d_in), "bW": rand(d_msg), "U": rand(d_out, d_msg + d_in), "bU": rand(d_out)} if kind == "sage" else \
        {"W": rand(d_out, 2 * d_in), "bW": rand(d_out)}
    ws = torch.empty(max(B.layer_workspace_bytes(desc, n, x) for x in (False, True)), dtype=torch.uint8, device="cuda")
    H, dY, Y, dX = rand(n, d_in), rand(n, d_out), torch.empty(n, d_out, device="cuda"), torch.empty(n, d_in, device="cuda")
    saved = {"Z": torch.empty(n, max(d_msg, 1), device="cuda"), "A": torch.empty(n, max(d_msg, d_in, d_out), device="cuda")}
    P, got = ring(B, n), []
    B.layer_fwd(P, None, 0, desc, H, p, Y, saved, ws)
    for overlap in ("0", "1"):
        monkeypatch.setenv("COFREE_OVERLAP", overlap)
        g = {k: torch.full_like(v, float("nan")) for k, v in p.items()}
        B.layer_bwd(P, None, 0, desc, H, Y, p, saved, dY, dX, g, False, ws)
        got.append(g)
    for k in p:
        assert bool(torch.isfinite(got[0][k]).all()) and torch.equal(got[0][k], got[1][k]), k


def test_bias_gradients_are_rounded_once_a_group_of_nodes(env):
    """Column sums beside a weight gradient, over 24 draws of 100,000 x 47: relative error 1.75e-7 where 16 nodes at a time were added
    to a sum, 2.0e-7 where every node is (3 % of it is the spread of the estimate)."""
    B, torch = env["B"], env["torch"]
    n, d_in, d_out = 100_000, 512, 47
    print("[case] bias gradients of a narrow layer", flush=True)
    P, desc = ring(B, n), B.layer_desc(B.SAGE_CONV, d_in, 0, d_out)
    ws = torch.empty(B.layer_workspace_bytes(desc, n, True), dtype=torch.uint8, device="cuda")
    H, Y = torch.zeros(n, d_in, device="cuda"), torch.zeros(n, d_out, device="cuda")
    p = {"W": torch.zeros(d_out, 2 * d_in, device="cuda"), "bW": torch.zeros(d_out, device="cuda")}
    g, err, size = {k: torch.empty_like(v) for k, v in p.items()}, 0.0, 0.0
    for seed in range(24):
        dY = torch.randn(n, d_out, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")
        B.layer_bwd(P, None, 0, desc, H, Y, p, {}, dY, None, g, False, ws)
        ref = dY.double().sum(0)
        err, size = err + float((g["bW"].double() - ref).square().sum()), size + float(ref.square().sum())
    assert (err / size) ** 0.5 < 1.85e-7
