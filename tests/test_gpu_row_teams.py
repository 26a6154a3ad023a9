"""The aggregation's teams of lanes: rows just below, at and above the degrees at which a row gets a wavefront, a
workgroup or a hub launch, for every lane layout (width) of the row kernel, against the oracle."""
import numpy as np
import pytest

from oracle import dropedge as o_dropedge
from oracle import layers as o_layers
from oracle import partition as o_partition
from paper_2308_03209_amd import inputs
from util import assert_close

pytestmark = pytest.mark.gpu

DEGREES = [4097, 4095, 1000, 257, 256, 255, 129, 128, 127, 65, 64, 63, 33, 32, 31, 17, 16, 15]


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2308_03209_amd import binding as B
    src, dst = inputs.hub_graph(5001, DEGREES, 6000, 21)
    P = B.build_partition(5001, src, dst, 1, 0, 1)
    return dict(B=B, torch=torch, P=P, O=o_partition.build_partition(5001, src, dst, 1, 0, 1), M=B.dropedge_k(P, 1, 0.5, 3))


# columns per 16-byte piece: 4 in float32, 8 in bfloat16; lane layouts change at 1, 2, 4, ... 64 and 128 pieces
@pytest.mark.parametrize("dtype,width", [("f32", w) for w in (1, 2, 3, 4, 7, 13, 31, 41, 100, 255, 300, 514)] +
                         [("bf16", w) for w in (1, 2, 3, 4, 5, 6, 7, 8, 15, 30, 47, 128, 172, 500, 1000)])
@pytest.mark.parametrize("masked", [False, True])
def test_rows_at_the_team_limits(env, dtype, width, masked):
    check(env, dtype, width, masked)


@pytest.mark.parametrize("dtype,width", [("f32", w) for w in (2, 8, 31, 41, 300)] + [("bf16", w) for w in (5, 8, 64, 128, 500)])
def test_a_wavefront_for_every_row(env, dtype, width, monkeypatch):
    """As in graphs of high average degree, where narrow rows are not shared by a workgroup's wavefronts."""
    monkeypatch.setenv("COFREE_AGG_SLICES", "1")
    check(env, dtype, width, False)


# without slices any width of 1 to 32 pieces, with slices 2 to 64 whole lines of 128 bytes (other widths take another kernel)
@pytest.mark.parametrize("launch,dtype,width",
                         [("2", "f32", w) for w in (4, 5, 31, 32, 33, 64, 100, 128)] + [("2", "bf16", w) for w in (8, 9, 47, 64, 100, 172, 256)] +
                         [("8", "f32", w) for w in (64, 128, 256, 512, 1024, 2048)] + [("8", "bf16", w) for w in (128, 256, 512, 1024, 4096)])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("slots", ["0", "1"])
def test_teams_of_equal_rows_and_column_slices(env, launch, dtype, width, masked, slots, monkeypatch):
    """As in graphs of high average degree; the last wavefront has lanes without a row and rows without neighbours."""
    monkeypatch.setenv("COFREE_AGG_SLICES", launch)
    monkeypatch.setenv("COFREE_AGG_SLOTS", slots)
    check(env, dtype, width, masked)


@pytest.mark.parametrize("launch,width", [("2", w) for w in (4, 8, 16, 31, 64)] + [("8", w) for w in (64, 128, 256, 512)])
def test_float32_sums_of_long_rows_are_short(env, launch, width, monkeypatch):
    """4000 neighbours of 1 + 0.45 2^-15: a chain of additions loses the fraction from 256 on (6e-6 of the sum in eight chains of
    500), one of up to 250 loses at most 1.3e-6."""
    B, torch = env["B"], env["torch"]
    monkeypatch.setenv("COFREE_AGG_SLICES", launch)
    print(f"[case] long row in float32, launch {launch}, {width} columns", flush=True)
    n = 4_100
    spokes = np.arange(1, 4_001, dtype=np.int64)
    ring = np.arange(4_000, n - 1, dtype=np.int64)
    P = B.build_partition(n, np.concatenate([np.zeros_like(spokes), ring]), np.concatenate([spokes, ring + 1]), 1, 0, 3)
    X = torch.full((n, width), 1.0 + 0.45 * 2.0 ** -15, device="cuda")
    Y = torch.empty_like(X)
    B.aggregate(P, None, 0, B.AGG_MEAN, X, Y, width, B.F32)
    assert float((Y[0].double() / X[0].double() - 1.0).abs().max()) < 2e-6


@pytest.mark.parametrize("launch,dtype,width",
                         [("2", "f32", w) for w in (4, 5, 12, 33, 36, 47, 64)] + [("2", "bf16", w) for w in (8, 12, 44, 47, 64, 100, 172)] +
                         [("8", "f32", w) for w in (64, 128, 256, 512)] + [("8", "bf16", w) for w in (128, 256, 512, 1024)])
def test_what_follows_a_sum_in_teams_and_slices(env, launch, dtype, width, monkeypatch):
    """Bias, ReLU and dropout of a layer that transforms first, the gate of the layer below in the backward pass of one that
    aggregates first: as in the row kernel, which other tests hold against the oracle, up to the order of the sums."""
    B, torch, P = env["B"], env["torch"], env["P"]
    print(f"[case] epilogue of launch {launch}, {width} {dtype} columns", flush=True)
    n, q = P.num_nodes, 0.3
    td, code, tol = (torch.float32, B.F32, 1e-5) if dtype == "f32" else (torch.bfloat16, B.BF16, 2.0 ** -7)
    gen = torch.Generator(device="cuda").manual_seed(width)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    first = B.layer_desc(B.GCN, width + 8, 0, width, 1, q, 2, 77, 5, code)
    H, W, b = rand(n, width + 8).to(td), rand(width, width + 8) / width ** 0.5, rand(width)
    last = B.layer_desc(B.GCN, width, 0, width + 4, 0, 0.0, 3, 77, 5, code, B.GRAD_IN_GATED, q)
    gate, dY = rand(n, width).clamp_min(0.0).to(td), rand(n, width + 4).to(td)
    W2, A = rand(width + 4, width) / width ** 0.5, rand(n, width).to(td)
    ws = torch.empty(max(B.layer_workspace_bytes(first, n, False), B.layer_workspace_bytes(last, n, True)), dtype=torch.uint8, device="cuda")
    g = {"W": torch.empty_like(W2), "bW": torch.empty(width + 4, device="cuda")}
    got = []
    for env_launch in ("0", launch):
        monkeypatch.setenv("COFREE_AGG_SLICES", env_launch)
        Y, dX = torch.full((n, width), float("nan"), device="cuda", dtype=td), torch.full((n, width), float("nan"), device="cuda", dtype=td)
        B.profile_enable(True)
        B.layer_fwd(P, None, 0, first, H, {"W": W, "bW": b}, Y, {}, ws)
        B.layer_bwd(P, None, 0, last, gate, dY, {"W": W2, "bW": g["bW"]}, {"A": A}, dY, dX, g, False, ws)
        names = [x for x in B.profile_read() if x.startswith("aggregate")]
        B.profile_enable(False)
        assert any(x.startswith("aggregate_sliced_kernel") for x in names) == (env_launch != "0"), names
        got.append((Y.float(), dX.float()))
    for (a, c), what in zip(zip(*got), ("output", "gradient")):
        assert bool(torch.isfinite(a).all()) and bool(torch.isfinite(c).all()), what
        assert float(((a == 0) != (c == 0)).float().mean()) <= 1e-5, what  # but for sums within rounding of zero
        assert float((a == 0).float().mean()) > 0.4, what  # ReLU and dropout, or the gate, were there
        assert float((a - c).norm()) <= tol * float(a.norm()) and float((a - c).abs().max()) <= 4 * tol * float(a.abs().max()), what


@pytest.fixture(scope="module")
def circulants(env):
    """Graphs in which node i is joined to the k nodes on either side of it: 2 k n entries."""
    made = {}

    def get(n, k):
        if (n, k) not in made:
            i = np.repeat(np.arange(n, dtype=np.int64), k)
            made.clear()
            made[n, k] = env["B"].build_partition(n, i, (i + np.tile(np.arange(1, k + 1, dtype=np.int64), n)) % n, 1, 0, 3)
        return made[n, k]
    return get


# launches: "rows" the row kernel, a number: lanes of a team, or of a slice
@pytest.mark.parametrize("n,k,dtype,width,mean,gcn",
                         [(65_535, 16, "f32", 4, "rows", "rows"), (65_536, 16, "f32", 4, 8, 8), (65_536, 16, "f32", 16, 8, 8),
                          (65_536, 16, "bf16", 8, 8, 8), (65_536, 16, "f32", 17, "rows", "rows"), (65_535, 24, "f32", 17, "rows", "rows"),
                          (65_536, 24, "f32", 17, 8, 8), (65_536, 24, "bf16", 64, 8, 8), (65_536, 24, "f32", 33, "rows", "rows"),
                          (262_144, 16, "f32", 33, 16, 16), (131_072, 32, "f32", 33, "rows", 16), (131_072, 32, "bf16", 72, "rows", 16),
                          (7_812, 8, "f32", 128, "rows", "rows"), (7_813, 8, "f32", 128, 8, 8), (7_813, 7, "f32", 128, "rows", "rows"),
                          (46_874, 8, "f32", 64, "rows", "rows"), (46_875, 8, "f32", 64, 8, 8), (46_875, 8, "f32", 96, "rows", "rows"),
                          (60_000, 8, "f32", 2048, 64, 64), (60_000, 8, "bf16", 4096, 64, 64), (62_000, 8, "bf16", 4096, "rows", "rows")])
def test_which_launch_of_dense_graphs(env, circulants, n, k, dtype, width, mean, gcn):
    """The launch on either side of the limits in entries, bytes and pieces; float32 rows of eight lines are cut at any size."""
    B, torch = env["B"], env["torch"]
    print(f"[case] launch for {n} nodes of {2 * k} neighbours, {width} {dtype} columns", flush=True)
    P = circulants(n, k)
    td, code = (torch.float32, B.F32) if dtype == "f32" else (torch.bfloat16, B.BF16)
    X = torch.ones(n, width, device="cuda", dtype=td)
    for mode, want in ((B.AGG_MEAN, mean), (B.AGG_GCN, gcn)):
        Y = torch.zeros_like(X)
        B.profile_enable(True)
        B.aggregate(P, None, 0, mode, X, Y, width, code)
        names = list(B.profile_read())
        B.profile_enable(False)
        assert all(name.startswith("aggregate_kernel<" if want == "rows" else "aggregate_sliced_kernel<") for name in names), names
        assert want == "rows" or f",{want}," in names[0], names
        assert float((Y.float() - 1).abs().max()) <= (2e-6 if dtype == "f32" else 2.0 ** -8)


@pytest.mark.parametrize("launch", ["2", "8"])
def test_teams_on_a_mask_that_drops_everything(env, launch, monkeypatch):
    B, torch = env["B"], env["torch"]
    monkeypatch.setenv("COFREE_AGG_SLICES", launch)
    masks = B.dropedge_k(env["P"], 1, 1.0 - 2.0 ** -31, 3)
    assert len(masks.host_graph(0)[1]) == 0
    X, Y = torch.ones(env["P"].num_nodes, 128, device="cuda"), torch.full((env["P"].num_nodes, 128), float("nan"), device="cuda")
    B.aggregate(env["P"], masks, 0, B.AGG_GCN, X, Y, 128, B.F32)
    assert torch.equal(Y, X)


def check(env, dtype, width, masked):
    B, torch, P, O = env["B"], env["torch"], env["P"], env["O"]
    print(f"[case] row teams dtype={dtype} width={width} masked={masked}", flush=True)
    g = o_dropedge.full_graph(O)
    masks = None
    if masked:
        masks = env["M"]
        g = o_dropedge.masked_graph(O, o_dropedge.masks(O["n_edges"], 1, 0.5, 3)[0])
    td, code, tol = (torch.float32, B.F32, 1e-4) if dtype == "f32" else (torch.bfloat16, B.BF16, 5e-3)
    X = torch.from_numpy(np.random.default_rng(width).standard_normal((P.num_nodes, width)).astype(np.float32)).to(td).cuda()
    X64, Y = X.float().cpu().numpy().astype(np.float64), torch.empty_like(X)
    for mode, ref in [(B.AGG_MEAN, o_layers.mean_aggregate), (B.AGG_GCN, o_layers.gcn_aggregate)]:
        Y.fill_(float("nan"))
        B.aggregate(P, masks, 0, mode, X, Y, width, code)
        assert_close(Y.float().cpu().numpy(), ref(g, X64), tol, f"mode {mode} width {width}")


@pytest.mark.parametrize("dtype,width", [("f32", w) for w in (3, 4, 13, 30, 41, 100)] + [("bf16", w) for w in (5, 8, 15, 30, 47, 100, 172)])
def test_short_rows(env, dtype, width):
    """Rows of 0 to 23 neighbours, whose batches are one, two or four neighbours a lane group, beside each other in a
    wavefront; an infinite row reaches its neighbours' sums only."""
    B, torch = env["B"], env["torch"]
    print(f"[case] short rows dtype={dtype} width={width}", flush=True)
    src, dst = inputs.hub_graph(701, list(range(1, 24)) * 2, 250, 5)
    P, O = B.build_partition(701, src, dst, 1, 0, 1), o_partition.build_partition(701, src, dst, 1, 0, 1)
    td, code, tol = (torch.float32, B.F32, 1e-5) if dtype == "f32" else (torch.bfloat16, B.BF16, 5e-3)
    masks = B.dropedge_k(P, 1, 0.5, 3)
    n = P.num_nodes
    X = torch.from_numpy(np.random.default_rng(width).standard_normal((n, width)).astype(np.float32)).to(td).cuda()
    X64 = X.float().cpu().numpy().astype(np.float64)
    bad = int(np.argmax(np.diff(O["rowptr"])))
    Xinf = X.clone()
    Xinf[bad] = float("inf")
    for m, g in ((None, o_dropedge.full_graph(O)), (masks, o_dropedge.masked_graph(O, o_dropedge.masks(O["n_edges"], 1, 0.5, 3)[0]))):
        rowptr, col = g[0], g[1]
        assert m is None or int(np.min(np.diff(rowptr))) == 0
        for mode, ref in ((B.AGG_MEAN, o_layers.mean_aggregate), (B.AGG_GCN, o_layers.gcn_aggregate)):
            Y = torch.full_like(X, float("nan"))
            B.aggregate(P, m, 0, mode, X, Y, width, code)
            assert_close(Y.float().cpu().numpy(), ref(g, X64), tol, f"mode {mode} width {width}")
            Z = torch.full_like(X, float("nan"))
            B.aggregate(P, m, 0, mode, Xinf, Z, width, code)
            reached = col[rowptr[bad]:rowptr[bad + 1]].tolist() + ([bad] if mode == B.AGG_GCN else [])
            other = np.setdiff1d(np.arange(n), reached)
            assert bool(torch.isposinf(Z[reached]).all()) and torch.equal(Z[other], Y[other])
