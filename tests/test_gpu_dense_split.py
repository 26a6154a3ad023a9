"""Float32 products on the bfloat16 matrix cores (three-way split of every operand) against float64, at the edges
of their tiles and steps, with infinities, and as weight and input gradients of a layer."""
import numpy as np
import pytest

from oracle import dropedge as o_dropedge
from oracle import layers as o_layers
from oracle import partition as o_partition
from paper_2308_03209_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2308_03209_amd import binding as B
    wl = inputs.WORKLOADS[0]
    src, dst = inputs.workload_graph(wl)
    return dict(B=B, torch=torch, P=B.build_partition(wl.n_nodes, src, dst, 4, 0, inputs.SEED_CUT),
                O=o_partition.build_partition(wl.n_nodes, src, dst, 4, 0, inputs.SEED_CUT))


def assert_rounding(got, ref, mag, K, what):
    """Every element within the bound of a float32 sum of K products, K 2^-24 of the sum of magnitudes, plus the
    2^-23 of each product that the split leaves out and the result's own rounding."""
    err = np.abs(got.astype(np.float64) - ref)
    bound = (K + 4.0) * 2.0 ** -24 * mag
    assert np.all(err <= bound), f"{what}: error {np.max(err / np.maximum(bound, 1e-300)):.2f} of its bound"


# tiles are 128 x 128 or (from 512 of them) 128 x 256, k steps 16 with groups of 8
@pytest.mark.parametrize("M,N,K", [(1, 65, 8), (127, 128, 9), (129, 129, 15), (300, 255, 16), (128, 256, 17), (130, 300, 31),
                                   (257, 100, 33), (64, 384, 602), (65_600, 256, 24), (33_000, 512, 41)])
def test_product_edges(env, M, N, K):
    B, torch = env["B"], env["torch"]
    print(f"[case] split product M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(M, K, generator=gen, device="cuda") * torch.exp2(torch.randint(-20, 21, (M, 1), generator=gen, device="cuda").float())
    W, b = torch.randn(N, K, generator=gen, device="cuda"), torch.zeros(N, device="cuda")
    C = torch.full((M, N), float("nan"), device="cuda")
    B.dense_nt_f32(A, W, b, C, False)
    ref, mag = A.double() @ W.double().T, A.double().abs() @ W.double().abs().T
    assert_rounding(C.cpu().numpy(), ref.cpu().numpy(), mag.cpu().numpy(), K, "product")


def test_non_finite_operands_follow_float32_arithmetic(env):
    """An infinity or a value next to the largest float32 has no finite split: its tile is computed in plain float32."""
    B, torch = env["B"], env["torch"]
    rng = np.random.default_rng(5)
    A, W = rng.standard_normal((200, 40)).astype(np.float32), (0.1 + rng.random((130, 40))).astype(np.float32)
    A[7, 3], A[9, 5] = np.inf, np.nan
    A[150], A[151, :] = 0.0, 0.0
    A[150, 11] = np.float32(3.4e38)
    A[151, 39] = -np.inf
    C = torch.empty(200, 130, device="cuda")
    B.dense_nt_f32(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda(), torch.zeros(130, device="cuda"), C, False)
    got = C.cpu().numpy()
    assert np.all(np.isposinf(got[7])) and np.all(np.isnan(got[9])) and np.all(np.isneginf(got[151]))
    np.testing.assert_array_equal(got[150], np.float32(3.4e38) * W[:, 11])
    rest = np.setdiff1d(np.arange(200), [7, 9, 150, 151])
    a, w = A[rest].astype(np.float64), W.astype(np.float64)
    assert_rounding(got[rest], a @ w.T, np.abs(a) @ np.abs(w).T, 40, "rows beside non-finite ones")


@pytest.mark.parametrize("d_in,d_out", [(65, 66), (66, 129), (127, 128), (128, 200), (100, 256), (257, 300), (384, 512)])
def test_weight_and_input_gradients(env, d_in, d_out):
    """Backward of an aggregate-first GCN layer without activation: dW = dH^T A with any saved A, db = column sums,
    dH_in = Ahat (dH W).  The node count is no multiple of the k step."""
    B, torch, P, O = env["B"], env["torch"], env["P"], env["O"]
    print(f"[case] split gradients {d_in} -> {d_out}", flush=True)
    n = P.num_nodes
    assert n % 16 != 0
    gen = torch.Generator(device="cuda").manual_seed(d_in)
    A, dH = torch.randn(n, d_in, generator=gen, device="cuda"), torch.randn(n, d_out, generator=gen, device="cuda")
    W = torch.randn(d_out, d_in, generator=gen, device="cuda")
    d = B.layer_desc(B.GCN, d_in, 0, d_out)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    g = {"W": torch.full_like(W, float("nan")), "bW": torch.full((d_out,), float("nan"), device="cuda")}
    dX = torch.full((n, d_in), float("nan"), device="cuda")
    B.layer_bwd(P, None, 0, d, A, dH, {"W": W, "bW": torch.zeros(d_out, device="cuda")}, {"A": A}, dH, dX, g, False, ws)
    a, h, w = (x.cpu().numpy().astype(np.float64) for x in (A, dH, W))
    assert_rounding(g["W"].cpu().numpy(), h.T @ a, np.abs(h).T @ np.abs(a), n, "dW")
    assert_rounding(g["bW"].cpu().numpy(), h.sum(0), np.abs(h).sum(0), n, "db")
    full = o_dropedge.full_graph(O)
    ref, mag = o_layers.gcn_aggregate(full, h @ w), o_layers.gcn_aggregate(full, np.abs(h) @ np.abs(w))
    # on top of the product: three roundings of scales and a sum over at most max-degree neighbours
    assert_rounding(dX.cpu().numpy(), ref, mag, d_out + 4 + int(np.max(np.diff(O["rowptr"]))), "dH_in")


def ring(env, n):
    src = np.arange(n, dtype=np.int64)
    return env["B"].build_partition(n, src, (src + 1) % n, 1, 0, 3)


def assert_no_lean(err, what):
    """Errors that lean to neither side: a sum of m of them is about sqrt(m) times one, and eight times that is beyond
    the largest of the few hundred sums looked at.  (Downstream such sums over all nodes are the bias gradients.)"""
    m = err.shape[0]
    lean = float(err.sum(0).abs().max() / (m ** 0.5 * err.square().mean().sqrt()))
    assert lean <= 8.0, f"{what}: column sums of the errors {lean:.1f} times those of independent errors"


@pytest.mark.parametrize("M,N,K", [(65_600, 128, 512), (40_000, 512, 96), (65_600, 256, 40)])
def test_product_errors_do_not_lean(env, M, N, K):
    B, torch = env["B"], env["torch"]
    print(f"[case] split product, sums of errors M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(K)
    A, W = (torch.randn(*s, generator=gen, device="cuda") for s in ((M, K), (N, K)))
    C = torch.full((M, N), float("nan"), device="cuda")
    B.dense_nt_f32(A, W, None, C, False)
    assert_no_lean(C.double() - A.double() @ W.double().T, "product")


@pytest.mark.parametrize("row,col", [(-118, 100), (-130, 110), (100, -118), (-118, 0), (-94, 90), (-112, -20)])
def test_small_operands(env, row, col):
    """Rows and columns of magnitudes at which three bfloat16 do not hold a float32 (below 2^-110), beside ordinary ones."""
    B, torch = env["B"], env["torch"]
    print(f"[case] split product of 2^{row} by 2^{col}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(9)
    A, W = (torch.randn(*s, generator=gen, device="cuda") for s in ((300, 41), (200, 41)))
    A[::3], W[::5] = torch.ldexp(A[::3], torch.tensor(row)), torch.ldexp(W[::5], torch.tensor(col))
    A[5], W[7] = 0.0, 0.0
    C = torch.full((300, 200), float("nan"), device="cuda")
    B.dense_nt_f32(A, W, None, C, False)
    ref, mag = A.double() @ W.double().T, A.double().abs() @ W.double().abs().T
    # float32 itself has steps of 2^-149
    assert bool(((C.double() - ref).abs() <= (41 + 4.0) * 2.0 ** -24 * mag + 41 * 2.0 ** -149).all())


def test_small_gradients(env):
    """The same in weight and input gradients: columns and rows of dH."""
    B, torch = env["B"], env["torch"]
    n, d_in, d_out = 5_000, 70, 140
    print("[case] split gradients of small values", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(4)
    A, dH, W = (torch.randn(*s, generator=gen, device="cuda") for s in ((n, d_in), (n, d_out), (d_out, d_in)))
    dH[:, ::3], dH[17::40] = torch.ldexp(dH[:, ::3], torch.tensor(-118)), torch.ldexp(dH[17::40], torch.tensor(-118))
    d = B.layer_desc(B.GCN, d_in, 0, d_out)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    g = {"W": torch.full_like(W, float("nan")), "bW": torch.full((d_out,), float("nan"), device="cuda")}
    dX = torch.full((n, d_in), float("nan"), device="cuda")
    src = np.arange(0, n, 2, dtype=np.int64)  # pairs: Ahat is the mean of a node and its partner
    P = B.build_partition(n, src, src + 1, 1, 0, 3)
    B.layer_bwd(P, None, 0, d, A, dH, {"W": W, "bW": torch.zeros(d_out, device="cuda")}, {"A": A}, dH, dX, g, False, ws)
    h = dH.double()
    assert bool(((g["W"].double() - h.T @ A.double()).abs() <= (n + 4.0) * 2.0 ** -24 * (h.abs().T @ A.double().abs())
                 + n * 2.0 ** -149).all())
    assert bool(((g["W"].double() - h.T @ A.double()).norm(dim=1) <= 2.0 ** -20 * (h.T @ A.double()).norm(dim=1)).all())

    def pairs(t):
        return (t + t.view(-1, 2, t.shape[1]).flip(1).reshape(t.shape)) / 2.0
    ref, mag = pairs(h @ W.double()), pairs(h.abs() @ W.double().abs())
    assert bool(((dX.double() - ref).abs() <= (d_out + 8.0) * 2.0 ** -24 * mag + d_out * 2.0 ** -149).all())


@pytest.mark.parametrize("nonzero", [1.0, 0.1])
def test_one_rounding_per_step(env, nonzero):
    """The sum of a product is rounded once per 16 k, by a random part of at most half a unit: relative to the result
    2^-24 sqrt(K / 16 / 3) at most, also where most operands are zero (and float32 instructions round less often)."""
    B, torch = env["B"], env["torch"]
    print(f"[case] split product, nonzero {nonzero}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    A, W = (torch.randn(*s, generator=gen, device="cuda") for s in ((20_000, 512), (512, 512)))
    A = A * (torch.rand(A.shape, generator=gen, device="cuda") < nonzero)
    C = torch.full((20_000, 512), float("nan"), device="cuda")
    B.dense_nt_f32(A, W, None, C, False)
    ref = A.double() @ W.double().T
    assert float((C.double() - ref).norm() / ref.norm()) <= 2.0 ** -24 * (512 / 16 / 3) ** 0.5


# 16-node steps of a chunk: 17, 33, 39 and 33 - the sign of the running sum changes every 16
@pytest.mark.parametrize("n,d_in,d_out", [(15_000, 257, 300), (117_003, 257, 300), (140_003, 257, 300), (88_001, 257, 512)])
def test_gradients_of_long_chunks(env, n, d_in, d_out):
    """dW, db and dH_in of an aggregate-first GCN layer on a ring, where Ahat is the mean over a node and its two
    neighbours.  A chunk's sum is rounded once per step and the sum of the chunks once for each, every time by at most
    half a unit of a sum that is no larger than about the result: 2^-24 sqrt(roundings) of its norm."""
    B, torch = env["B"], env["torch"]
    print(f"[case] split gradients of long chunks n={n} {d_in} -> {d_out}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    A, dH, W = (torch.randn(*s, generator=gen, device="cuda") for s in ((n, d_in), (n, d_out), (d_out, d_in)))
    d = B.layer_desc(B.GCN, d_in, 0, d_out)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    g = {"W": torch.full_like(W, float("nan")), "bW": torch.full((d_out,), float("nan"), device="cuda")}
    dX = torch.full((n, d_in), float("nan"), device="cuda")
    B.layer_bwd(ring(env, n), None, 0, d, A, dH, {"W": W, "bW": torch.zeros(d_out, device="cuda")}, {"A": A}, dH, dX, g, False, ws)

    def rel(got, ref):
        return float((got.double() - ref).norm() / ref.norm())
    h = dH.double()
    roundings = 39 + 227
    dW = h.T @ A.double()
    assert rel(g["W"], dW) <= 2.0 ** -24 * roundings ** 0.5
    assert_no_lean(g["W"].double().flatten()[:, None] - dW.flatten()[:, None], "dW")
    assert rel(g["bW"], h.sum(0)) <= 2.0 ** -24 * roundings ** 0.5
    t = h @ W.double()
    ref = (t + t.roll(1, 0) + t.roll(-1, 0)) / 3.0
    assert rel(dX, ref) <= 2.0 ** -24 * ((d_out + 15) // 16) ** 0.5 + 4 * 2.0 ** -24
    assert_no_lean(dX.double() - ref, "dH_in")


@pytest.mark.parametrize("special", ["none", "small", "infinite"])
def test_parameters_split_beforehand(env, special):
    """Both directions of a square conventional GraphSAGE layer large enough that its parameters are split by a launch of
    their own: two ranges of 417 k, a ragged column tile and row tile; some rows of parameters at magnitudes that three
    bfloat16 do not hold, or with an infinity.  On a ring the mean is over two neighbours: one rounding."""
    B, torch = env["B"], env["torch"]
    n, d = 60_001, 417
    print(f"[case] parameters split beforehand, {special}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(17)
    H, dH, W = (torch.randn(*s, generator=gen, device="cuda") for s in ((n, d), (n, d), (d, 2 * d)))
    if special == "small":
        W[::3], W[:, 5::7] = torch.ldexp(W[::3], torch.tensor(-118)), torch.ldexp(W[:, 5::7], torch.tensor(-118))
    if special == "infinite":
        H, dH = H.abs() + 0.1, dH.abs() + 0.1  # no sum of opposite infinities
        W[400, 416] = float("inf")
    b = torch.randn(d, generator=gen, device="cuda")
    P, desc = ring(env, n), B.layer_desc(B.SAGE_CONV, d, 0, d)
    ws = torch.empty(max(B.layer_workspace_bytes(desc, n, x) for x in (False, True)), dtype=torch.uint8, device="cuda")
    prm, sv = {"W": W, "bW": b}, {"A": torch.empty(n, d, device="cuda")}
    Y, dX, g = torch.full_like(H, float("nan")), torch.full_like(H, float("nan")), {k: torch.empty_like(v) for k, v in prm.items()}
    B.layer_fwd(P, None, 0, desc, H, prm, Y, sv, ws)
    B.layer_bwd(P, None, 0, desc, H, Y, prm, sv, dH, dX, g, False, ws)

    def mean(t):
        return (t.roll(1, 0) + t.roll(-1, 0)) / 2.0
    h, gr, w = H.double(), dH.double(), W.double()
    for what, got, ref, mag in (
            ("forward", Y, h @ w[:, :d].T + mean(h) @ w[:, d:].T + b.double(),
             h.abs() @ w[:, :d].abs().T + mean(h.abs()) @ w[:, d:].abs().T + b.double().abs()),
            ("dH_in", dX, gr @ w[:, :d] + mean(gr) @ w[:, d:], gr.abs() @ w[:, :d].abs() + mean(gr.abs()) @ w[:, d:].abs())):
        finite = torch.isfinite(ref)
        assert bool((got[~finite] == ref[~finite]).all()) and bool(torch.isfinite(got[finite]).all()), what
        bound = (2 * d + 8.0) * 2.0 ** -24 * mag + 2 * d * 2.0 ** -149
        assert bool(((got.double() - ref).abs()[finite] <= bound[finite]).all()), what


# few rows: 64 x 64 tiles; eleven to forty times as many: more than 64 tiles of 128 x 128
@pytest.mark.parametrize("M,N,K", [(1, 65, 8), (63, 66, 31), (64, 128, 16), (65, 129, 17), (129, 100, 500), (700, 300, 90), (1_000, 512, 15)])
def test_few_rows_give_the_same_bits(env, M, N, K):
    """A result of few tiles is computed in smaller ones; its sums are formed in the same order."""
    B, torch = env["B"], env["torch"]
    print(f"[case] split product of few rows M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    many = 65 * 128 + M
    A, W, b = (torch.randn(*s, generator=gen, device="cuda") for s in ((many, K), (N, K), (N,)))
    long, few = torch.full((many, N), float("nan"), device="cuda"), torch.full((M + 1, N), float("nan"), device="cuda")
    B.dense_nt_f32(A, W, b, long, True)
    B.dense_nt_f32(A[:M], W, b, few[:M], True)
    assert torch.equal(few[:M], long[:M]) and bool(few[M].isnan().all())


@pytest.mark.parametrize("row,value", [(7, float("inf")), (8_000, float("nan")), (7, 2.0 ** -118), (8_000, 2.0 ** -118)])
def test_blocks_computed_again(env, row, value):
    """What the split does not hold, in tiles of either size: the first 300 rows by themselves and among 10,000."""
    B, torch = env["B"], env["torch"]
    print(f"[case] split product, row {row} of {value}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    A, W = torch.rand(10_000, 41, generator=gen, device="cuda") + 0.1, torch.rand(200, 41, generator=gen, device="cuda") + 0.1
    A[row] = value
    for rows in (300, 10_000):
        C = torch.full((rows, 200), 7.0, device="cuda")
        B.dense_nt_f32(A[:rows], W, None, C, False)
        ref = A[:rows].double() @ W.double().T
        finite = torch.isfinite(ref)
        assert torch.equal(C[~finite].double().nan_to_num(nan=-1.0), ref[~finite].nan_to_num(nan=-1.0)) and bool(torch.isfinite(C[finite]).all())
        assert bool(((C.double() - ref).abs()[finite] <= (41 + 4.0) * 2.0 ** -24 * ref[finite]).all())


@pytest.mark.parametrize("q", [0.0, 0.3])
@pytest.mark.parametrize("kind,d_in,d_out", [("gcn", 100, 70), ("gcn", 70, 129), ("sage", 130, 90), ("sage", 70, 200), ("sage_conv", 70, 130),
                                             ("sage_conv", 200, 66)])
def test_layers_of_few_nodes_give_the_same_bits(env, kind, d_in, d_out, q):
    """Both directions of a layer on one ring and on 30 copies of it: the first copy's rows are the same bits with products in
    64 x 64 tiles and in 128 x 128 ones, through every gate, scale, second range and addition of the layers."""
    B, torch = env["B"], env["torch"]
    print(f"[case] split products of few nodes {kind} {d_in} -> {d_out} q={q}", flush=True)
    one, copies, d_msg = 333, 30, 96 if kind == "sage" else 0
    code = {"gcn": B.GCN, "sage": B.SAGE_MEAN, "sage_conv": B.SAGE_CONV}[kind]
    gen = torch.Generator(device="cuda").manual_seed(d_in)

    def rand(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")
    prm = {"W": rand(d_msg or d_out, d_in * (2 if kind == "sage_conv" else 1)) / d_in ** 0.5, "bW": rand(d_msg or d_out)}
    if kind == "sage":
        prm.update(U=rand(d_out, d_msg + d_in) / d_in ** 0.5, bU=rand(d_out))
    X, G = rand(copies * one, d_in), rand(copies * one, d_out)
    out = []
    for c in (1, copies):
        n = c * one
        src = np.arange(n, dtype=np.int64)
        P = B.build_partition(n, src, src // one * one + (src + 1) % one, 1, 0, 3)
        d = B.layer_desc(code, d_in, d_msg, d_out, act=1, dropout_q=q, layer_id=2, seed=5, epoch=3)
        ws = torch.empty(max(B.layer_workspace_bytes(d, n, x) for x in (False, True)), dtype=torch.uint8, device="cuda")
        sv = {"Z": torch.empty(n, max(d_msg, 1), device="cuda"), "A": torch.empty(n, max(d_msg, d_in, d_out), device="cuda")}
        H, dY = X[:n].clone(), G[:n].clone()
        Y, dX = torch.full((n, d_out), float("nan"), device="cuda"), torch.full((n, d_in), float("nan"), device="cuda")
        grads = {k: torch.empty_like(v) for k, v in prm.items()}
        B.layer_fwd(P, None, 0, d, H, prm, Y, sv, ws)
        B.layer_bwd(P, None, 0, d, H, Y, prm, sv, dY, dX, grads, False, ws)
        out.append((Y[:one], dX[:one]))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
