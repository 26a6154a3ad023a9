"""Both weight gradients of a conventional GraphSAGE layer that transforms first, of dPre and mean^T(dPre), in one launch: against
float64, at widths where the second gradient begins inside a tile or a piece of eight columns, with a ragged number of nodes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d_in,d_out", [("f32", 66, 33), ("f32", 129, 64), ("f32", 200, 65), ("f32", 300, 128), ("f32", 602, 129),
                                              ("bf16", 12, 8), ("bf16", 40, 9), ("bf16", 100, 33), ("bf16", 129, 64), ("bf16", 256, 65),
                                              ("bf16", 300, 128), ("bf16", 300, 129)])
@pytest.mark.parametrize("n", [33, 2_005, 40_011])
@pytest.mark.parametrize("accumulate", [False, True])
def test_against_float64(dtype, d_in, d_out, n, accumulate):
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] two gradients {dtype} n={n} {d_in} -> {d_out}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(d_in + n)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    # multiples of 1/4: the mean of two neighbours is exact in bfloat16 too, and so are products; sums of n of them are not
    H = (torch.randint(-8, 9, (n, d_in), generator=gen, device="cuda") * 0.25).to(td)
    dO = (torch.randint(-8, 9, (n, d_out), generator=gen, device="cuda") * 0.25).to(td)
    W = torch.zeros(d_out, 2 * d_in, device="cuda")
    b = torch.zeros(d_out, device="cuda")
    d = B.layer_desc(B.SAGE_CONV, d_in, 0, d_out, dtype=B.F32 if dtype == "f32" else B.BF16)
    ws = torch.full((B.layer_workspace_bytes(d, n, True),), 0xff, dtype=torch.uint8, device="cuda")
    before = {"W": torch.ones(d_out, 2 * d_in, device="cuda"), "bW": torch.ones(d_out, device="cuda")}
    g = {k: v.clone() for k, v in before.items()}
    B.layer_bwd(P, None, 0, d, H, dO, {"W": W, "bW": b}, {}, dO, None, g, accumulate, ws)
    h, z = H.double(), dO.double()
    t = 0.5 * (z.roll(1, 0) + z.roll(-1, 0))
    ref = torch.cat([z.T @ h, t.T @ h], 1)
    mag = torch.cat([z.abs().T @ h.abs(), t.abs().T @ h.abs()], 1)
    base = 1.0 if accumulate else 0.0
    assert bool(((g["W"].double() - base - ref).abs() <= (n + 8.0) * 2.0 ** -24 * (mag + base)).all())
    assert bool(((g["bW"].double() - base - z.sum(0)).abs() <= (n + 8.0) * 2.0 ** -24 * (z.abs().sum(0) + base)).all())


@pytest.mark.parametrize("dtype,d_in,d_out", [("f32", 66, 33), ("f32", 129, 64), ("f32", 200, 65), ("f32", 300, 128), ("f32", 602, 129),
                                              ("bf16", 12, 8), ("bf16", 40, 9), ("bf16", 100, 33), ("bf16", 129, 64), ("bf16", 256, 65),
                                              ("bf16", 300, 128), ("bf16", 300, 129)])
@pytest.mark.parametrize("n", [33, 2_005, 40_011])
@pytest.mark.parametrize("accumulate", [False, True])
def test_exact_sums(dtype, d_in, d_out, n, accumulate):
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] two gradients {dtype} n={n} {d_in} -> {d_out}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(d_in + n)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    # multiples of 1/4: the mean of two neighbours is exact in bfloat16 too, products are multiples of 1/32 of at most 4, and n of them
    # stay below 2^24 / 32: every partial sum is exact, in any order
    H = (torch.randint(-8, 9, (n, d_in), generator=gen, device="cuda") * 0.25).to(td)
    dO = (torch.randint(-8, 9, (n, d_out), generator=gen, device="cuda") * 0.25).to(td)
    W = torch.zeros(d_out, 2 * d_in, device="cuda")
    b = torch.zeros(d_out, device="cuda")
    d = B.layer_desc(B.SAGE_CONV, d_in, 0, d_out, dtype=B.F32 if dtype == "f32" else B.BF16)
    ws = torch.full((B.layer_workspace_bytes(d, n, True),), 0xff, dtype=torch.uint8, device="cuda")
    before = {"W": torch.ones(d_out, 2 * d_in, device="cuda"), "bW": torch.ones(d_out, device="cuda")}
    g = {k: v.clone() for k, v in before.items()}
    B.layer_bwd(P, None, 0, d, H, dO, {"W": W, "bW": b}, {}, dO, None, g, accumulate, ws)
    h, z = H.double(), dO.double()
    t = 0.5 * (z.roll(1, 0) + z.roll(-1, 0))
    ref = torch.cat([z.T @ h, t.T @ h], 1)
    base = 1.0 if accumulate else 0.0
    assert torch.equal(g["W"].double(), base + ref)
    assert torch.equal(g["bW"].double(), base + z.sum(0))


@pytest.mark.parametrize("dtype,n,d_in,d_out", [("f32", 5_003, 200, 100), ("f32", 40_011, 129, 47), ("bf16", 5_003, 100, 47)])
def test_a_second_stream_has_dW_self(dtype, n, d_in, d_out, monkeypatch):
    """With COFREE_OVERLAP=1 dW_self, which does not wait for the aggregation, is a launch of its own on the second stream."""
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] two gradients on two streams {dtype} n={n} {d_in} -> {d_out}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(n)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    H = (torch.randint(-8, 9, (n, d_in), generator=gen, device="cuda") * 0.25).to(td)
    # products are multiples of 1/32 of at most 4: every partial sum is exact
    dO = (torch.randint(-8, 9, (n, d_out), generator=gen, device="cuda") * 0.25).to(td)
    p = {"W": torch.zeros(d_out, 2 * d_in, device="cuda"), "bW": torch.zeros(d_out, device="cuda")}
    d = B.layer_desc(B.SAGE_CONV, d_in, 0, d_out, dtype=B.F32 if dtype == "f32" else B.BF16)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    got = []
    for overlap, launches in (("0", 1), ("1", 2)):
        monkeypatch.setenv("COFREE_OVERLAP", overlap)
        g = {k: torch.full_like(v, float("nan")) for k, v in p.items()}
        B.profile_enable(True)
        B.layer_bwd(P, None, 0, d, H, dO, p, {}, dO, None, g, False, ws)
        stats = B.profile_read()
        B.profile_enable(False)
        assert sum(v["launches"] for k, v in stats.items() if f"x{d_in}" in k) == launches, list(stats)
        got.append(g)
    assert all(torch.equal(got[0][k], got[1][k]) for k in p)


# pairs of tiles that one gradient alone would cut into more chunks: tiles of 128 rows (float32), of up to 256 (bfloat16); 64 and less: the same tiles
@pytest.mark.parametrize("dtype,n,d_in,d_out", [("f32", 115_001, 602, 256), ("f32", 150_001, 512, 100), ("f32", 40_003, 300, 128), ("f32", 9_001, 140, 66),
                                                ("bf16", 150_001, 300, 128), ("bf16", 70_001, 256, 100), ("bf16", 300_001, 200, 64)])
def test_sums_as_short_as_one_gradients(dtype, n, d_in, d_out, monkeypatch):
    """Both gradients and the bias gradient have the bits of launches of their own (COFREE_OVERLAP=1): as many chunks of nodes."""
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] sums of two gradients {dtype} n={n} {d_in} -> {d_out}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(n)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    H = torch.randn(n, d_in, generator=gen, device="cuda").to(td)
    dO = torch.randn(n, d_out, generator=gen, device="cuda").to(td)
    p = {"W": torch.zeros(d_out, 2 * d_in, device="cuda"), "bW": torch.zeros(d_out, device="cuda")}
    d = B.layer_desc(B.SAGE_CONV, d_in, 0, d_out, dtype=B.F32 if dtype == "f32" else B.BF16)
    room = B.layer_workspace_bytes(d, n, True)
    ws = torch.full((room + 4096,), 0xa5, dtype=torch.uint8, device="cuda")
    got = []
    for overlap in ("0", "1"):
        monkeypatch.setenv("COFREE_OVERLAP", overlap)
        g = {k: torch.full_like(v, float("nan")) for k, v in p.items()}
        B.layer_bwd(P, None, 0, d, H, dO, p, {}, dO, None, g, False, ws[:room])
        got.append(g)
    assert bool((ws[room:] == 0xa5).all())
    assert all(bool(torch.isfinite(got[0][k]).all()) and torch.equal(got[0][k], got[1][k]) for k in p)


# rms of both gradients' and the bias gradient's errors over eight draws, in 1e-7 of their norms, where gemm_narrow.hip's pair computes them
@pytest.mark.parametrize("n,d_in,d_out,pair", [(40_000, 100, 64, (1.82, 1.83, 1.39)), (200_000, 70, 50, (2.97, 3.00, 1.66)),
                                               (115_000, 256, 41, (2.56, 2.55, 1.56))])
def test_narrow_gradients_are_as_accurate_as_the_pairs(n, d_in, d_out, pair):
    """Sums of float32 partials over up to 512 chunks had up to 1.11 times its error in dW, chains of a chunk's nodes 1.41 times in db."""
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] accuracy of two gradients n={n} {d_in} -> {d_out}", flush=True)
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    p = {"W": torch.zeros(d_out, 2 * d_in, device="cuda"), "bW": torch.zeros(d_out, device="cuda")}
    d = B.layer_desc(B.SAGE_CONV, d_in, 0, d_out)
    ws = torch.empty(B.layer_workspace_bytes(d, n, True), dtype=torch.uint8, device="cuda")
    g, err, size = {k: torch.empty_like(v) for k, v in p.items()}, [0.0] * 3, [0.0] * 3
    for seed in range(8):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        H = torch.randn(n, d_in, generator=gen, device="cuda")
        dO = torch.randn(n, d_out, generator=gen, device="cuda")
        B.layer_bwd(P, None, 0, d, H, dO, p, {}, dO, None, g, False, ws)
        h, z = H.double(), dO.double()
        t = 0.5 * (z.roll(1, 0) + z.roll(-1, 0))
        for i, (got, ref) in enumerate(((g["W"][:, :d_in], z.T @ h), (g["W"][:, d_in:], t.T @ h), (g["bW"], z.sum(0)))):
            err[i] += float((got.double() - ref).square().sum())
            size[i] += float(ref.square().sum())
    assert all((e / s) ** 0.5 <= most * 1e-7 for e, s, most in zip(err, size, pair)), [(e / s) ** 0.5 for e, s in zip(err, size)]
