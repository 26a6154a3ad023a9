"""Results that are written past the caches (160 MB and more): the same values as below that size, ragged rows included, and the
next launch reads them."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,width", [("f32", 100), ("f32", 256), ("bf16", 47), ("bf16", 128)])
def test_large_results(dtype, width):
    import numpy as np
    import torch
    from paper_2308_03209_amd import binding as B
    td, code = (torch.float32, B.F32) if dtype == "f32" else (torch.bfloat16, B.BF16)
    es = 4 if dtype == "f32" else 2
    n = int(170e6) // (width * es) | 1
    print(f"[case] result past the caches {dtype} {n} x {width}", flush=True)
    src = np.arange(n, dtype=np.int64)
    ring = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    ids = torch.from_numpy(ring.host_array(B.ARR_LOCAL2GLOBAL)).cuda()
    assert torch.equal(ids, torch.arange(n, device="cuda"))
    gen = torch.Generator(device="cuda").manual_seed(width)
    # multiples of 2^-4 below 2^3: sums and halves of neighbours are exact in either type
    X = (torch.randint(-8, 8, (n, width), generator=gen, device="cuda") * 0.5).to(td)
    Y, Z = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
    B.aggregate(ring, None, 0, B.AGG_MEAN, X, Y, width, code)
    B.aggregate(ring, None, 0, B.AGG_MEAN, Y, Z, width, code)

    def mean(v):
        return (v.roll(1, 0).float() + v.roll(-1, 0).float()) * 0.5

    assert torch.equal(Y.float(), mean(X))
    assert torch.equal(Z.float(), mean(mean(X)))


@pytest.mark.parametrize("dtype,width,n", [("f32", 260, 250_001), ("f32", 381, 165_001), ("bf16", 520, 200_001), ("bf16", 765, 140_001)])
def test_wide_rows_in_two_launches(dtype, width, n):
    """Rows of 65 to 96 pieces of 16 bytes in a large matrix: the columns at the seam and at the ragged end."""
    import numpy as np
    import torch
    from paper_2308_03209_amd import binding as B
    td, code = (torch.float32, B.F32) if dtype == "f32" else (torch.bfloat16, B.BF16)
    print(f"[case] two launches {dtype} {n} x {width}", flush=True)
    src = np.arange(n, dtype=np.int64)
    ring = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(width)
    X = (torch.randint(-8, 8, (n, width), generator=gen, device="cuda") * 0.5).to(td)
    Y = torch.full_like(X, float("nan"))
    B.aggregate(ring, None, 0, B.AGG_MEAN, X, Y, width, code)
    assert torch.equal(Y.float(), (X.roll(1, 0).float() + X.roll(-1, 0).float()) * 0.5)


@pytest.mark.parametrize("dtype,width,n", [("f32", 261, 240_001), ("bf16", 525, 191_001)])
def test_dropout_at_the_seam_of_two_launches(dtype, width, n):
    """A GCN layer that transforms first: rows of 66 pieces in two launches, whose lanes begin inside draws of the generator."""
    import numpy as np
    import torch
    from oracle import counter_rng as crng
    from paper_2308_03209_amd import binding as B
    td, code = (torch.float32, B.F32) if dtype == "f32" else (torch.bfloat16, B.BF16)
    print(f"[case] dropout in two launches {dtype} {n} x {width}", flush=True)
    src = np.arange(n, dtype=np.int64)
    ring = B.build_partition(n, src, (src + 1) % n, 1, 0, 3)
    gen = torch.Generator(device="cuda").manual_seed(width)
    d_in, q, seed = width + 3, 0.3, 2 ** 40 + 9
    H = torch.randn(n, d_in, generator=gen, device="cuda").to(td)
    p = {"W": torch.randn(width, d_in, generator=gen, device="cuda") / d_in ** 0.5, "bW": torch.randn(width, generator=gen, device="cuda")}
    out = []
    for rate in (0.0, q):
        d = B.layer_desc(B.GCN, d_in, 0, width, act=1, dropout_q=rate, layer_id=3, seed=seed, epoch=6, dtype=code)
        Y = torch.full((n, width), float("nan"), dtype=td, device="cuda")
        B.profile_enable(True)
        B.layer_fwd(ring, None, 0, d, H, p, Y, {}, torch.empty(B.layer_workspace_bytes(d, n, False), dtype=torch.uint8, device="cuda"))
        stats = {k: v["launches"] for k, v in B.profile_read().items()}
        B.profile_enable(False)
        assert sum(v for k, v in stats.items() if k.startswith("aggregate_kernel")) == 2, stats
        assert not any(k.startswith("mask_grad") for k in stats), stats
        out.append(Y)
    rows = torch.cat([torch.arange(500), torch.randint(0, n, (2_000,), generator=torch.Generator().manual_seed(1)), torch.arange(n - 500, n)])
    e = rows.numpy().astype(np.uint64)[:, None] * np.uint64(width) + np.arange(width, dtype=np.uint64)
    words = np.stack(crng.words(seed, crng.STREAM_DROPOUT + 256 * 3, e // 4, 6), -1)
    word = np.take_along_axis(words, (e % 4).astype(np.int64)[..., None], -1)[..., 0]
    keep = torch.from_numpy(word >= np.uint32(crng.threshold(float(np.float32(q))))).cuda()
    plain, got = (y[rows.cuda()].double() for y in out)
    want = torch.where(keep, plain * float(np.float32(1.0 / (1.0 - np.float32(q)))), 0.0)
    assert bool(torch.isfinite(plain).all()) and bool((got[~keep] == 0).all())
    # float32: one more product; bfloat16: both runs round once, by at most 2^-8
    assert bool(((got - want).abs() <= (2e-7 if dtype == "f32" else 2.0 ** -7) * want.abs()).all())
