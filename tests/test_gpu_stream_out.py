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
