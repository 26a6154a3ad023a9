"""The losses at the edges of their groups of lanes and pieces of 16 bytes, over few and many nodes, against float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def setup(torch, B, n, C, dtype, seed):
    src = np.arange(n, dtype=np.int64)
    P = B.build_partition(n, src, (src + 1) % n, 1, 0, 3) if n > 2 else B.build_partition(3, src[:1] * 0, src[:1] + 1, 1, 0, 3)
    n = P.num_nodes
    gen = torch.Generator(device="cuda").manual_seed(seed)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    z = (3 * torch.randn(n, C, generator=gen, device="cuda")).to(td)
    w = torch.rand(n, generator=gen, device="cuda") + 0.1
    mask = (torch.rand(n, generator=gen, device="cuda") < 0.7).to(torch.uint8)
    mask[0] = 1
    room = torch.full((n * C + 64,), 7.0, device="cuda", dtype=td)  # a store past the end is seen
    ws = torch.full((B.loss_workspace_bytes(),), 0xff, dtype=torch.uint8, device="cuda")
    return P, n, gen, z, w, mask, room, ws, torch.full((1,), float("nan"), device="cuda"), B.F32 if dtype == "f32" else B.BF16


def check(torch, dtype, C, n, z, room, loss, k, each, mag, grad):
    """Softmax and sigmoid to a few units of float32 (the exponent's argument is rounded: |z| < 40), the gradient rounded
    once more where it is stored, the loss a float32 sum in chains of at most 64 terms and trees above them."""
    got = room[: n * C].view(n, C).double()
    eps = 2.0 ** -24 if dtype == "f32" else 2.0 ** -8
    assert bool(((got - grad).abs() <= eps * grad.abs() + (C / 8 + 64) * 2.0 ** -24 * k[:, None].abs()).all())
    assert bool((room[n * C:] == 7.0).all())
    assert abs(float(loss) - float((k * each).sum())) <= (C / 8 + 128) * 2.0 ** -24 * float((k.abs() * mag).sum())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C", [1, 3, 4, 5, 7, 8, 9, 16, 17, 31, 33, 63, 65, 127, 129, 255, 257, 511, 513, 1024, 1025])
@pytest.mark.parametrize("n", [1, 130, 3_001])
def test_softmax(C, dtype, n):
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] softmax loss n={n} C={C} {dtype}", flush=True)
    P, n, gen, z, w, mask, room, ws, loss, code = setup(torch, B, n, C, dtype, C)
    y = torch.randint(0, C, (n,), generator=gen, device="cuda", dtype=torch.int32)
    y[n // 2] = C  # outside: does not contribute
    if C > 2:
        z[n - 1, C - 1], y[n - 1] = float("-inf"), 0
    B.loss_weighted(P, B.W_CUSTOM, w, z, y, mask, C, 0.37, loss, room, ws, code)
    known = (y < C)
    k = 0.37 * w.double() * mask * known
    z64, yy = z.double(), torch.where(known, y, 0).long()
    p = torch.softmax(z64, 1)
    each = torch.logsumexp(z64, 1) - z64.gather(1, yy[:, None])[:, 0]
    hot = torch.zeros_like(p).scatter_(1, yy[:, None], 1.0)
    check(torch, dtype, C, n, z, room, loss, k, each, each + 40, k[:, None] * (p - hot))


# C: the widest rows of a group of 1, 1, 2, 4, ... 64 lanes, then of a wavefront.  A workgroup takes 512 / lanes rows at a time (a wavefront
# a row: four) and there are 1,280 of them at most (2,048): one row more is a second iteration of one group, its other row past the
# run's end, and leaves the last workgroups without rows; some more is two iterations and a ragged third.
@pytest.mark.parametrize("C,dtype,lanes", [(c * w, d, l) for d, w in (("f32", 4), ("bf16", 8))
                                           for c, l in ((1, 1), (2, 1), (4, 2), (8, 4), (16, 8), (32, 16), (64, 32), (128, 64), (129, 0))])
@pytest.mark.parametrize("more", ["one", "some"])
def test_softmax_of_several_iterations(C, dtype, lanes, more):
    once = 1_280 * 512 // lanes if lanes else 2_048 * 4
    test_softmax(C - 1 if C > 4 and lanes else C, dtype, once + 1 if more == "one" else 2 * once + once // 3 + 5)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C", [1, 2, 3, 4, 5, 41, 100, 1027])
@pytest.mark.parametrize("n", [1, 130, 3_001])
def test_sigmoid(C, dtype, n):
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] sigmoid loss n={n} C={C} {dtype}", flush=True)
    P, n, gen, z, w, mask, room, ws, loss, code = setup(torch, B, n, C, dtype, C)
    z[0] *= 20
    t = (torch.rand(n, C, generator=gen, device="cuda") < 0.3).to(torch.uint8)
    B.loss_bce_weighted(P, B.W_CUSTOM, w, z, t, mask, C, 0.37, loss, room, ws, code)
    k = 0.37 * w.double() * mask
    z64 = z.double()
    each = torch.nn.functional.softplus(z64) - t * z64
    check(torch, dtype, C, n, z, room, loss, k, each.sum(1), (each.abs() + z64.abs()).sum(1), k[:, None] * (torch.sigmoid(z64) - t))


def test_softplus_of_any_size():
    """One node: the loss of one logit to a few units of float32, where 1 + e^-|z| rounds to 1, to 2 and between."""
    import torch
    from paper_2308_03209_amd import binding as B
    print("[case] softplus", flush=True)
    src = np.zeros(1, dtype=np.int64)
    P = B.build_partition(2, src, src + 1, 1, 0, 3)
    ws = torch.empty(B.loss_workspace_bytes(), dtype=torch.uint8, device="cuda")
    loss, t = torch.empty(1, device="cuda"), torch.zeros(P.num_nodes, 1, dtype=torch.uint8, device="cuda")
    mask = torch.zeros(P.num_nodes, dtype=torch.uint8, device="cuda")
    mask[0] = 1
    for v in (0.0, -1e-6, -1e-3, -0.1, -1.0, -2.5, -5.0, -9.0, -12.0, -16.0, -16.7, -17.5, -30.0, -80.0, 0.5, 3.0, 17.0, 200.0):
        z = torch.full((P.num_nodes, 1), v, device="cuda")
        B.loss_bce_weighted(P, B.W_NONE, None, z, t, mask, 1, 1.0, loss, torch.empty_like(z), ws)
        ref = float(torch.nn.functional.softplus(z[0, 0].double(), threshold=1e9))
        assert abs(float(loss) - ref) <= 6 * 2.0 ** -24 * ref + 2.0 ** -149, v


# 2,048 workgroups take 2,097,152 elements at a time: a thread's second and third pieces, rows of one, two and more elements
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C,n", [(1, 2_097_155), (2, 1_050_001), (3, 700_001), (100, 50_003), (1027, 2_045)])
def test_sigmoid_of_several_iterations(C, n, dtype):
    test_sigmoid(C, dtype, n)
