"""Conventional GraphSAGE layers that transform first, in float32: both products of a layer's input in one launch (blocks of 16 columns
up to 32 columns a result, tiles of 128 beyond), the self part added by the aggregation; against float64, and bit for bit against the
three launches that a workspace without room for a second result takes."""
import numpy as np
import pytest

from paper_2308_03209_amd import inputs

pytestmark = pytest.mark.gpu


def layer(B, torch, P, d_in, d_out, act, q, n, seed, room=None, bad=False):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    H = torch.randn(n, d_in, generator=gen, device="cuda")
    if bad:
        H[n // 2, d_in // 2] = float("inf")
    W = torch.randn(d_out, 2 * d_in, generator=gen, device="cuda") / d_in ** 0.5
    b = torch.randn(d_out, generator=gen, device="cuda")
    d = B.layer_desc(B.SAGE_CONV, d_in, 0, d_out, act=act, dropout_q=q, seed=5)
    size = B.layer_workspace_bytes(d, n, False)
    ws = torch.empty(size if room is None else room, dtype=torch.uint8, device="cuda")
    Y = torch.full((n, d_out), float("nan"), device="cuda")
    B.layer_fwd(P, None, 0, d, H, {"W": W, "bW": b}, Y, {}, ws)
    return H, W, b, Y


def ring(B, n):
    src = np.arange(n, dtype=np.int64)
    return B.build_partition(n, src, (src + 1) % n, 1, 0, 3)


def exact(H, W, b, act):
    d_in = H.shape[1]
    h, w = H.double(), W.double()
    t = h @ w[:, d_in:].T
    y = 0.5 * (t.roll(1, 0) + t.roll(-1, 0)) + h @ w[:, :d_in].T + b.double()
    return y.clamp_(min=0) if act else y


# 16 / 17 and 32 / 33 columns: one and two blocks, blocks and tiles; 64 / 65 and 128 / 129: where the second result begins inside a
# tile; k: less than a step, ragged steps, parameters beyond LDS; rows: one tile, a ragged last one, several rounds
@pytest.mark.parametrize("d_in,d_out", [(4, 1), (5, 3), (9, 4), (20, 16), (33, 17), (70, 32), (1500, 30), (34, 33), (64, 47), (100, 64),
                                        (129, 65), (200, 128), (300, 129), (602, 41)])
@pytest.mark.parametrize("n", [33, 2_005, 40_011])
def test_against_float64(d_in, d_out, n):
    import torch
    from paper_2308_03209_amd import binding as B
    print(f"[case] two results n={n} {d_in} -> {d_out}", flush=True)
    H, W, b, Y = layer(B, torch, ring(B, n), d_in, d_out, 1, 0.0, n, d_in + n)
    ref = exact(H, W, b, 1)
    h, w = H.double().abs(), W.double().abs()
    t = h @ w[:, d_in:].T
    mag = 0.5 * (t.roll(1, 0) + t.roll(-1, 0)) + h @ w[:, :d_in].T + b.double().abs()
    # a float32 sum of d_in products, then the mean, two additions and the result's rounding
    assert bool(((Y.double() - ref).abs() <= (d_in + 8.0) * 2.0 ** -24 * mag).all())


@pytest.mark.parametrize("d_in,d_out", [(64, 16), (200, 48), (64, 33), (200, 41)])
def test_dropout_and_without_room(d_in, d_out):
    """Dropout keeps the same elements, and a workspace without room for a second result gives the same values."""
    import torch
    from paper_2308_03209_amd import binding as B
    n = 3_001
    P = ring(B, n)
    print(f"[case] two results, dropout {d_in} -> {d_out}", flush=True)
    _, _, _, Y = layer(B, torch, P, d_in, d_out, 1, 0.0, n, 3)
    _, _, _, D = layer(B, torch, P, d_in, d_out, 1, 0.5, n, 3)
    T = (n * d_out * 4 + 255) // 256 * 256
    _, _, _, Z = layer(B, torch, P, d_in, d_out, 1, 0.5, n, 3, room=T)
    kept = D != 0
    open_ = Y > 0  # half of them kept, within six deviations of a binomial count
    assert torch.equal(D[kept], 2 * Y[kept])
    assert abs(int(kept[open_].sum()) - int(open_.sum()) / 2) <= 3 * int(open_.sum()) ** 0.5
    clear = (Y > 1e-3) | (Y == 0)  # away from zero both routes agree on the sign
    assert torch.equal(kept[clear], (Z != 0)[clear])
    assert float((D - Z).abs().max()) <= 1e-5


# rows of every degree class, hubs among them; slices: the aggregation's launches (see COFREE_AGG_SLICES)
@pytest.mark.parametrize("slices,widths", [("0", (66, 100, 128, 129)), ("1", (66, 128)), ("2", (68, 128)), ("8", (128, 256))])
@pytest.mark.parametrize("q", [0.0, 0.3])
def test_the_bits_of_three_launches(slices, widths, q, monkeypatch):
    """Products of more than 64 columns are the same tiles in both forms, and mean + (self part + bias) is rounded alike: with
    another order of these additions ReLUs within rounding of zero open or close."""
    import torch
    from paper_2308_03209_amd import binding as B
    monkeypatch.setenv("COFREE_AGG_SLICES", slices)
    src, dst = inputs.hub_graph(5_001, [4_097, 4_095, 1_000, 257, 255, 128, 65, 64, 33, 31, 17, 15], 6_000, 21)
    P = B.build_partition(5_001, src, dst, 1, 0, 1)
    n = P.num_nodes
    for d_out in widths:
        d_in = 2 * d_out + 3
        print(f"[case] two results against three launches, slices {slices}, {d_in} -> {d_out}, dropout {q}", flush=True)
        B.profile_enable(True)
        _, _, _, Y = layer(B, torch, P, d_in, d_out, 1, q, n, d_out)
        names = list(B.profile_read())
        B.profile_enable(False)
        assert sum("gemm" in x for x in names) == 1 and (slices != "0" or any(x.startswith("aggregate_hub_kernel") for x in names)), names
        assert slices in "01" or any(x.startswith("aggregate_sliced_kernel") for x in names), names
        _, _, _, Z = layer(B, torch, P, d_in, d_out, 1, q, n, d_out, room=(n * d_out * 4 + 255) // 256 * 256)
        assert bool(torch.isfinite(Y).all()) and float((Y > 0).float().mean()) > 0.2
        assert torch.equal(Y, Z)


@pytest.mark.parametrize("d_in,d_out", [(70, 20), (70, 40)])
def test_infinite_feature(d_in, d_out):
    import torch
    from paper_2308_03209_amd import binding as B
    n = 501
    print(f"[case] two results, an infinity {d_in} -> {d_out}", flush=True)
    H, W, b, Y = layer(B, torch, ring(B, n), d_in, d_out, 0, 0.0, n, 7, bad=True)
    bad = torch.zeros(n, dtype=torch.bool, device="cuda")
    bad[n // 2 - 1:n // 2 + 2] = True
    assert bool(torch.isfinite(Y[~bad]).all()) and not bool(torch.isfinite(Y[bad]).any())
    ref = exact(H, W, b, 0)
    assert bool((torch.sign(Y[bad]) == torch.sign(ref[bad])).all())
    assert bool(((Y[~bad].double() - ref[~bad]).abs() <= 1e-5).all())
