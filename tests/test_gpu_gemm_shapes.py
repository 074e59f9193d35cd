"""The projection GEMMs with large tiles, 192 x 192, 256 x 256 and the shape that the row count decides on the device
(192 x 192 with fewer rounds of the units, or one each), one and several tiles per resident workgroup, rows, columns and contraction on
and next to the tile edges; against products in fp64.

Bound: both sides take the same bf16 operands; the products are summed in fp32 (K terms, error below K 2^-24 sum |a b|)
and the result is rounded to bf16 once (2^-9 of its size), the residual sum once more (2^-9 of its size)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# cap, live rows, contraction, columns: 192 x 192 in one round; edges of 192 and of a deep block of 64; two rounds of it;
# 256 x 256 in one round where 192 x 192 takes two; and its edges; two rounds of each
SHAPES = [(500, 384, 64, 192), (500, 193, 136, 328), (400, 191, 8, 200), (4300, 4225, 72, 2312),
          (4400, 4097, 72, 3840), (4400, 4351, 136, 3768), (8300, 8193, 64, 3848)]


@pytest.mark.parametrize("cap,T,K,N", SHAPES)
@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("tile", ["14", "6", "8"])
def test_row_gemms_of_every_tile_shape(cap, T, K, N, ordered, tile):
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(cap + T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, W, b, res, d = rnd(cap, K), rnd(N, K), rnd(N), rnd(cap, N), rnd(cap, K)
    Wd = rnd(K, N)
    idx = torch.randperm(cap, generator=g, device="cuda")[:T].sort().values
    gi = torch.zeros(cap, dtype=torch.int32, device="cuda")
    gi[:T] = idx.int()
    inv = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    inv[idx] = torch.arange(T, dtype=torch.int32, device="cuda")
    s = torch.randn(cap, generator=g, device="cuda")
    tot = torch.tensor([T], dtype=torch.int32, device="cuda")
    rows = torch.arange(T, device="cuda") if ordered else idx
    spa.spa_set_option("gemm_tm", tile)
    try:
        out = torch.full((cap, N), float("nan"), device="cuda", dtype=torch.bfloat16)
        spa.spa_linear_packed(x, None if ordered else gi, None if ordered else s, tot, W, b, out)
        y = torch.full((cap, N), float("nan"), device="cuda", dtype=torch.bfloat16)
        spa.spa_linear_packed_unpack(x, tot, W, b, gi, inv, res, y)
        dx = torch.full((cap, N), float("nan"), device="cuda", dtype=torch.bfloat16)
        spa.spa_linear_packed_bwd_input(d, None if ordered else gi, tot, Wd, cap, gi, inv, dx)
        torch.cuda.synchronize()
    finally:
        spa.spa_set_option("gemm_tm")

    def check(got, a, w, add, more=None):
        scale = torch.ones(T, 1, device="cuda") if more is None else more
        ref = (a.double() @ w.double()) * scale.double() + add.double()
        size = (a.double().abs() @ w.double().abs()) * scale.double() + add.double().abs()
        bound = K * 2.0 ** -24 * size + 2.0 ** -22 * size + 2.0 ** -8 * ref.abs() + 2.0 ** -8 * add.double().abs() + 1e-30
        assert ((got.double() - ref).abs() <= bound).all()

    check(out[:T], x[rows], W.T, b.expand(T, N), None if ordered else torch.sigmoid(s.double())[rows, None])
    assert torch.isnan(out[T:]).all()
    prod = x[:T].double() @ W.double().T + b.double()
    size = x[:T].double().abs() @ W.double().abs().T + b.double().abs()
    bound = (K + 4) * 2.0 ** -24 * size + 2.0 ** -8 * (2 * prod.abs() + res[idx].double().abs())
    assert ((y[idx].double() - prod - res[idx].double()).abs() <= bound).all()
    assert torch.equal(y[inv < 0], res[inv < 0])
    check(dx[idx], d[rows], Wd, torch.zeros(T, N, device="cuda"))
    assert (dx[inv < 0] == 0).all()


@pytest.mark.parametrize("T,K,N", [(1001, 1032, 1544), (4225, 264, 2312), (130, 2304, 768)])
def test_every_shape_gives_the_same_bits(T, K, N):
    """A product sums in the same order whatever the tile (both matrix instructions add their elements in the same
    order): which shape the row count or the capacity chooses does not show in the results."""
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, W, Wd, b, tot = rnd(T, K), rnd(N, K), rnd(K, N), rnd(N), torch.tensor([T], dtype=torch.int32, device="cuda")
    s, idx = torch.randn(T, generator=g, device="cuda"), torch.randperm(T, generator=g, device="cuda").int()
    got = []
    for tile in ("2", "6", "8", "14"):
        spa.spa_set_option("gemm_tm", tile)
        try:
            out = [torch.empty(T, N, device="cuda", dtype=torch.bfloat16) for _ in range(2)]
            spa.spa_linear_packed(x, idx, s, tot, W, b, out[0])
            spa.spa_linear_packed_bwd_input(x, idx, tot, Wd, T, None, None, out[1])
        finally:
            spa.spa_set_option("gemm_tm")
        got.append(out)
    torch.cuda.synchronize()
    for other in got[1:]:
        assert torch.equal(got[0][0], other[0]) and torch.equal(got[0][1], other[1])
