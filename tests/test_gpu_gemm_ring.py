"""128 x 128 tiles of the projections with one tile a unit (four steps of both operands in LDS, eight waves), against 256 x 192 tiles, which sum
every product in the same order: the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _rnd(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()


# cap, live rows, contraction (1 to 9 steps of 64: fewer than the ring, as many, more; whole and partial), columns; the capacity at the rule's
# line on either side (43520 and 43776 rows of one tile of columns: 255 and 257 tiles by three quarters), with more live tiles than units
@pytest.mark.parametrize("cap,T,K,N", [(1, 1, 8, 8), (300, 0, 64, 64), (130, 129, 120, 136), (400, 256, 192, 128), (200, 128, 248, 200),
                                       (257, 257, 256, 264), (500, 333, 264, 8), (129, 100, 320, 384), (1000, 1, 576, 248),
                                       (43520, 33000, 72, 128), (43776, 33000, 72, 128),
                                       # capacities of more tiles than units: eight waves two a unit up to 320 elements, one a unit beyond
                                       (33000, 30000, 320, 120), (33000, 16000, 8, 128), (16600, 16001, 248, 200), (33000, 30000, 328, 120)])
def test_one_tile_a_unit(cap, T, K, N):
    from paper_2410_23608_amd import spa
    rnd = _rnd(cap + T + K)
    x, W, Wd, b, res, s = rnd(cap, K), rnd(N, K), rnd(K, N), rnd(N), rnd(cap, N), rnd(cap).float()
    idx = torch.randperm(cap, device="cuda")[:T].sort().values
    gi = torch.zeros(cap, dtype=torch.int32, device="cuda")
    gi[:T] = idx.int()
    inv = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    inv[idx] = torch.arange(T, dtype=torch.int32, device="cuda")
    tot = torch.tensor([T], dtype=torch.int32, device="cuda")
    got = []
    for tm in ("2", "10"):
        spa.spa_set_option("gemm_tm", tm)
        try:
            out, y, dx = (torch.full((cap, N), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(3))
            spa.spa_linear_packed(x, gi, s, tot, W, b, out)
            spa.spa_linear_packed_unpack(x, tot, W, b, gi, inv, res, y)
            spa.spa_linear_packed_bwd_input(x, gi, tot, Wd, cap, gi, inv, dx)
        finally:
            spa.spa_set_option("gemm_tm")
        got.append((out, y, dx))
    torch.cuda.synchronize()
    (out, y, dx), (out2, y2, dx2) = got
    assert torch.equal(out[:T], out2[:T]) and torch.isnan(out[T:]).all()
    assert torch.equal(y, y2) and torch.equal(y[inv < 0], res[inv < 0])
    assert torch.equal(dx, dx2) and (dx[inv < 0] == 0).all()
