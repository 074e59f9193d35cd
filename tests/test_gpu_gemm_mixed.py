"""256 x 192 tiles of the projection GEMMs, launches of 256 x 256 tiles whose last rows take 256 x 192, and the rows of out that no packed
row maps to, in all their shares; against 128 x 128 tiles, which sum every product in the same order: the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# cap, live rows, contraction (1 to 10 steps of 64, whole and partial), columns.  By the rule (14): one or two whole rounds of 256 x 256 and
# one or two of 256 x 192 behind them, in all three calls (tests/test_large_plan.py asks the rule).
SPLIT = [(11000, 10913, 584, 2304), (12300, 12193, 200, 2304), (12460, 12449, 8, 2304), (16600, 16545, 72, 2304), (23600, 23554, 136, 1544),
         (32800, 32770, 264, 768)]
# 192 x 192 or 256 x 192 alone: edges, few rows, their copy left to units with a tile and without; one row; none.
SHAPES = SPLIT + [(500, 257, 8, 192), (700, 511, 64, 200), (900, 769, 136, 376), (300, 256, 264, 584), (300, 1, 328, 8), (64, 0, 64, 64),
          (4400, 4097, 72, 4096), (4400, 4351, 200, 4088), (9000, 4609, 64, 4096), (30000, 300, 64, 1024), (9000, 8300, 64, 768)]


@pytest.mark.parametrize("tile", ["10", "14"])
@pytest.mark.parametrize("cap,T,K,N", SHAPES)
def test_same_bits_as_small_tiles(cap, T, K, N, tile):
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(cap + T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, W, Wd, b, res, s = rnd(cap, K), rnd(N, K), rnd(K, N), rnd(N), rnd(cap, N), torch.randn(cap, generator=g, device="cuda")
    idx = torch.randperm(cap, generator=g, device="cuda")[:T].sort().values
    gi = torch.zeros(cap, dtype=torch.int32, device="cuda")
    gi[:T] = idx.int()
    inv = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    inv[idx] = torch.arange(T, dtype=torch.int32, device="cuda")
    tot = torch.tensor([T], dtype=torch.int32, device="cuda")
    got = []
    for tm in ("2", tile):
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
    assert torch.equal(out[:T], out2[:T]) and torch.isnan(out2[T:]).all()
    assert torch.equal(y, y2) and torch.equal(y2[inv < 0], res[inv < 0])
    assert torch.equal(dx, dx2) and (dx2[inv < 0] == 0).all()
