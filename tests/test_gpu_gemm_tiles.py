"""The pipelined projection GEMMs at the edges of their tiles: row counts, widths and contraction
lengths on and next to 64 / 128 / 256, one and no live row, every tile shape, one and several token
chunks of the weight side, and the output projection with the scatter and the copy of the other rows;
against products in fp32."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spa():
    from paper_2410_23608_amd import spa as mod
    return mod


def _close(got, ref, tol):
    assert torch.isfinite(got.float()).all()
    err = (got.float() - ref).abs().max().item() if ref.numel() else 0.0
    assert err <= tol * max(1.0, ref.abs().max().item() if ref.numel() else 1.0), err


@pytest.mark.parametrize("tile", ["2", "6", "8"])
@pytest.mark.parametrize("cap,T,K,N", [(40, 0, 64, 64), (40, 1, 8, 8), (300, 127, 64, 128), (300, 129, 72, 136),
                                       (700, 257, 200, 264), (600, 511, 64, 520), (2000, 1025, 328, 248)])
def test_row_gemms_at_tile_edges(spa, tile, cap, T, K, N):
    g = torch.Generator(device="cuda")
    g.manual_seed(cap + T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, W, b, res, d = rnd(cap, K), (rnd(N, K) / K ** 0.5).bfloat16(), rnd(N), rnd(cap, N), rnd(cap, N)
    idx = torch.randperm(cap, generator=g, device="cuda")[:T].sort().values
    inv = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    inv[idx] = torch.arange(T, dtype=torch.int32, device="cuda")
    gi = torch.zeros(cap, dtype=torch.int32, device="cuda")
    gi[:T] = idx.int()
    tot = torch.tensor([T], dtype=torch.int32, device="cuda")
    spa.spa_set_option("gemm_tm", tile)
    try:
        out = torch.full((cap, N), float("nan"), device="cuda", dtype=torch.bfloat16)
        spa.spa_linear_packed(x, gi, None, tot, W, b, out)
        y = torch.full((cap, N), float("nan"), device="cuda", dtype=torch.bfloat16)
        spa.spa_linear_packed_unpack(x, tot, W, b, gi, inv, res, y)
        dx = torch.full((cap, K), float("nan"), device="cuda", dtype=torch.bfloat16)
        spa.spa_linear_packed_bwd_input(d, gi, tot, W, cap, gi, inv, dx)
        torch.cuda.synchronize()
    finally:
        spa.spa_set_option("gemm_tm")
    ref = x[idx].float() @ W.float().T + b.float()
    _close(out[:T], ref, 1e-2)
    assert torch.isnan(out[T:]).all()
    ref_y = res.float().clone()
    ref_y[idx] += (x[:T].float() @ W.float().T + b.float()).bfloat16().float()
    _close(y, ref_y, 1e-2)
    assert torch.equal(y[inv < 0], res[inv < 0])
    ref_dx = torch.zeros(cap, K, device="cuda")
    ref_dx[idx] = d[idx].float() @ W.float()
    _close(dx, ref_dx, 1e-2)
    assert (dx[inv < 0] == 0).all()


@pytest.mark.parametrize("splits", ["1", "2", "5"])
@pytest.mark.parametrize("cap,T,K,N", [(40, 0, 64, 64), (300, 1, 8, 8), (300, 64, 128, 136), (500, 65, 136, 128), (3000, 1281, 264, 392)])
@pytest.mark.parametrize("gather", [False, True])
def test_weight_gemm_at_tile_edges(spa, splits, cap, T, K, N, gather):
    g = torch.Generator(device="cuda")
    g.manual_seed(cap + T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, d = rnd(cap, K), rnd(cap, N)
    x[T:] = float("inf")                                   # rows past the live ones are never multiplied
    rows = torch.randperm(cap, generator=g, device="cuda")[:T] if gather else torch.arange(T, device="cuda")
    gi = torch.zeros(cap, dtype=torch.int32, device="cuda")
    gi[:T] = rows.int()
    tot = torch.tensor([T], dtype=torch.int32, device="cuda")
    spa.spa_set_option("gemm_splits", splits)
    try:
        ws = torch.empty(max(256, spa.spa_linear_bwd_weight_workspace_bytes(cap, K, N, torch.bfloat16)), dtype=torch.uint8,
                         device="cuda")
        dW = torch.full((N, K), float("nan"), device="cuda")
        db = torch.full((N,), float("nan"), device="cuda")
        spa.spa_linear_packed_bwd_weight(d, gi if gather else None, x, None, None, tot, cap, dW, db, ws)
        torch.cuda.synchronize()
    finally:
        spa.spa_set_option("gemm_splits")
    _close(dW, d[rows].float().T @ x[:T].float(), 2e-3)
    _close(db, d[rows].float().sum(0), 2e-3)
