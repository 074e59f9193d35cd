"""The weight side of the projections' backward in 256 x 256 tiles: chunk ends and widths on and next to tile edges, rows in
order and named by an index on either side, no live row; the same bits as 128 x 128 tiles with as many chunks, and two
calls of a group in one launch the same as each alone."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spa():
    from paper_2410_23608_amd import spa as mod
    yield mod
    mod.spa_set_option("gemm_tm")
    mod.spa_set_option("gemm_splits")


def _operands(cap, T, K, N, gi, xi):
    g = torch.Generator(device="cuda")
    g.manual_seed(cap + T)
    x, d = (torch.randn(cap, w, generator=g, device="cuda").bfloat16() for w in (K, N))
    rows = lambda named: torch.randperm(cap, generator=g, device="cuda")[:T] if named else torch.arange(T, device="cuda")
    idx = lambda r: torch.cat([r, torch.zeros(cap - T, dtype=r.dtype, device="cuda")]).int()
    rg, rx = rows(gi), rows(xi)
    return x, d, rg, rx, idx(rg) if gi else None, idx(rx) if xi else None, torch.tensor([T], dtype=torch.int32, device="cuda")


def _call(spa, cap, K, N, x, d, gi, xi, tot):
    ws = torch.empty(max(256, spa.spa_linear_bwd_weight_workspace_bytes(cap, K, N, torch.bfloat16)), dtype=torch.uint8, device="cuda")
    dW, db = torch.full((N, K), float("nan"), device="cuda"), torch.full((N,), float("nan"), device="cuda")
    return dW, db, spa.spa_linear_packed_bwd_weight(d, gi, x, xi, None, tot, cap, dW, db, ws, prepare=True)


@pytest.mark.parametrize("gi,xi", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("splits", ["1", "3"])
@pytest.mark.parametrize("cap,T,K,N", [(40, 0, 64, 64), (300, 1, 8, 8), (300, 64, 256, 264), (500, 193, 248, 256), (3000, 1281, 264, 520)])
def test_large_tiles(spa, cap, T, K, N, splits, gi, xi):
    x, d, rg, rx, ig, ix, tot = _operands(cap, T, K, N, gi, xi)
    if not gi and not xi:
        x[T:] = float("inf")                               # rows past the live ones are never multiplied
    got = []
    spa.spa_set_option("gemm_splits", splits)
    for tm in ("8", "2"):
        spa.spa_set_option("gemm_tm", tm)
        dW, db, call = _call(spa, cap, K, N, x, d, ig, ix, tot)
        call()
        torch.cuda.synchronize()
        got.append((dW, db))
    ref, ref_b = d[rg].double().T @ x[rx].double(), d[rg].double().sum(0)
    # fp32 sums of T products of ~1 in chunks: 2^-24 a step of 16, over sqrt(T) as the size of the result
    tol = 2.0 ** -24 * (T / 16 + 16) * 4
    assert (got[0][0].double() - ref).abs().max() <= tol * max(1.0, T ** 0.5)
    assert (got[0][1].double() - ref_b).abs().max() <= tol * max(1.0, T ** 0.5)
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("cap,T,C", [(700, 401, 72), (5200, 2601, 264)])
def test_two_calls_of_a_group_in_one_launch(spa, cap, T, C):
    a = _operands(cap, T, C, C, True, False)
    b = _operands(cap + 1, T, C, 3 * C, False, False)
    spa.spa_set_option("gemm_tm", "8")
    spa.spa_set_option("gemm_splits", "2")
    one = [_call(spa, cap, C, C, a[0], a[1], a[4], None, a[6]), _call(spa, cap + 1, C, 3 * C, b[0], b[1], None, None, b[6])]
    two = [_call(spa, cap, C, C, a[0], a[1], a[4], None, a[6]), _call(spa, cap + 1, C, 3 * C, b[0], b[1], None, None, b[6])]
    for _, _, call in one:
        call()
    spa.group(*(call for _, _, call in two))()
    torch.cuda.synchronize()
    for (dW, db, _), (eW, eb, _) in zip(one, two):
        assert torch.equal(dW, eW) and torch.equal(db, eb) and torch.isfinite(dW).all()
