"""The weight side of the projections' backward in 256 x 256 tiles: chunk ends and widths on and next to tile edges, rows in
order and named by an index on either side, no live row; the same bits as 128 x 128 tiles with as many chunks, and two
calls of a group in one launch the same as each alone, by the default rules too, beside the input side or not."""
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


@pytest.mark.parametrize("cap,T,C", [(2049, 1000, 64), (3000, 3000, 136), (6272, 3136, 384), (6272, 3001, 768), (6100, 0, 1024), (12544, 0, 768),
                                     (12544, 6273, 768), (12544, 12544, 768), (25088, 11000, 520), (6300, 3200, 1000), (8192, 4100, 1032)])
def test_a_group_by_the_default_rules(spa, cap, T, C):
    """The weight sides of a block, gathered C x C and 3 C x C: alone, as a group of their own and with the input side, the
    same bits on both sides of 2.4e10 multiplications; and the sums themselves."""
    spa.spa_set_option("gemm_tm")
    spa.spa_set_option("gemm_splits")
    a = _operands(cap, T, C, C, True, False)
    b = _operands(cap, T, C, 3 * C, False, False)
    W = torch.randn(3 * C, C, device="cuda").bfloat16()
    dx = torch.empty(cap, C, dtype=torch.bfloat16, device="cuda")
    got = []
    for how in ("alone", "group", "with the input side"):
        w_o, w_qkv = _call(spa, cap, C, C, a[0], a[1], a[4], None, a[6]), _call(spa, cap, C, 3 * C, b[0], b[1], None, None, b[6])
        if how == "alone":
            w_o[2]()
            w_qkv[2]()
        elif how == "group":
            spa.group(w_o[2], w_qkv[2])()
        else:
            spa.group(spa.spa_linear_packed_bwd_input(b[1], None, b[6], W, cap, None, None, dx, prepare=True), w_o[2], w_qkv[2])()
        torch.cuda.synchronize()
        got.append((*w_o[:2], *w_qkv[:2]))
    for other in got[1:]:
        assert all(torch.equal(s, t) for s, t in zip(got[0], other))
    # fp32 sums of T products of ~1 in chunks: 2^-24 a step of 16, over sqrt(T) as the size of the result
    tol = 2.0 ** -24 * (T / 16 + 16) * 4 * max(1.0, T ** 0.5)
    for (dW, db), (x, d, rg, rx, *_) in zip((got[0][:2], got[0][2:]), (a, b)):
        for n0 in range(0, dW.shape[0], 512):              # (64 bits, a part of the columns of d at a time)
            g = d[rg][:, n0:n0 + 512].double()
            assert (dW[n0:n0 + 512].double() - g.T.contiguous() @ x[rx].double()).abs().max() <= tol
            assert (db[n0:n0 + 512].double() - g.sum(0)).abs().max() <= tol
