"""The bf16 attention backward kernels at the edges of their tiles (32 tokens per wave, 64-token tiles and
128-row blocks of the long-segment form) and with scores far below zero, where a key past the segment would
have an unbounded probability; packed and token-position rows, against fp32 autograd."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LENS = [1, 0, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193]


@pytest.mark.parametrize("shift", [0.0, 8.0])
@pytest.mark.parametrize("Dh,N", [(32, 224), (64, 224), (32, 260), (64, 330)])
def test_backward_at_tile_edges(Dh, N, shift):
    from paper_2410_23608_amd import spa
    H, C, lens = 2, 2 * Dh, LENS + [N]
    B = len(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(Dh + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    cu = torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).int().cuda()
    T, cap = sum(lens), B * N
    idx = torch.cat([b * N + torch.randperm(N)[:n].sort().values for b, n in enumerate(lens)]).cuda()
    gather = torch.zeros(cap, dtype=torch.int32, device="cuda")
    gather[:T] = idx.int()
    inv = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    inv[idx] = torch.arange(T, dtype=torch.int32, device="cuda")
    qkv = rnd(cap, 3 * C)
    qkv[:, :C] += shift
    qkv[:, C:2 * C] -= shift                       # scores around -shift^2 sqrt(Dh)
    qkv = qkv.bfloat16()
    q, k, v = qkv[:, :C], qkv[:, C:2 * C], qkv[:, 2 * C:]
    dy = rnd(cap, C).bfloat16()
    out = torch.zeros(cap, C, device="cuda", dtype=torch.bfloat16)
    lse = torch.zeros(H, cap, device="cuda")
    spa.spa_packed_attention(q, k, v, cu, B, N, H, Dh, out, lse)
    ws = torch.empty(spa.spa_attention_bwd_workspace_bytes(B, N, H, Dh, spa.dtype_code(out)), dtype=torch.uint8, device="cuda")
    got = []
    for tokens in (False, True):
        d = torch.full((cap, 3 * C), float("nan"), device="cuda", dtype=torch.bfloat16)
        dq, dk, dv = d[:, :C], d[:, C:2 * C], d[:, 2 * C:]
        if tokens:
            spa.spa_packed_attention_bwd_tokens(q, k, v, out, dy, lse, cu, B, N, H, Dh, gather, inv, dq, dk, dv, ws)
            assert (d[inv < 0] == 0).all()
            d = d[idx]
        else:
            dout = torch.zeros_like(dy)
            dout[:T] = dy[idx]
            spa.spa_packed_attention_bwd(q, k, v, out, dout, lse, cu, B, N, H, Dh, dq, dk, dv, ws)
            assert torch.isnan(d[T:]).all()
            d = d[:T]
        got.append(d.float())
    assert torch.equal(got[0], got[1])
    for b, n in enumerate(lens):
        r = slice(int(cu[b]), int(cu[b]) + n)
        p = qkv[r].float().reshape(n, 3, H, Dh).permute(1, 2, 0, 3).contiguous().requires_grad_()
        s = (p[0] @ p[1].transpose(1, 2).contiguous()) / Dh ** 0.5
        o = torch.softmax(s, -1) @ p[2]
        o.backward(dy[idx[r]].float().reshape(n, H, Dh).transpose(0, 1).contiguous())
        ref = p.grad.permute(2, 0, 1, 3).reshape(n, 3 * C)
        if n:
            err = (got[0][r] - ref).abs().max() / max(1.0, ref.abs().max())
            assert err < 3e-2, (b, n, err)


@pytest.mark.parametrize("Dh,N", [(32, 40), (64, 196), (32, 256), (64, 260), (32, 400)])
@pytest.mark.parametrize("shift", [0.0, 8.0])
def test_running_max_form_equals_the_default_form(Dh, N, shift):
    from paper_2410_23608_amd import spa
    H, C, lens = 2, 2 * Dh, [n for n in LENS if n < N] + [N]
    B, cap = len(lens), len(lens) * N
    g = torch.Generator(device="cuda")
    g.manual_seed(Dh + N)
    cu = torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).int().cuda()
    T = sum(lens)
    qkv = torch.randn(cap, 3 * C, generator=g, device="cuda")
    qkv[:, :C] += shift
    qkv[:, C:2 * C] -= shift
    qkv = qkv.bfloat16()
    got = []
    for fn in (spa.spa_packed_attention, spa.spa_packed_attention_running_max):
        out = torch.full((cap, C), float("nan"), device="cuda", dtype=torch.bfloat16)
        lse = torch.full((H, cap), float("nan"), device="cuda")
        fn(qkv[:, :C], qkv[:, C:2 * C], qkv[:, 2 * C:], cu, B, N, H, Dh, out, lse)
        assert torch.isnan(out[T:]).all()
        got.append((out[:T].float(), lse[:, :T]))
    (o0, l0), (o1, l1) = got
    assert torch.isfinite(o1).all() and (o0 - o1).abs().max() <= 2e-2
    assert (l0 - l1).abs().max() <= 1e-4 * max(1.0, float(l0.abs().max()))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("ntok,C", [(1, 64), (17, 128), (2047, 64), (2048, 256), (2049, 128), (8191, 96), (8192, 136), (8193, 128),
                                    (8193, 256)])
def test_gate_backward_at_its_shares(dtype, ntok, C):
    """The forms of the gate backward: 128 and 512 partial rows, shares of 16 tokens and longer ones, a last short share."""
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(ntok + C)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    x, w, d = rnd(1, ntok, C).to(dtype), (rnd(C) / C ** 0.5).to(dtype), rnd(1, ntok, C).to(dtype)
    scores, lab = rnd(1, ntok), (rnd(1, ntok) > 0).to(torch.uint8)
    ws = torch.empty(spa.spa_gate_bwd_workspace_bytes(1, ntok, C, spa.dtype_code(x)), dtype=torch.uint8, device="cuda")
    f = lambda n: torch.full((n,), float("nan"), device="cuda")
    loss, dw, db, dx = f(1), f(C), f(1), torch.full_like(x, float("nan"))
    spa.spa_gate_bwd(x, w, 0.0, scores, None, lab, d, True, 0.25, loss, dx, dw, db, ws)
    torch.cuda.synchronize()
    xf, df, s, y = x[0].double(), d[0].double(), scores[0].double(), lab[0].double()
    p = torch.sigmoid(s)
    ds = 0.25 * (p - y) + p * (1 - p) * (df * xf).sum(1)
    rel = lambda a, b: float((a.double() - b).norm() / b.norm())
    assert rel(dx[0], ds[:, None] * w.double() + p[:, None] * df) <= (1e-5 if dtype == torch.float32 else 1e-2)
    assert rel(dw, (ds[:, None] * xf).sum(0)) <= 1e-4
    assert abs(float(db) - float(ds.sum())) <= 1e-4 * float(ds.abs().sum())
    ref = 0.25 * float((torch.nn.functional.softplus(s) - y * s).sum())
    assert abs(float(loss) - ref) <= 1e-4 * ref


@pytest.mark.parametrize("B,H,Dh,N", [(4, 4, 64, 97), (2, 8, 64, 256), (9, 32, 64, 130), (17, 17, 64, 130), (2, 16, 32, 161),
                                      (8, 32, 32, 200)])
def test_spread_backward_of_few_pairs(B, H, Dh, N):
    """Short segments with few (image, head) pairs, on both sides of the line: the same gradients but for rounding, packed
    and gated operands, an image without a token and a full one; without the workspace the one-kernel form."""
    from paper_2410_23608_amd import spa
    C, cap = H * Dh, B * N
    g = torch.Generator(device="cuda")
    g.manual_seed(cap)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    lens = [0, N] + [(37 * b) % (N + 1) for b in range(2, B)]
    cu = torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).int().cuda()
    T = sum(lens)
    idx = torch.cat([b * N + torch.randperm(N)[:n].sort().values for b, n in enumerate(lens)]).cuda()
    gather = torch.zeros(cap, dtype=torch.int32, device="cuda")
    gather[:T] = idx.int()
    inv = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    inv[idx] = torch.arange(T, dtype=torch.int32, device="cuda")
    q, k, x, dy, scores = rnd(cap, C).bfloat16(), rnd(cap, C).bfloat16(), rnd(cap, C).bfloat16(), rnd(cap, C).bfloat16(), rnd(cap)
    out, lse = torch.zeros(cap, C, device="cuda", dtype=torch.bfloat16), torch.zeros(H, cap, device="cuda")
    y = torch.empty(B, N, C, device="cuda", dtype=torch.bfloat16)
    spa.spa_gated_attention_unpack(q, k, x, scores, cu, gather, inv, None, H, Dh, y, out, lse)
    ws = torch.empty(spa.spa_attention_bwd_workspace_bytes(B, N, H, Dh, spa.dtype_code(out)), dtype=torch.uint8, device="cuda")
    rel = lambda a, b: float((a.float() - b.float()).norm() / b.float().norm())
    new = lambda: [torch.full((cap, C), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(3)]
    runs = []
    for spread, w in ((False, ws), (True, ws), (True, None)):
        d = new()
        spa.spa_gated_attention_bwd_tokens(q, k, x, scores, out, dy, lse, cu, B, N, H, Dh, gather, inv, *d, w, spread=spread)
        runs.append(d)
    assert all(torch.equal(a, b) for a, b in zip(runs[0], runs[2]))
    assert all((b[inv < 0] == 0).all() and rel(b, a) <= 5e-3 for a, b in zip(runs[0], runs[1]))
    pq, pk, pv, pdo = (torch.zeros(cap, C, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    pq[:T], pk[:T], pdo[:T] = q[idx], k[idx], dy[idx]
    pv[:T] = (torch.sigmoid(scores[idx])[:, None] * x[idx].float()).bfloat16()
    a, b = new(), new()
    spa.spa_packed_attention_bwd(pq, pk, pv, out, pdo, lse, cu, B, N, H, Dh, *a, ws)
    spa.spa_packed_attention_bwd(pq, pk, pv, out, pdo, lse, cu, B, N, H, Dh, *b, ws, spread=True)
    assert all(torch.isnan(v[T:]).all() and rel(v[:T], u[:T]) <= 5e-3 for u, v in zip(a, b))


@pytest.mark.parametrize("B,H,Dh,N", [(65, 2, 32, 260), (40, 16, 32, 300), (130, 1, 64, 513), (256, 3, 64, 257), (257, 2, 32, 290),
                                      (66, 2, 64, 196), (129, 1, 32, 130), (513, 1, 64, 40)])
def test_many_segments_equal_few(B, H, Dh, N):
    """Batches past the order of up to 64 segments and 512 pairs, bit for bit the same as image by image in small ones:
    more than 64, 128, 256 and 512 segments, more than 512 pairs, short and long ones, images without a token."""
    from paper_2410_23608_amd import spa
    C = H * Dh
    g = torch.Generator(device="cuda")
    g.manual_seed(B + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    lens = [min(N, (0, N, 1, 129, 64, 200)[b % 6]) if b % 5 else (53 * b) % (N + 1) for b in range(B)]
    starts = [0]
    for n in lens:
        starts.append(starts[-1] + n)
    T = starts[-1]
    q, k, v, dout = rnd(T, C), rnd(T, C), rnd(T, C), rnd(T, C)

    def run(b0, b1):
        r, nb = slice(starts[b0], starts[b1]), b1 - b0
        cu = torch.tensor([s - starts[b0] for s in starts[b0:b1 + 1]], dtype=torch.int32, device="cuda")
        t = [x[r].contiguous() for x in (q, k, v, dout)]
        out, lse = torch.zeros_like(t[0]), torch.zeros(H, nb * N, device="cuda")
        ws = torch.empty(spa.spa_attention_bwd_workspace_bytes(nb, N, H, Dh, spa.SPA_BF16), dtype=torch.uint8, device="cuda")
        d = [torch.full_like(out, float("nan")) for _ in range(3)]
        spa.spa_packed_attention(*t[:3], cu, nb, N, H, Dh, out, lse)
        spa.spa_packed_attention_bwd(*t[:3], out, t[3], lse, cu, nb, N, H, Dh, *d, ws)
        torch.cuda.synchronize()
        return [out, *d]

    whole, step = run(0, B), 20
    parts = [run(b, min(B, b + step)) for b in range(0, B, step)]
    assert all(torch.equal(a, torch.cat(p)) for a, p in zip(whole, zip(*parts)))


@pytest.mark.parametrize("dtype,C", [(t, k * c) for t, k in ((torch.bfloat16, 8), (torch.float32, 4))
                                     for c in (8, 16, 17, 25, 32, 33, 48, 64, 65, 96, 128, 129, 256, 257, 512)])
def test_gate_backward_decides_ties_as_the_forward(dtype, C):
    """Up-scale scores at the gate's own value (a tie: the gate's), one step of fp32 above (theirs) and one below it, for
    every way the backward spreads a row over lanes: (w, x) get a gradient exactly where the gate won."""
    from paper_2410_23608_amd import spa
    ntok = 600
    g = torch.Generator(device="cuda")
    g.manual_seed(C)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    x, w, lab = rnd(1, ntok, C).to(dtype), (rnd(C) / C ** 0.5).to(dtype), (rnd(1, ntok) > 0).to(torch.uint8)
    own, scores = torch.empty(1, ntok, device="cuda"), torch.empty(1, ntok, device="cuda")
    mask = torch.empty(1, ntok, dtype=torch.uint8, device="cuda")
    spa.spa_gate_select(x, w, 0.3, None, 0.5, own, mask)
    step = torch.arange(ntok, device="cuda")[None] % 3 - 1
    inf = torch.full_like(own, float("inf"))
    up = torch.where(step > 0, torch.nextafter(own, inf), torch.where(step < 0, torch.nextafter(own, -inf), own))
    spa.spa_gate_select(x, w, 0.3, up, 0.5, scores, mask)
    assert torch.equal(scores, torch.maximum(own, up))
    ws = torch.empty(spa.spa_gate_bwd_workspace_bytes(1, ntok, C, spa.dtype_code(x)), dtype=torch.uint8, device="cuda")
    f = lambda n: torch.full((n,), float("nan"), device="cuda")
    loss, dw, db, dx = f(1), f(C), f(1), torch.full_like(x, float("nan"))
    spa.spa_gate_bwd(x, w, 0.3, scores, up, lab, None, False, 1.0, loss, dx, dw, db, ws)
    torch.cuda.synchronize()
    assert torch.equal((dx != 0).any(-1), step <= 0)
