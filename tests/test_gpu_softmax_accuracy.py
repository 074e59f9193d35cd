"""What the reference of the forward's exponentials decides: rows whose weight lies on one key return that key's value
exactly, the error against 64 bits is that of probabilities taken against the row's maximum, whatever the scores' spread,
and scores may rise along a segment by any factor."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

FORMS = ["packed", "gathered", "gated", "selected", "tiled", "whole", "group"]


def _forms(forms, shapes):
    """form, Dh, N: the forms that take such a call."""
    return [(f, Dh, N) for Dh, N in shapes for f in forms
            if not (f in ("selected", "whole") and N > 256) and not (f == "group" and Dh != 32)]


def _forward(form, q, k, v, lens, N, H, Dh, scale=0.0):
    """y rows of the tokens, in packed order, of one of the forms of the bf16 forward; q, k, v: packed rows."""
    from paper_2410_23608_amd import spa
    C, B, T = H * Dh, len(lens), sum(lens)
    cu = torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).int().cuda()
    idx = torch.cat([b * N + torch.randperm(N, generator=torch.Generator().manual_seed(b))[:n].sort().values
                     for b, n in enumerate(lens)]).cuda()
    gather = torch.zeros(B * N, dtype=torch.int32, device="cuda")
    gather[:T] = idx.int()
    inv = torch.full((B * N,), -1, dtype=torch.int32, device="cuda")
    inv[idx] = torch.arange(T, dtype=torch.int32, device="cuda")
    y = torch.full((B, N, C), float("nan"), device="cuda", dtype=torch.bfloat16)
    out, lse = torch.zeros(B * N, C, device="cuda", dtype=torch.bfloat16), torch.zeros(H, B * N, device="cuda")

    def at_tokens(t):
        full = torch.zeros(B * N, C, device="cuda", dtype=torch.bfloat16)
        full[idx] = t
        return full

    if form in ("packed", "tiled", "whole"):
        opt = {"tiled": ("attn_fwd_cfg", "4,64"), "whole": ("attn_fwd_short", "whole")}.get(form)
        if opt:
            spa.spa_set_option(*opt)
        try:
            spa.spa_packed_attention_unpack(q, k, v, cu, gather, inv, None, H, Dh, y, out, lse, softmax_scale=scale)
        finally:
            if opt:
                spa.spa_set_option(opt[0])
    elif form == "gated":       # a score of 100: Sigmoid = 1 in fp32
        scores = torch.full((B * N,), 100.0, device="cuda")
        spa.spa_gated_attention_unpack(at_tokens(q), at_tokens(k), at_tokens(v), scores, cu, gather, inv, None, H, Dh, y, out,
                                       lse, softmax_scale=scale)
    elif form == "selected":
        mask = (inv >= 0).to(torch.uint8).view(B, N)
        spa.spa_selected_attention_unpack(at_tokens(q), at_tokens(k), at_tokens(v), mask, None, H, Dh, y, softmax_scale=scale)
        lse = None
    else:
        if form == "group":
            spa.spa_group_begin()
        if N > 256 or form == "gathered":
            spa.spa_gathered_attention_unpack(at_tokens(q), at_tokens(k), at_tokens(v), cu, gather, inv, None, H, Dh, y, out,
                                              lse, softmax_scale=scale)
        else:
            spa.spa_packed_attention_unpack(q, k, v, cu, gather, inv, None, H, Dh, y, out, lse, softmax_scale=scale)
        if form == "group":
            spa.spa_group_end()
    torch.cuda.synchronize()
    assert (y.view(B * N, C)[inv < 0] == 0).all()
    return y.view(B * N, C)[idx], out[:T], None if lse is None else lse[:, :T], cu


@pytest.mark.parametrize("form,Dh,N", _forms(FORMS, [(32, 33), (64, 196), (32, 256), (64, 300), (32, 700)]))
def test_a_key_with_all_the_weight_gives_its_value(form, Dh, N):
    """Keys are rows of a Hadamard matrix and their negatives, so that each query scores Dh b on its own key and 0 or less
    on the others: at a score of 17 and more in natural units these weigh less than 2^-24 together and the output is the
    V row of that key, bit for bit (equal keys carry equal V rows)."""
    had = torch.ones(1, 1)
    while had.shape[0] < Dh:
        had = torch.cat([torch.cat([had, had], 1), torch.cat([had, -had], 1)])
    codes = torch.cat([had, -had]).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(Dh + N)
    H, lens = 3, [N, 1, 0, N - 1, N // 2 + 1]
    at = torch.cat([torch.randperm(max(n, 1), generator=g, device="cuda")[:n] % (2 * Dh) for n in lens])      # key j: this code
    own = torch.cat([at[s:s + n][torch.randint(max(n, 1), (n,), generator=g, device="cuda")]
                     for s, n in zip([sum(lens[:b]) for b in range(len(lens))], lens) if n])
    for score in (23.1, 24.96, 25.4, 26.6):
        table = 1 + torch.rand(2 * Dh, H, Dh, generator=g, device="cuda")
        table = (table * torch.randn(table.shape, generator=g, device="cuda").sign()).bfloat16()
        k = codes[at][:, None].expand(-1, H, -1).reshape(len(at), H * Dh).bfloat16()
        q = codes[own][:, None].expand(-1, H, -1).reshape(len(at), H * Dh).bfloat16()
        v = table[at].reshape(len(at), H * Dh)
        got = _forward(form, q.contiguous(), k.contiguous(), v.contiguous(), lens, N, H, Dh, scale=score / Dh)
        want = table[own].reshape(len(at), H * Dh)
        assert torch.equal(got[0], want), (score, int((got[0] != want).sum()))


def _rounded(p):
    return p.bfloat16().double()


@pytest.mark.parametrize("form,Dh,N", _forms(["packed", "gated", "selected", "tiled", "group"],
                                             [(32, 64), (64, 64), (64, 196), (32, 400)]))
@pytest.mark.parametrize("sigma", [1.0, 1.5, 2.0, 3.0])
def test_error_against_64_bits(form, sigma, Dh, N):
    """The error of y, and of dq, dk and dv behind it, against 64 bits, is at most 5 % above that of the same arithmetic
    (probabilities against the row's maximum, rounded to bf16) carried out in 64 bits otherwise."""
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(int(16 * sigma) + Dh + N)
    H, B = 4, 8
    C, lens, T = H * Dh, [N] * B, B * N
    rnd = lambda s=1.0: (s * torch.randn(T, C, generator=g, device="cuda")).bfloat16()
    q, k, v, do = rnd(sigma), rnd(sigma), rnd(), rnd()
    y, out, lse, cu = _forward(form, q, k, v, lens, N, H, Dh)
    heads = lambda t: t.double().view(B, N, H, Dh).transpose(1, 2).contiguous()
    scale = 1 / math.sqrt(Dh)
    Q, K, V, G = (heads(t) for t in (q, k, v, do))
    S = Q @ K.transpose(2, 3).contiguous() * scale

    def backward(p, ps, o):          # p, ps: the probabilities of dV and of dS; rounding: what the kernels round
        dp = G @ V.transpose(2, 3).contiguous()
        ds = p * (dp - (G * o).sum(-1, keepdim=True))
        ds = ds if ps is None else _rounded(ds)
        p = p if ps is None else _rounded(p)
        return (ds @ K * scale, ds.transpose(2, 3).contiguous() @ Q * scale, p.transpose(2, 3).contiguous() @ G)

    P = torch.softmax(S, -1)
    exact = (P @ V, *backward(P, None, P @ V))
    E = torch.exp(S - S.amax(-1, keepdim=True))
    o = _rounded(_rounded(E) @ V / E.sum(-1, keepdim=True))
    model = (o, *(_rounded(t) for t in backward(P, True, o)))
    got = [heads(y)]
    if lse is not None:
        assert torch.equal(out, y)
        ws = torch.empty(spa.spa_attention_bwd_workspace_bytes(B, N, H, Dh, spa.SPA_BF16), dtype=torch.uint8, device="cuda")
        d = [torch.full_like(q, float("nan")) for _ in range(3)]
        spa.spa_packed_attention_bwd(q, k, v, out, do, lse.new_zeros(H, B * N).copy_(lse), cu, B, N, H, Dh, *d, ws)
        got += [heads(t) for t in d]
    for name, a, m, e in zip(("y", "dq", "dk", "dv"), got, model, exact):
        err, want = float((a - e).norm() / e.norm()), float((m - e).norm() / e.norm())
        assert err <= 1.05 * want, (name, err, want)


@pytest.mark.parametrize("form,Dh,N", _forms(FORMS, [(32, 250), (64, 196), (64, 700)]))
@pytest.mark.parametrize("rise", [0.02, 0.5, 8.0, -8.0])
def test_scores_that_rise_or_fall_along_the_segment(form, Dh, N, rise):
    """Scores near rise * j at key j, from -100 to +1000 and more in natural units: past 2^40 within a segment, from
    below the range of fp32 exponentials, and the other way round."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    H, lens = 2, [N, N - 5]
    C, T = H * Dh, sum(lens)
    j = torch.cat([torch.arange(n, device="cuda") for n in lens]).float()
    q, k, v = (torch.randn(T, H, Dh, generator=g, device="cuda") for _ in range(3))
    q[..., 0], k[..., 0] = 4.0, (rise * (j - 0.4 * N) * math.sqrt(Dh) / 4)[:, None]
    q, k, v = (t.reshape(T, C).bfloat16() for t in (q, k, v))
    y, _, lse, _ = _forward(form, q, k, v, lens, N, H, Dh)
    s0 = 0
    for n in lens:
        r = slice(s0, s0 + n)
        Q, K, V = (t[r].double().view(n, H, Dh).transpose(0, 1).contiguous() for t in (q, k, v))
        S = Q @ K.transpose(1, 2).contiguous() / math.sqrt(Dh)
        want = (torch.softmax(S, -1) @ V).transpose(0, 1).reshape(n, C)
        # probabilities and results rounded to bf16: 2^-9 each of the largest |v|
        assert torch.isfinite(y[r]).all() and (y[r].double() - want).abs().max() <= 2 ** -7 * float(V.abs().max())
        if lse is not None:
            ref = torch.logsumexp(S, -1)
            assert (lse[:, r] - ref).abs().max() <= 2 ** -20 * (1 + float(S.abs().max()))
        s0 += n


@pytest.mark.parametrize("form,Dh,N", _forms(FORMS, [(32, 100), (64, 196), (64, 300)]))
def test_infinities_and_nan_stay_where_they_belong(form, Dh, N):
    """A NaN in a K row makes its image's outputs NaN and no other image's; NaN and infinities in a V row (the last
    one of the segment among them) pass to that column of its image alone, an infinity as itself."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    H, lens = 2, [N - 3, N - 3, N - 3, N - 3]
    C, n = H * Dh, N - 3
    q, k, v = (torch.randn(4 * n, C, generator=g, device="cuda").bfloat16() for _ in range(3))
    clean = _forward(form, q, k, v, lens, N, H, Dh)[0]
    k[n + 7, 3] = float("nan")
    v[2 * n + n - 1, 5] = float("inf")
    v[3 * n + 2, 1] = -float("inf")
    v[3 * n + n - 1, Dh + 1] = float("nan")
    y = _forward(form, q, k, v, lens, N, H, Dh)[0]
    assert torch.equal(y[:n], clean[:n])
    assert torch.isnan(y[n:2 * n, :Dh]).all() and torch.equal(y[n:2 * n, Dh:], clean[n:2 * n, Dh:])
    for r, cols in ((slice(2 * n, 3 * n), {5: float("inf")}), (slice(3 * n, 4 * n), {1: -float("inf"), Dh + 1: float("nan")})):
        rest = [c for c in range(C) if c not in cols]
        assert torch.equal(y[r][:, rest], clean[r][:, rest])
        for c, val in cols.items():
            assert torch.isnan(y[r, c]).all() if math.isnan(val) else (y[r, c] == val).all(), (c, val)


@pytest.mark.parametrize("steps", [(0,), (1,), (2,), (3,), (0, 1), (0, 1, 2, 3)])
@pytest.mark.parametrize("form,Dh,N", _forms(FORMS, [(32, 256), (64, 196), (64, 300), (32, 700)]))
def test_scores_of_minus_infinity_weigh_nothing(form, Dh, N, steps):
    """Products that overflow to -inf on whole steps of 32 keys, from the first one on or in between: those keys weigh 0
    and the other rows are what they are without them.  Of an image all of whose scores are -inf y is NaN, lse -inf."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + Dh)
    H, lens = 2, [N, N - 3, 161, 40]
    C, T = H * Dh, sum(lens)
    q, k, v = (torch.randn(T, H, Dh, generator=g, device="cuda") for _ in range(3))
    q[..., 0], k[..., 0] = 2.0 ** 120, 0.0
    starts = [sum(lens[:b]) for b in range(len(lens))]
    for s0 in starts[:3]:
        for j in steps:
            k[s0 + 32 * j:s0 + 32 * (j + 1), :, 0] = -2.0 ** 120
    k[starts[3]:, :, 0] = -2.0 ** 120
    q, k, v = (t.reshape(T, C).bfloat16() for t in (q, k, v))
    y, _, lse, _ = _forward(form, q, k, v, lens, N, H, Dh)
    for s0, n in zip(starts[:3], lens[:3]):
        r = slice(s0, s0 + n)
        Q, K, V = (t[r].double().view(n, H, Dh).transpose(0, 1).contiguous() for t in (q, k, v))
        S = Q @ K.transpose(1, 2).contiguous() / math.sqrt(Dh)
        want = (torch.softmax(S, -1) @ V).transpose(0, 1).reshape(n, C)
        # probabilities and results rounded to bf16: 2^-9 each of the largest |v|
        assert torch.isfinite(y[r]).all() and (y[r].double() - want).abs().max() <= 2 ** -7 * float(V.abs().max())
        if lse is not None:
            assert (lse[:, r] - torch.logsumexp(S, -1)).abs().max() <= 1e-4      # sums of up to 700 terms in fp32
    assert torch.isnan(y[starts[3]:]).all()
    if lse is not None:
        assert (lse[:, starts[3]:] == -float("inf")).all()


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("Dh,N", [(32, 300), (64, 290)])
def test_an_infinite_gradient_reaches_dv_as_itself(Dh, N, gated):
    """dO = inf in the last row of a segment: that column of dV is inf, the others are what they are without it."""
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    H, n = 2, N - 3
    C = H * Dh
    q, k, v, do = (torch.randn(n, C, generator=g, device="cuda").bfloat16() for _ in range(4))
    do[n - 1, 5] = float("inf")
    cu = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    ident = torch.arange(N, dtype=torch.int32, device="cuda")
    inv = torch.where(ident < n, ident, -1)
    ws = torch.empty(spa.spa_attention_bwd_workspace_bytes(1, N, H, Dh, spa.SPA_BF16), dtype=torch.uint8, device="cuda")
    got = []
    for clean in (True, False):
        pad = lambda t: torch.cat([t, torch.zeros(N - n, C, device="cuda", dtype=torch.bfloat16)])
        d = pad(do if not clean else torch.where(torch.isinf(do), torch.zeros_like(do), do))
        a = [pad(t) for t in (q, k, v)]
        out, lse = torch.zeros(N, C, device="cuda", dtype=torch.bfloat16), torch.zeros(H, N, device="cuda")
        spa.spa_packed_attention(*a, cu, 1, N, H, Dh, out, lse)
        r = [torch.full((N, C), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(3)]
        if gated:
            spa.spa_gated_attention_bwd_tokens(*a, torch.full((N,), 100.0, device="cuda"), out, d, lse, cu, 1, N, H, Dh, ident, inv,
                                               *r, ws)
        else:
            spa.spa_packed_attention_bwd(*a, out, d, lse, cu, 1, N, H, Dh, *r, ws)
        torch.cuda.synchronize()
        got.append(r[2][:n])
    rest = [c for c in range(C) if c != 5]
    assert (got[1][:, 5] == float("inf")).all() and torch.equal(got[0][:, rest], got[1][:, rest])
