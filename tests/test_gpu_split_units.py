"""Short-segment forward with the keys of a unit shared by several waves (small launches): lengths at the edges of the
waves' steps of 32 keys, down to units whose second wave has no keys, images without and with all tokens selected."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LENS = [0, 1, 31, 32, 33, 63, 64, 65, 95, 97, 128, 129, 160, 193]


def _reference(q, k, v, lens, H, Dh):
    """softmax(q k^T / sqrt(Dh)) v and its log-sum-exp of every segment, in float64."""
    out, lse, at = torch.zeros_like(q), torch.zeros(H, q.shape[0], dtype=torch.float64), 0
    for n in lens:
        if n == 0:
            continue
        h = lambda t: t[at:at + n].view(n, H, Dh).transpose(0, 1)
        s = (h(q) @ h(k).transpose(1, 2).contiguous()) / Dh ** 0.5
        out[at:at + n] = (torch.softmax(s, 2) @ h(v).contiguous()).transpose(0, 1).reshape(n, H * Dh)
        lse[:, at:at + n] = torch.logsumexp(s, 2)
        at += n
    return out, lse


@pytest.mark.parametrize("form", ["packed", "gathered", "selected"])
@pytest.mark.parametrize("dtype,H,Dh,N", [("bf16", 2, 64, 193), ("bf16", 3, 32, 256), ("bf16", 1, 32, 97), ("f32", 2, 32, 196),
                                          ("f32", 1, 64, 193), ("f32", 2, 32, 300)])
def test_units_of_several_waves(form, dtype, H, Dh, N):
    from paper_2410_23608_amd import spa
    if form == "selected" and N > 256:
        pytest.skip("the mask form takes images of up to 256 tokens")
    lens = [n for n in LENS if n <= N] + [N]
    B, C, T, td = len(lens), H * Dh, sum(lens), torch.bfloat16 if dtype == "bf16" else torch.float32
    assert N > 96 and B * H * ((N + 31) // 32) <= 768               # what makes several waves share a unit
    g = torch.Generator().manual_seed(N + Dh)
    rows = torch.cat([b * N + torch.randperm(N, generator=g)[:n].sort().values for b, n in enumerate(lens)])
    mask = torch.zeros(B * N, dtype=torch.uint8)
    mask[rows] = 1
    mask = mask.cuda().view(B, N)
    qkv = (1.5 * torch.randn(B * N, 3 * C, generator=g)).to(td)
    ref, ref_lse = _reference(*(qkv[rows].double()[:, i * C:(i + 1) * C] for i in range(3)), lens, H, Dh)
    t = qkv.cuda()
    ints = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
    cu, gather, inv = ints(B + 1), ints(B * N), ints(B * N)
    spa.spa_pack(None, mask, None, None, 0, None, cu, gather, inv, None)
    y = torch.full((B, N, C), float("nan"), dtype=td, device="cuda")
    out, lse = torch.zeros(B * N, C, dtype=td, device="cuda"), torch.zeros(H, B * N, device="cuda")
    cols = lambda m: (m[:, :C], m[:, C:2 * C], m[:, 2 * C:])
    if form == "selected":
        spa.spa_selected_attention_unpack(*cols(t), mask, None, H, Dh, y)
    elif form == "gathered":
        spa.spa_gathered_attention_unpack(*cols(t), cu, gather, inv, None, H, Dh, y, out, lse)
    else:
        packed = torch.zeros_like(t)
        packed[:T] = t[gather[:T].long()]
        spa.spa_packed_attention_unpack(*cols(packed), cu, gather, inv, None, H, Dh, y, out, lse)
    torch.cuda.synchronize()
    got = y.view(B * N, C).cpu().double()
    assert (got[mask.view(-1).cpu() == 0] == 0).all()
    # bf16: probabilities and the result rounded once each (2^-9 of values up to 4 sigma = 6); fp32: sums of up to 300
    # products of rounding 2^-24 on each, values up to 6
    assert (got[rows] - ref).abs().max() <= (3e-2 if dtype == "bf16" else 1e-5)
    if form != "selected":
        assert (out[:T].cpu().double() - got[rows]).abs().max() == 0
        assert (lse[:, :T].cpu().double() - ref_lse).abs().max() <= 1e-5


@pytest.mark.parametrize("steps", [(0,), (1,), (2,), (3,), (0, 1, 2, 3)])
@pytest.mark.parametrize("H,Dh,N", [(2, 32, 196), (1, 64, 193), (300, 32, 196), (1, 32, 64)])
def test_fp32_scores_of_minus_infinity_weigh_nothing(H, Dh, N, steps):
    """Products that overflow to -inf on whole steps of 32 keys (the first four steps are the first of a wave each where
    four share a unit; 300 heads and 64 tokens: one wave a unit): those keys weigh 0."""
    from paper_2410_23608_amd import spa
    g = torch.Generator().manual_seed(N + Dh)
    C = H * Dh
    q, k, v = (torch.randn(N, H, Dh, generator=g) for _ in range(3))
    q[..., 0], k[..., 0] = 2.0 ** 120, 0.0
    steps = [j for j in steps if 32 * (j + 1) < N]
    for j in steps:
        k[32 * j:32 * (j + 1), :, 0] = -2.0 ** 120
    q, k, v = (t.reshape(N, C) for t in (q, k, v))
    ref, ref_lse = _reference(q.double(), k.double(), v.double(), [N], H, Dh)
    cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    out, lse = torch.full((N, C), float("nan"), device="cuda"), torch.zeros(H, N, device="cuda")
    spa.spa_packed_attention(q.cuda(), k.cuda(), v.cuda(), cu, 1, N, H, Dh, out, lse)
    torch.cuda.synchronize()
    # sums of up to 196 products of rounding 2^-24 on each, values up to 6
    assert (out.cpu().double() - ref).abs().max() <= 1e-5 and (lse.cpu().double() - ref_lse).abs().max() <= 1e-5


@pytest.mark.parametrize("dtype,H,Dh,N,same,other", [("bf16", 6, 64, 196, (1, 8, 36), (37, 64)), ("bf16", 4, 32, 97, (1, 64), (65, 80)),
                                                     ("f32", 2, 32, 196, (1, 52), (53, 64)), ("bf16", 6, 64, 96, (1, 36, 64), ()),
                                                     ("bf16", 8, 32, 300, (1, 30), ())])
def test_what_the_bits_of_an_image_depend_on(dtype, H, Dh, N, same, other):
    """The first image alone and with others behind it: the same bits in all batches on one side of the line of units
    (8 ceil(H B / 8) ceil(N / 32) at most 1536, 1024 or 768), the same bits on the other side, rounding between them."""
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(N + Dh)
    C, td, most = H * Dh, torch.bfloat16 if dtype == "bf16" else torch.float32, max(same + other)
    q, k, v = (torch.randn(most * N, C, generator=g, device="cuda").to(td) for _ in range(3))
    lens = [N - 3] + [(7 * b) % (N + 1) for b in range(1, most)]
    line = {("bf16", 64): 1536, ("bf16", 32): 1024, ("f32", 32): 768}[dtype, Dh]
    units = lambda B: (H * B + 7) // 8 * 8 * ((N + 31) // 32)
    assert not 96 < N <= 256 or units(max(same)) <= line < units(min(other))
    got = []
    for B in same + other:
        cu = torch.tensor([0] + lens[:B], dtype=torch.int32).cumsum(0).int().cuda()
        out, lse = torch.zeros(B * N, C, dtype=td, device="cuda"), torch.zeros(H, B * N, device="cuda")
        spa.spa_packed_attention(q[:B * N], k[:B * N], v[:B * N], cu, B, N, H, Dh, out, lse)
        got.append((out[:N - 3], lse[:, :N - 3].contiguous()))
    torch.cuda.synchronize()
    for group in (got[:len(same)], got[len(same):]):
        for out, lse in group[1:]:
            assert torch.equal(out, group[0][0]) and torch.equal(lse, group[0][1])
    for out, lse in got[len(same):]:
        # bf16: probabilities of a wave rounded against its own maximum, 2^-9 of |v| up to 4.5 on either side; fp32: sums of
        # up to 196 terms in another order
        assert (out.double() - got[0][0].double()).abs().max() <= (2e-2 if dtype == "bf16" else 2e-6)
        assert (lse - got[0][1]).abs().max() <= 2e-6
