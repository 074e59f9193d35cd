"""Long segments: up to 768 blocks of capacity the tiles' fragments are read early at 32 columns a head, above where they are
used; at 64 some of them are.  The same bits on both sides of the line, for segments that end on and next to tile and
block edges, against fp32; scores that overflow, in a first tile and in a last one."""
import pytest
import torch

pytestmark = pytest.mark.gpu
LENS = (1, 31, 64, 65, 127, 128, 129, 192, 257, 700)


@pytest.mark.parametrize("H,Dh,capacities", [(2, 32, (768, 769)), (8, 32, (1280, 1281)), (2, 64, (768, 769))])      # first: 768 and 896 blocks
@pytest.mark.parametrize("form", ["packed", "gathered", "gated"])
def test_both_sides_of_the_line(form, H, Dh, capacities):
    from paper_2410_23608_amd import spa
    B = 64
    C = H * Dh
    g = torch.Generator(device="cuda")
    g.manual_seed(len(form))
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    lens = torch.tensor([LENS[i] if i < len(LENS) else 0 for i in range(B)])
    cu = torch.cat([torch.zeros(1, dtype=torch.long), lens.cumsum(0)])
    T = int(cu[-1])
    got = []
    for N in capacities:
        g.manual_seed(7)
        rows = rnd(T, 3 * C)
        rows[int(cu[3]) + 1, C:2 * C] = float("-inf")      # a key whose scores are -inf, inf or NaN: the same on both sides
        rows[int(cu[9]) + 699, 2 * C:] = float("inf")      # the last row's value, beside rows past the segment
        sc = torch.randn(T, generator=g, device="cuda")
        at = torch.cat([torch.randperm(N, generator=torch.Generator().manual_seed(b))[:n].sort()[0] + b * N
                        for b, n in enumerate(lens.tolist())]).cuda()
        gather = torch.zeros(B * N, dtype=torch.int32, device="cuda")
        gather[:T] = at.int()
        inv = torch.full((B * N,), -1, dtype=torch.int32, device="cuda")
        inv[at] = torch.arange(T, dtype=torch.int32, device="cuda")
        out, lse = torch.zeros(B * N, C, device="cuda").bfloat16(), torch.zeros(H, B * N, device="cuda")
        y = torch.full((B, N, C), float("nan"), device="cuda").bfloat16()
        cud = cu.int().cuda()
        if form == "packed":
            spa.spa_packed_attention_unpack(rows[:, :C], rows[:, C:2 * C], rows[:, 2 * C:], cud, gather, inv, None, H, Dh, y, out, lse)
        else:
            t = torch.zeros(B * N, 3 * C, device="cuda").bfloat16()
            t[at] = rows
            s = torch.zeros(B * N, device="cuda")
            s[at] = sc
            q, k, v = t[:, :C], t[:, C:2 * C], t[:, 2 * C:]
            if form == "gathered":
                spa.spa_gathered_attention_unpack(q, k, v, cud, gather, inv, None, H, Dh, y, out, lse)
            else:
                spa.spa_gated_attention_unpack(q, k, v, s, cud, gather, inv, None, H, Dh, y, out, lse)
        torch.cuda.synchronize()
        flat = y.view(B * N, C)
        assert torch.equal(flat[at].view(torch.int16), out[:T].view(torch.int16)) and not flat[inv < 0].any()
        got.append((out[:T].clone(), lse[:, :T].clone()))
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    v = rows[:, 2 * C:].float()
    if form == "gated":
        v = (v * torch.sigmoid(sc)[:, None]).bfloat16().float()
    for b, n in enumerate(lens.tolist()):
        if n == 0 or b in (3, 9):
            continue
        r = slice(int(cu[b]), int(cu[b + 1]))
        q, k, x = (z[r].float().view(n, H, Dh).transpose(0, 1) for z in (rows[:, :C], rows[:, C:2 * C], v))
        p = torch.softmax(q @ k.transpose(1, 2).contiguous() / Dh ** 0.5, -1)
        ref = (p @ x.contiguous()).transpose(0, 1).reshape(n, C)
        # probabilities and the output rounded to bf16: 2^-9 each of values below max |v| ~ 4.5
        assert (got[0][0][r].float() - ref).abs().max() <= 2 * 2.0 ** -9 * 5
    assert torch.isinf(got[0][0][int(cu[9]):int(cu[10])].float()).all() if form != "gated" else True
