"""Short segments whose rows are named by an index or by the mask keep a step's K rows in registers: the same bits as packed
rows, whose K goes through LDS, for segments that end on and next to a step, one and two waves a unit, and with infinities
in the last key, whose row stands in for the keys past the end."""
import pytest
import torch

pytestmark = pytest.mark.gpu
LENS = (1, 2, 31, 32, 33, 63, 64, 65, 95, 97, 127, 128, 160, 193, 224, 225, 255, 256, 0, 17)


@pytest.mark.parametrize("H,Dh", [(6, 64), (2, 64), (3, 32)])
@pytest.mark.parametrize("B", [20, 64, 72])                 # two waves a unit; by weight; more images than it ranks
def test_same_bits_as_packed_rows(B, H, Dh):
    from paper_2410_23608_amd import spa
    N, C = 256, H * Dh
    g = torch.Generator(device="cuda")
    g.manual_seed(B + H)
    lens = torch.tensor([LENS[b % len(LENS)] for b in range(B)])
    cu = torch.cat([torch.zeros(1, dtype=torch.long), lens.cumsum(0)])
    T = int(cu[-1])
    rows = torch.randn(T, 3 * C, generator=g, device="cuda").bfloat16()
    rows[int(cu[5]) - 1, C:2 * C] = float("inf")            # of the segment of 33
    rows[int(cu[9]) - 1, C] = float("-inf")
    at = torch.cat([torch.randperm(N, generator=torch.Generator().manual_seed(b))[:n].sort()[0] + b * N
                    for b, n in enumerate(lens.tolist())]).cuda()
    gather = torch.zeros(B * N, dtype=torch.int32, device="cuda")
    gather[:T] = at.int()
    inv = torch.full((B * N,), -1, dtype=torch.int32, device="cuda")
    inv[at] = torch.arange(T, dtype=torch.int32, device="cuda")
    t = torch.full((B * N, 3 * C), float("nan"), device="cuda").bfloat16()
    t[at] = rows
    cols = lambda z: (z[:, :C], z[:, C:2 * C], z[:, 2 * C:])
    ys = [torch.full((B, N, C), 7.0, device="cuda").bfloat16() for _ in range(3)]
    spa.spa_packed_attention_unpack(*cols(rows), cu.int().cuda(), gather, inv, None, H, Dh, ys[0])
    spa.spa_gathered_attention_unpack(*cols(t), cu.int().cuda(), gather, inv, None, H, Dh, ys[1])
    spa.spa_selected_attention_unpack(*cols(t), (inv >= 0).to(torch.uint8).view(B, N), None, H, Dh, ys[2])
    torch.cuda.synchronize()
    for y in ys[1:]:
        same = ys[0].view(torch.int16) == y.view(torch.int16)
        assert (same | (ys[0].isnan() & y.isnan())).all()
    b = 12                                                   # 160 keys, no infinity
    q, k, v = (z[int(cu[b]):int(cu[b + 1])].float().view(-1, H, Dh).transpose(0, 1).contiguous() for z in cols(rows))
    ref = (torch.softmax(q @ k.transpose(1, 2).contiguous() / Dh ** 0.5, -1) @ v).transpose(0, 1).reshape(-1, C)
    got = ys[1].view(B * N, C)[at[int(cu[b]):int(cu[b + 1])]].float()
    # probabilities and the output rounded to bf16: 2^-9 each of values below max |v| ~ 5
    assert (got - ref).abs().max() <= 2 * 2.0 ** -9 * 5
