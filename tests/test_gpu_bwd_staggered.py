"""The one-kernel attention backward from 832 (image, head) pairs on, where its workgroups take the images in another order than by
weight alone: an image's gradients are the same bits as in calls of fewer images."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,N", [(52, 16, 192), (70, 12, 161), (104, 8, 256), (280, 3, 170), (6, 160, 200)])
def test_an_image_alone_and_among_many(B, H, N):
    from paper_2410_23608_amd import spa
    Dh, C = 64, 64 * H
    g = torch.Generator(device="cuda")
    g.manual_seed(B)
    lens = torch.randint(0, N + 1, (B,), generator=g, device="cuda")
    lens[B // 2] = N
    cu = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
    cu[1:] = lens.cumsum(0).int()
    T = int(cu[-1])
    rnd = lambda: torch.randn(T, C, generator=g, device="cuda").bfloat16()
    q, k, v, dy = rnd(), rnd(), rnd(), rnd()
    out, lse = torch.empty_like(q), torch.zeros(H, B * N, device="cuda")
    spa.spa_packed_attention(q, k, v, cu, B, N, H, Dh, out, lse)
    ws = torch.empty(max(256, spa.spa_attention_bwd_workspace_bytes(B, N, H, Dh, spa.SPA_BF16)), dtype=torch.uint8, device="cuda")
    whole = [torch.full_like(q, float("nan")) for _ in range(3)]
    spa.spa_packed_attention_bwd(q, k, v, out, dy, lse, cu, B, N, H, Dh, *whole, ws)
    parts = [torch.full_like(q, float("nan")) for _ in range(3)]
    step = max(1, min(B // 3, 831 // H))
    for b0 in range(0, B, step):
        b1 = min(B, b0 + step)
        r0, r1 = int(cu[b0]), int(cu[b1])
        if r0 == r1:
            continue
        s = slice(r0, r1)
        l = torch.zeros(H, (b1 - b0) * N, device="cuda")
        l[:, :r1 - r0] = lse[:, s]
        spa.spa_packed_attention_bwd(q[s], k[s], v[s], out[s], dy[s], l, (cu[b0:b1 + 1] - r0).contiguous(), b1 - b0, N, H, Dh,
                                     *(t[s] for t in parts), ws)
    torch.cuda.synchronize()
    for a, b in zip(whole, parts):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
