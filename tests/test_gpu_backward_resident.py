"""Attention backward with as many workgroups as are resident (segments of up to 512 tokens, up to 512 pairs): batches
whose workgroups take several blocks each, and batches that leave workgroups without one, against every image on its own,
bit for bit; the gradients of unselected tokens are zero."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("B,H,Dh,N", [(64, 8, 32, 500), (64, 5, 64, 400), (33, 4, 64, 257), (3, 2, 32, 512), (64, 8, 32, 270)])
def test_batch_equals_single_images(gated, B, H, Dh, N):
    from paper_2410_23608_amd import spa
    C, g = H * Dh, torch.Generator(device="cuda").manual_seed(B + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    mask = (torch.rand(B, N, generator=g, device="cuda") < torch.rand(B, 1, generator=g, device="cuda")).to(torch.uint8)
    mask[0], mask[1], mask[2, 1:] = 0, 1, 0
    qk, x, dy = rnd(B * N, 2 * C), rnd(B * N, C), rnd(B, N, C)
    scores = torch.randn(B * N, generator=g, device="cuda")

    def run(b0, b1):
        nb, r = b1 - b0, slice(b0 * N, b1 * N)
        ints = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
        cu, gather, inv = ints(nb + 1), ints(nb * N), ints(nb * N)
        spa.spa_pack(None, mask[b0:b1].contiguous(), None, None, 0, None, cu, gather, inv, None)
        t, v, sc, up = qk[r].contiguous(), x[r].contiguous(), scores[r].contiguous(), dy[b0:b1].contiguous()
        y, out = torch.empty(nb, N, C, dtype=torch.bfloat16, device="cuda"), torch.zeros_like(v)
        lse = torch.zeros(H, nb * N, device="cuda")
        ws = torch.empty(spa.spa_attention_bwd_workspace_bytes(nb, N, H, Dh, spa.SPA_BF16), dtype=torch.uint8, device="cuda")
        d = [torch.full_like(v, float("nan")) for _ in range(3)]
        if gated:
            spa.spa_gated_attention_unpack(t[:, :C], t[:, C:], v, sc, cu, gather, inv, None, H, Dh, y, out, lse)
            spa.spa_gated_attention_bwd_tokens(t[:, :C], t[:, C:], v, sc, out, up, lse, cu, nb, N, H, Dh, gather, inv, *d, ws)
        else:
            idx = gather[:int(cu[-1])].long()
            p, pv = torch.zeros_like(t), torch.zeros_like(v)
            p[:len(idx)], pv[:len(idx)] = t[idx], v[idx]
            spa.spa_packed_attention_unpack(p[:, :C], p[:, C:], pv, cu, gather, inv, None, H, Dh, y, out, lse)
            spa.spa_packed_attention_bwd_tokens(p[:, :C], p[:, C:], pv, out, up, lse, cu, nb, N, H, Dh, gather, inv, *d, ws)
        torch.cuda.synchronize()
        return d

    whole = run(0, B)
    parts = [run(b, b + 1) for b in range(B)]
    for i, a in enumerate(whole):
        assert torch.equal(a, torch.cat([p[i] for p in parts]))
        assert (a[mask.view(-1) == 0] == 0).all()
