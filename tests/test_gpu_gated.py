"""Attention whose values are gated on the way (spa_gated_attention_unpack and its backward) against packed q|k and a
packed gated x, bit for bit: every forward and backward kernel form, images without and with every token."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Dh,H,N", [(32, 2, 33), (64, 3, 196), (32, 3, 256), (64, 2, 300), (32, 2, 700)])
def test_gated_equals_packed(Dh, H, N):
    from paper_2410_23608_amd import pipeline
    B, C = 5, H * Dh
    g = torch.Generator(device="cuda")
    g.manual_seed(Dh + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    x, w = rnd(B, N, C), rnd(C)
    w /= w.norm()
    x += (rnd(B, 1, 1) - x @ w[:, None].expand(C, 1) * 0.5) * w
    x[1] -= 50 * w                                     # nothing selected
    x[2] += 50 * w                                     # everything
    x, w, qk, dy = x.bfloat16(), w.bfloat16(), rnd(B, N, 2 * C).bfloat16(), rnd(B, N, C).bfloat16()
    lab = (rnd(B, N) > 0).to(torch.uint8)
    a, b = pipeline.TrainPass(B, N, C, H, "bf16"), pipeline.TrainPass(B, N, C, H, "bf16", pack_pair=False)
    assert a.gated and not b.gated
    for tp in (a, b):
        tp.run(x, w, qk, lab, dy)
    torch.cuda.synchronize()
    T = int(b.total)
    counts = b.mask.sum(1).tolist()
    assert counts[1] == 0 and counts[2] == N
    for name in ("scores", "mask", "cu_seqlens", "inv_pos", "total", "y", "dqk", "d_rg", "dx", "dw", "db", "loss"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    assert torch.equal(a.gather_idx[:T], b.gather_idx[:T]) and torch.equal(a.out[:T], b.out[:T])
    for b0, b1 in zip(b.cu_seqlens[:-1].tolist(), b.cu_seqlens[1:].tolist()):
        assert torch.equal(a.lse[:, b0:b1], b.lse[:, b0:b1])
