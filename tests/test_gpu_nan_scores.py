"""A NaN among the scores of the forward's units (tiled, one wave, several waves, launch group): the rows that attend to it are NaN, and every
other row, in the same tile, the next head and the images before and behind, has the same bits as without it."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["packed", "gathered", "selected", "group"])
@pytest.mark.parametrize("B,H,Dh,N", [(4, 2, 64, 480), (4, 3, 32, 300), (70, 6, 64, 60), (40, 8, 32, 100), (5, 2, 64, 193), (5, 1, 32, 97)])
def test_only_the_rows_that_attend_to_it(form, B, H, Dh, N):
    from paper_2410_23608_amd import spa
    if (form == "selected" and N > 256) or (form == "group" and Dh != 32):
        pytest.skip("the mask form takes images of up to 256 tokens, a launch group heads of 32")
    C = H * Dh
    g = torch.Generator().manual_seed(N + B)
    mask = torch.rand(B, N, generator=g) < 0.7
    mask[1, 3] = mask[2, 0] = mask[1, N - 1] = True
    qkv = torch.randn(B * N, 3 * C, generator=g).bfloat16().cuda()
    m = mask.to(torch.uint8).cuda()
    T, td = int(mask.sum()), qkv.dtype
    ints = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
    cu, gather, inv = ints(B + 1), ints(B * N), ints(B * N)
    spa.spa_pack(None, m, None, None, 0, None, cu, gather, inv, None)
    cols = lambda t: (t[:, :C], t[:, C:2 * C], t[:, 2 * C:])

    def forward(t):
        y = torch.full((B, N, C), float("inf"), dtype=td, device="cuda")
        lse = torch.zeros(H, B * N, device="cuda")
        if form == "selected":
            spa.spa_selected_attention_unpack(*cols(t), m, None, H, Dh, y)
        elif form == "packed":
            packed = torch.zeros_like(t)
            packed[:T] = t[gather[:T].long()]
            spa.spa_packed_attention_unpack(*cols(packed), cu, gather, inv, None, H, Dh, y, torch.zeros(B * N, C, dtype=td, device="cuda"), lse)
        else:
            call = lambda out, **kw: spa.spa_gathered_attention_unpack(*cols(t), cu, gather, inv, None, H, Dh, out, None, None, **kw)
            if form == "group" and N <= 256:                            # (in a group short images go by the mask)
                call = lambda out, **kw: spa.spa_selected_attention_unpack(*cols(t), m, None, H, Dh, out, **kw)
            if form == "gathered":
                call(y)
            else:
                other = torch.empty_like(y)
                spa.group(call(y, prepare=True), call(other, prepare=True))()
                torch.cuda.synchronize()
                assert torch.equal(y.view(torch.int16), other.view(torch.int16))
        torch.cuda.synchronize()
        return y

    clean = forward(qkv)
    assert torch.isfinite(clean).all()
    bad = qkv.clone()
    bad[N + 3, Dh - 1] = float("nan")                                   # a query of image 1, head 0
    bad[2 * N, C + (H - 1) * Dh + 5] = float("nan")                     # the first key of image 2, last head
    expect = torch.zeros(B, N, H, dtype=torch.bool)
    expect[1, 3, 0] = True
    expect[2, :, H - 1] = mask[2]
    expect = expect.cuda()[..., None].expand(B, N, H, Dh).reshape(B, N, C)
    got = forward(bad)
    assert torch.equal(torch.isnan(got), expect)
    assert torch.equal(got[~expect], clean[~expect])
