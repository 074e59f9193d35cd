"""Weight sides of a block: chunks that add up the sums of every 256 rows apart, of less than a step up to several times 256 rows, and chunks of one
sum, alone and beside the input side (the same bits), against 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# Capacity and columns; chunks whose products go into one sum, None: sums of 256 rows in one chunk and several, up to 7.3e9 = cap C^2.  Beyond, and
# where as many chunks as fill the chip are no more than a block's, one sum a chunk.  Live rows: none, a row, on either side of whole sums of 256, all.
@pytest.mark.parametrize("cap,C,chunks", [(2049, 1024, None), (3136, 768, None), (6272, 768, None), (4704, 512, None), (2500, 520, None),
                                          (6800, 1024, None), (9408, 768, None), (11000, 768, None), (9800, 136, 16), (7840, 1024, 4), (12544, 768, 7)])
@pytest.mark.parametrize("part", ["none", "one", "255", "257", "512", "half", "all"])
def test_sums_apart(cap, C, chunks, part):
    from paper_2410_23608_amd import spa
    T = {"none": 0, "one": 1, "half": cap // 2, "all": cap}.get(part) if not part.isdigit() else int(part)
    g = torch.Generator(device="cuda")
    g.manual_seed(cap + T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    d, x, d3, W = rnd(cap, C), rnd(cap, C), rnd(cap, 3 * C), rnd(3 * C, C)
    tot = torch.tensor([T], dtype=torch.int32, device="cuda")
    got = []
    for together in (False, True):
        dx = torch.empty(cap, C, dtype=torch.bfloat16, device="cuda")
        calls, out = [spa.spa_linear_packed_bwd_input(d3, None, tot, W, cap, None, None, dx, prepare=True)], []
        for dout, n in ((d, C), (d3, 3 * C)):
            dW, db = torch.full((n, C), float("nan"), device="cuda"), torch.full((n,), float("nan"), device="cuda")
            ws = torch.empty(max(256, spa.spa_linear_bwd_weight_workspace_bytes(cap, C, n, "bf16")), dtype=torch.uint8, device="cuda")
            calls.append(spa.spa_linear_packed_bwd_weight(dout, None, x, None, None, tot, cap, dW, db, ws, prepare=True))
            out += [dW, db]
        if together:
            spa.group(*calls)()
        else:
            for call in calls:
                call()
        torch.cuda.synchronize()
        got.append(out + [dx[:T]])
    assert all(torch.equal(a, b) for a, b in zip(*got))
    # Each addition rounds by 2^-24 times 0.42 in the mean of squares (evenly spread, over mantissas of a normal sum), to the sum so far; an
    # instruction adds 8 products at a time, a chunk is a multiple of 64 rows.  Measured .9 of that.  Sums of 256 rows in one sum instead of apart are 1.8 times as far off or
    # more, 12544 rows in five chunks instead of seven 1.18 times.
    additions = min(T, 256) / 16 + T / 512 if chunks is None else min(T, -(-T // (64 * chunks)) * 64) / 16 + chunks / 2
    rel = 1.03 * 0.42 * 2.0 ** -24 * additions ** 0.5
    for (dW, db), dout in ((got[0][:2], d), (got[0][2:4], d3)):
        for a, ref, bound in ((dW, dout[:T].double().T.contiguous() @ x[:T].double(), rel),
                              (db, dout[:T].double().sum(0), 2.0 ** -24 * (16 + cap / 256 + 16) ** 0.5)):
            assert float((a.double() - ref).norm()) <= bound * float(ref.norm()) + (0 if T else 1e-30)


# a call of its own keeps the indices of its named rows in LDS: one chunk and several, fewer rows than the steps in LDS hold, no row; the last
# capacity in one chunk where the indices of both operands are too many for that
@pytest.mark.parametrize("gi,xi", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("cap,C,T", [(2100, 1024, 2100), (3136, 768, 1601), (2500, 520, 0), (2500, 520, 65), (9408, 768, 4704), (5096, 1024, 5033)])
def test_named_rows_alone_and_in_a_group(cap, C, T, gi, xi):
    from paper_2410_23608_amd import spa
    g = torch.Generator(device="cuda")
    g.manual_seed(cap + T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, tot, calls, out = rnd(cap, C), torch.tensor([T], dtype=torch.int32, device="cuda"), [], []
    named = lambda: torch.randperm(cap, generator=g, device="cuda").int()
    ig, ix = named() if gi else None, named() if xi else None
    d = {n: rnd(cap, n) for n in (C, 3 * C)}
    for n in 2 * (C, 3 * C):
        out.append((torch.full((n, C), float("nan"), device="cuda"), torch.full((n,), float("nan"), device="cuda")))
        ws = torch.empty(max(256, spa.spa_linear_bwd_weight_workspace_bytes(cap, C, n, "bf16")), dtype=torch.uint8, device="cuda")
        calls.append(spa.spa_linear_packed_bwd_weight(d[n], ig, x, ix, None, tot, cap, *out[-1], ws, prepare=True))
    dx = torch.empty(cap, C, dtype=torch.bfloat16, device="cuda")
    for call in calls[:2]:
        call()
    spa.group(spa.spa_linear_packed_bwd_input(d[3 * C], None, tot, rnd(3 * C, C), cap, None, None, dx, prepare=True), *calls[2:])()
    torch.cuda.synchronize()
    for (a, b), (a2, b2) in zip(out[:2], out[2:]):
        assert torch.isfinite(a).all() and torch.equal(a, a2) and torch.equal(b, b2)
