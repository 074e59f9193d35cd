"""Weight sides of a block whose chunks add up the sums of every 256 rows apart: chunks of less than a step up to several times 256 rows, alone
and beside the input side (the same bits), against 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# capacity and columns: one chunk and several; live rows: none, a row, on either side of whole sums of 256, all
@pytest.mark.parametrize("cap,C", [(2049, 1024), (3136, 768), (6272, 768), (4704, 512), (2500, 520), (9800, 136)])
@pytest.mark.parametrize("part", ["none", "one", "255", "257", "512", "half", "all"])
def test_sums_apart(cap, C, part):
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
    for (dW, db), dout in ((got[0][:2], d), (got[0][2:4], d3)):
        # roundings of 2^-24: at most 16 products of 16 rows, then cap / 256 sums and 16 chunks, random in sign
        rel = 2.0 ** -24 * (16 + cap / 256 + 16) ** 0.5
        for a, ref in ((dW, dout[:T].double().T.contiguous() @ x[:T].double()), (db, dout[:T].double().sum(0))):
            assert float((a.double() - ref).norm()) <= rel * float(ref.norm()) + (0 if T else 1e-30)
