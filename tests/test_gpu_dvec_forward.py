"""A training run knows dy before its forward pass and takes D of the backward from the forward's launch; single stages form
it in a launch of their own: the same bits, also where dy is the buffer that the forward pass writes."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(B, N, C, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    return rnd(B, N, C), rnd(C), rnd(B, N, 2 * C), (torch.rand(B, N, generator=g, device="cuda") < 0.4).to(torch.uint8), rnd(B, N, C)


def _outputs(p):
    return [t.clone() for t in (p.y, p.out, p.lse, p.loss, p.dx, p.dqk, p.d_rg, p.dw, p.db)]


def _same(a, b):
    assert all(torch.equal(s.view(torch.uint8), t.view(torch.uint8)) for s, t in zip(a, b))


@pytest.mark.parametrize("B,N,H,Dh", [(2, 257, 2, 32), (3, 385, 3, 64), (1, 1100, 2, 32), (70, 300, 1, 32), (5, 300, 104, 32)])
@pytest.mark.parametrize("alias", [False, True])
def test_run_and_stages(B, N, H, Dh, alias):
    from paper_2410_23608_amd.pipeline import TrainPass
    x, w, qk, lab, dy = _inputs(B, N, H * Dh, B + N)
    p = TrainPass(B, N, H * Dh, H, "bf16")
    got = []
    for i in range(4):                                     # stages, then runs: call by call, recorded, replayed
        p.ws_attn.fill_(255)
        p.y.copy_(dy)
        args = (x, w, qk, lab, p.y if alias else dy)
        if i == 0:
            for _, call in p.stages(*args):
                call()
        else:
            p.run(*args)
        torch.cuda.synchronize()
        got.append(_outputs(p))
    for g in got[1:]:
        _same(got[0], g)
    assert got[0][6].isfinite().all() and got[0][6].any()


@pytest.mark.parametrize("grids,B,C", [((28, 14, 7), 3, 32), ((40, 20), 2, 64)])
def test_hierarchy(grids, B, C):
    from paper_2410_23608_amd.pipeline import HierarchyTrainPass
    cfg = [(B, h, h, C << i, (C << i) // 32, "bf16", 0.5, 0.0) for i, h in enumerate(grids)]
    args = [list(t) for t in zip(*(_inputs(B, c[1] * c[2], c[3], i) for i, c in enumerate(cfg)))]
    p = HierarchyTrainPass(cfg)
    got = []
    for i in range(4):
        for tp in p.passes:
            tp.ws_attn.fill_(255)
        if i == 0:
            for _, call in p.stages(*args):
                call()
        else:
            p.run(*args)
        torch.cuda.synchronize()
        got.append([t for tp in p.passes for t in _outputs(tp)])
    for g in got[1:]:
        _same(got[0], g)
