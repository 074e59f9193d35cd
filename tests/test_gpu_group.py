"""Launch groups: the stages of a hierarchy with one launch per step against the same calls one by one, for two to
four stages, grids that do not divide the workgroups' shares and images without a selected token; and what a group
refuses."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    from paper_2410_23608_amd import pipeline, spa
    return spa, pipeline


def _inputs(B, h, w, H, stages, train):
    g = torch.Generator(device="cuda")
    g.manual_seed(B * h + w + stages)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    cfg, cols = [], []
    for i in range(stages):
        hi, wi, Hi = h << (stages - 1 - i), w << (stages - 1 - i), H << i
        C = 32 * Hi
        cfg.append((B, hi, wi, C, Hi, "bf16", 0.5, -1.0 if i == 0 else -2.0))
        x = rnd(B, hi * wi, C).bfloat16()
        x[0] = 0                                   # (bias < 0: nothing selected, whatever a finer stage hands down)
        wt = (2 * rnd(C) / C ** 0.5).bfloat16()
        qkv = rnd(B, hi * wi, (2 if train else 3) * C).bfloat16()
        lab = (rnd(B, hi * wi) > 0).to(torch.uint8)
        cols.append((x, wt, qkv, lab, rnd(B, hi * wi, C).bfloat16()) if train else (x, wt, qkv))
    return cfg, [list(c) for c in zip(*cols)]


@pytest.mark.parametrize("form", ["lean", "packed", "train"])
@pytest.mark.parametrize("B,h,w,H,stages", [(3, 3, 5, 2, 4), (1, 7, 3, 3, 4), (5, 5, 3, 4, 3), (7, 9, 5, 2, 2), (2, 3, 3, 3, 2)])
def test_grouped_equals_one_by_one(mods, monkeypatch, B, h, w, H, stages, form):
    spa, pipeline = mods
    cfg, args = _inputs(B, h, w, H, stages, form == "train")
    make = (lambda: pipeline.HierarchyTrainPass(cfg)) if form == "train" else \
        (lambda: pipeline.HierarchyPass(cfg, lean=form == "lean"))
    grouped = make()
    calls = grouped.stages(*args)
    assert len(calls) <= 5
    for _ in range(2):
        for _, fn in calls:
            fn()
    monkeypatch.setattr(pipeline, "_groupable", lambda cfg: False)
    single = make()
    for _, fn in single.stages(*args):
        fn()
    torch.cuda.synchronize()
    for a, b in zip(grouped.passes, single.passes):
        T = int(b.mask.sum())
        assert int(b.mask[0].sum()) == 0
        for name in ("scores", "mask", "y"):
            assert torch.equal(getattr(a, name), getattr(b, name)), name
        if form != "lean":
            assert int(a.total) == T and torch.equal(a.cu_seqlens, b.cu_seqlens) and torch.equal(a.inv_pos, b.inv_pos)
            assert torch.equal(a.gather_idx[:T], b.gather_idx[:T]) and torch.equal(a.out[:T], b.out[:T])
        if form == "train":
            for name in ("dqk", "d_rg", "dx", "dw", "db", "loss"):
                u, v = getattr(a, name).float(), getattr(b, name).float()
                assert (u - v).abs().max() <= 2e-2 * max(1.0, float(v.abs().max())), name
    if form != "train":
        for a, b in zip(grouped.s_up[1:], single.s_up[1:]):
            assert torch.equal(a, b)


@pytest.mark.parametrize("B,N,C,H,tm", [(1, 1, 64, 2, None), (1, 50, 384, 6, None), (3, 129, 192, 3, None), (32, 196, 384, 6, None),
                                        (8, 400, 256, 8, "8"), (64, 196, 768, 12, None)])
def test_block_backward_projections_in_one_launch(mods, B, N, C, H, tm):
    """The weight sides beside other work (a launch group; two streams past its line) against everything in order: one
    chunk of rows and several, no row at all, 256 x 256 tiles (gemm_tm = 8: a group of separate launches)."""
    spa, pipeline = mods
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, w, dy = rnd(B, N, C), rnd(C) / C ** 0.5, rnd(B, N, C)
    if B > 1 or N == 1:
        x[0] = 0                                   # (nothing selected there)
    W = [rnd(3 * C, C) / C ** 0.5, rnd(3 * C), rnd(C, C) / C ** 0.5, rnd(C)]
    lab = (rnd(B, N) > 0).to(torch.uint8)
    got = []
    spa.spa_set_option("gemm_tm", tm)
    try:
        for beside in (True, False):
            p = pipeline.BlockTrainPass(B, N, C, H, "bf16", bias=-0.5, overlap_weight_grads=beside)
            assert not beside or p.grouped == (B * N * C * C <= 6e9)
            for t in (p.dW_qkv, p.db_qkv, p.dW_o, p.db_o, p.d_rg):
                t.fill_(float("nan"))
            for _ in range(2):
                p.run(x, w, *W, lab, dy)
            torch.cuda.synchronize()
            got.append(p)
    finally:
        spa.spa_set_option("gemm_tm")
    assert (int(got[1].mask[0].sum()) == 0) == (B > 1 or N == 1)
    for name in ("y", "d_rg", "dx", "dW_qkv", "db_qkv", "dW_o", "db_o", "dw", "db", "loss"):
        assert torch.equal(getattr(got[0], name), getattr(got[1], name)), name


def test_what_a_group_refuses(mods):
    spa, _ = mods
    x, w = torch.randn(1, 40, 64, device="cuda"), torch.randn(64, device="cuda")
    scores, mask = torch.zeros(1, 40, device="cuda"), torch.full((1, 40), 7, dtype=torch.uint8, device="cuda")
    with pytest.raises(spa.SpaError):
        spa.spa_group_end()
    for bad in (lambda: spa.spa_gate_select(x, w, 0.0, None, 0.5, scores, mask),            # fp32
                lambda: spa.spa_maxpool2x2(torch.zeros(1, 4, 4, device="cuda"), 4, 4, torch.zeros(1, 4, device="cuda"))):
        spa.spa_group_begin()
        spa.spa_gate_select(x.bfloat16(), w.bfloat16(), 0.0, None, 0.5, scores, mask)
        with pytest.raises(spa.SpaError):
            bad()
        with pytest.raises(spa.SpaError):          # the error ended the group
            spa.spa_group_end()
    torch.cuda.synchronize()
    assert (mask == 7).all()
    spa.spa_gate_select(x, w, 0.0, None, 0.5, scores, mask)
    torch.cuda.synchronize()
    assert (mask != 7).all()
