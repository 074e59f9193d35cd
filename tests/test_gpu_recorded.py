"""run() replays a recorded step from the second run on: every run on new tensors, on another
stream, after an attribute changed or with other optional inputs must give what the stages issued
one by one give, bit for bit, and refuse what they refuse."""
import copy
import dataclasses
import gc
import weakref

import pytest
import torch

from paper_2410_23608_amd import workloads as wlmod
from spa_harness import dev

pytestmark = pytest.mark.gpu

WL = dataclasses.replace(wlmod.WORKLOADS["vit_s"], B=3)


@pytest.fixture(scope="module")
def pipeline():
    from paper_2410_23608_amd import pipeline as mod
    return mod


def _inputs(kind, seed):
    b = wlmod.generate(dataclasses.replace(WL, train=True), seed)
    x, w, qkv = (dev(b[k], "bf16") for k in ("x", "w", "qkv"))
    if kind == "train":
        return x, w, qkv[:, :, :2 * WL.C].contiguous(), dev(b["labels"]), dev(b["dy"], "bf16")
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    weights = [(torch.randn(*s, generator=g, device="cuda") / WL.C ** 0.5).bfloat16()
               for s in ((3 * WL.C, WL.C), (3 * WL.C,), (WL.C, WL.C), (WL.C,))]
    return {"forward": (x, w, qkv), "container": (x, w, qkv), "block": (x, w, *weights),
            "block_train": (x, w, *weights, dev(b["labels"]), dev(b["dy"], "bf16"))}[kind]


def _make(pipeline, kind):
    args = (WL.B, WL.N, WL.C, WL.H, "bf16")
    if kind == "forward":
        return pipeline.ForwardPass(*args)
    if kind == "container":
        return pipeline.ContainerForwardPass(WL.B, *WL.grid, WL.C, WL.H, "bf16", 49, (3, 3))
    return {"train": pipeline.TrainPass, "block": pipeline.BlockPass, "block_train": pipeline.BlockTrainPass}[kind](*args)


def _results(p):
    names = ("y", "scores", "mask", "loss", "dx", "dw", "dqk", "dW_qkv", "dW_o")
    return [getattr(p, n).clone() for n in names if hasattr(p, n)]


@pytest.mark.parametrize("kind", ["forward", "train", "block", "block_train", "container"])
def test_recorded_runs_equal_stages(pipeline, kind):
    p, ref = _make(pipeline, kind), _make(pipeline, kind)
    other = torch.cuda.Stream()
    for i in range(6):
        if i == 4:
            p.bias = ref.bias = 0.75
        ins = _inputs(kind, 40 + i)                     # new tensors every time
        torch.cuda.synchronize()
        if i == 3:
            with torch.cuda.stream(other):
                p.run(*ins)
        else:
            p.run(*ins)
        for _, fn in ref.stages(*ins):
            fn()
        torch.cuda.synchronize()
        for a, b in zip(_results(p), _results(ref)):
            assert torch.equal(a, b), (kind, i)


def test_recorded_run_with_optional_inputs_and_refusals(pipeline):
    p = _make(pipeline, "forward")
    x, w, qkv = _inputs("forward", 7)
    base = torch.randn_like(x)
    plain = p.run(x, w, qkv).clone()
    for _ in range(3):
        assert torch.equal(p.run(x, w, qkv), plain)
    want = None
    for _ in range(3):
        got = p.run(x, w, qkv, base=base)
        want = got.clone() if want is None else want
        assert torch.equal(got, want) and not torch.equal(got, plain)
    assert torch.equal(p.run(x, w, qkv), plain)
    for bad in ((x.float(), w, qkv), (x, w, qkv.cpu()), (x.transpose(0, 1).contiguous().transpose(0, 1), w, qkv)):
        with pytest.raises(ValueError):
            p.run(*bad)


@pytest.mark.parametrize("form", [dict(gathered=True), dict(gathered=True, keep_packed_out=False, from_mask=True)])
def test_rows_inside_a_wider_buffer_are_not_recorded(pipeline, monkeypatch, form):
    """q | k | v as a column slice is taken stage by stage on every run, with no attempt at a recording of it."""
    made = []
    record = pipeline.spa.record
    monkeypatch.setattr(pipeline.spa, "record", lambda *a: made.append(1) or record(*a))
    p, ref = (pipeline.ForwardPass(WL.B, WL.N, WL.C, WL.H, "bf16", **form) for _ in range(2))
    x, w, qkv = _inputs("forward", 3)
    wide = torch.cat([qkv, torch.full_like(x, float("nan"))], -1)
    for _ in range(4):
        p.y.fill_(float("nan"))
        y = p.run(x, w, wide[..., :3 * WL.C])
        for _, fn in ref.stages(x, w, qkv):
            fn()
        assert torch.equal(y, ref.y)
    assert not made
    for _ in range(3):
        assert torch.equal(p.run(x, w, qkv), ref.y)
    assert len(made) == 1
    assert torch.equal(p.run(x, w, wide[..., :3 * WL.C]), ref.y) and len(made) == 1


@pytest.fixture
def recordings(pipeline, monkeypatch):
    """The recordings made while the test runs."""
    made, record = [], pipeline.spa.record
    monkeypatch.setattr(pipeline.spa, "record", lambda *a: made.append(record(*a)) or made[-1])
    return made


def _hierarchy(pipeline, train):
    """Two stages and their inputs per seed."""
    cfg = [(2, 8, 12, 64, 2, "bf16", 0.5, 0.0), (2, 4, 6, 128, 4, "bf16", 0.5, 0.1)]

    def inputs(seed):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
        cols = []
        for B, h, w, C, H, *_ in cfg:
            N = h * w
            col = (rnd(B, N, C), rnd(C) / C ** 0.5, rnd(B, N, (2 if train else 3) * C))
            cols.append(col + ((rnd(B, N) > 0).to(torch.uint8), rnd(B, N, C)) if train else col)
        return [list(c) for c in zip(*cols)]
    make = (lambda: pipeline.HierarchyTrainPass(cfg)) if train else (lambda: pipeline.HierarchyPass(cfg))
    return make, inputs


def test_attributes_of_one_pass_leave_the_others_recorded(pipeline, recordings):
    a, b = _make(pipeline, "forward"), _make(pipeline, "forward")
    ins = _inputs("forward", 1)
    for _ in range(2):
        a.run(*ins)
        b.run(*ins)
    assert len(recordings) == 2
    for i in range(4):
        b.note = i
        b.lse = torch.zeros_like(b.lse)
        a.run(*ins)
    assert len(recordings) == 2 and recordings[0].runs == 5


@pytest.mark.parametrize("how", ["attribute", "data", "set_"])
def test_a_replaced_buffer_is_written(pipeline, recordings, how):
    """y under another name, in other memory: the attribute assigned, its data assigned, its storage set."""
    p, ref = _make(pipeline, "forward"), _make(pipeline, "forward")
    for i in range(6):
        ins = _inputs("forward", 60 + i)
        if i == 3:
            old, new = p.y.detach(), torch.empty_like(p.y)
            kept = old.clone()
            if how == "attribute":
                p.y = new
            elif how == "data":
                old = p.y.data
                p.y.data = new
            else:
                p.y.set_(new.untyped_storage(), 0, new.shape, new.stride())
            assert p.y.data_ptr() == new.data_ptr()
        y = p.run(*ins)
        for _, fn in ref.stages(*ins):
            fn()
        torch.cuda.synchronize()
        assert y is p.y and torch.equal(y, ref.y)
    assert torch.equal(old, kept) and len(recordings) == 1      # other memory is no reason to record again


def test_a_buffer_of_another_shape_takes_the_stages(pipeline):
    p = _make(pipeline, "forward")
    ins = _inputs("forward", 2)
    for _ in range(3):
        y = p.run(*ins).clone()
    p.y = torch.empty(1, dtype=torch.bfloat16, device="cuda")
    for _ in range(2):
        with pytest.raises((ValueError, TypeError)):
            p.run(*ins)
    p.y = torch.empty_like(y)
    assert torch.equal(p.run(*ins), y)


@pytest.mark.parametrize("train", [False, True])
def test_a_replaced_stage_of_a_hierarchy_is_run(pipeline, recordings, train):
    make, inputs = _hierarchy(pipeline, train)
    p, ref = make(), make()
    for i in range(8):
        ins = inputs(i)
        if i == 3:
            old = p.passes[1]
            p.passes[1] = make().passes[1]
            before = old.y.clone()
        if i == 5 and not train:
            p.s_up[1] = torch.full_like(p.s_up[1], float("nan"))
        if i == 6:
            p.passes[0].scores = torch.empty_like(p.passes[0].scores)
            p.passes[1].container_len = 0
        got = p.run(*ins)
        for _, fn in ref.stages(*ins):
            fn()
        torch.cuda.synchronize()
        assert all(a is (q.loss if train else q.y) for a, q in zip(got, p.passes))
        for q, r in zip(p.passes, ref.passes):
            for name in ("y", "scores", "mask", "cu_seqlens") + (("dx", "dqk", "dw", "db", "loss") if train else ()):
                assert torch.equal(getattr(q, name), getattr(r, name)), (i, name)
        if not train:
            assert torch.equal(p.s_up[1], ref.s_up[1])
        if i >= 3:
            assert torch.equal(old.y, before)
    assert recordings[0].runs >= 4


def test_what_changes_on_every_run_is_not_recorded_on_every_run(pipeline, recordings):
    p = _make(pipeline, "forward")
    ins = _inputs("forward", 4)
    want = p.run(*ins).clone()
    for i in range(40):
        p.note = object()
        p.y.zero_()
        assert torch.equal(p.run(*ins), want)
    assert len(recordings) <= 6
    for _ in range(80):                                  # and once it stays as it is the step is recorded
        p.run(*ins)
    assert recordings[-1].runs >= 2


def test_recordings_hold_nothing_alive(pipeline):
    make, inputs = _hierarchy(pipeline, True)
    p, q = make(), _make(pipeline, "forward")
    for _ in range(3):
        p.run(*inputs(0))
        q.run(*_inputs("forward", 0))
    refs = [weakref.ref(o) for o in (p, p.passes[1], p.passes[1].y, q, q.y)]
    dup = copy.deepcopy(q)                               # (a copy starts without recordings)
    assert dup._plan is None and torch.equal(dup.run(*_inputs("forward", 0)), q.y)
    gc.disable()
    try:
        del p, q
        assert all(r() is None for r in refs)
    finally:
        gc.enable()


@pytest.mark.parametrize("kind", ["forward", "train", "block", "block_train", "container", "hierarchy", "hierarchy_train"])
def test_a_bias_that_is_learned_keeps_the_recording(pipeline, recordings, kind):
    """A new bias before every step, as a training program assigns it, and other thresholds and loss scales: one
    recording, and what the stages give."""
    if kind.startswith("hierarchy"):
        make, inputs = _hierarchy(pipeline, kind == "hierarchy_train")
    else:
        make, inputs = lambda: _make(pipeline, kind), lambda seed: _inputs(kind, seed)
    p, ref = make(), make()
    for i in range(7):
        ins = inputs(i)
        for o in (p, ref):
            for n, q in enumerate(getattr(o, "passes", [o])):
                q.bias = [0.0, -0.25, 0.5, 1, -1.0, 0.125, 0][i] + 0.01 * n      # (whole numbers too)
                q.tau = 0.5 if i < 4 else 0.4
                if hasattr(q, "loss_scale") and i == 5:
                    q.loss_scale = 0.02
        p.run(*ins)
        for _, fn in ref.stages(*ins):
            fn()
        torch.cuda.synchronize()
        for q, r in zip(getattr(p, "passes", [p]), getattr(ref, "passes", [ref])):
            assert all(torch.equal(a, b) for a, b in zip(_results(q), _results(r))), i
    assert len(recordings) == 1 and recordings[0].runs == 6


def test_numbers_a_step_refuses(pipeline, recordings):
    p = _make(pipeline, "forward")
    ins = _inputs("forward", 1)
    for _ in range(3):
        want = p.run(*ins).clone()
    p.tau = 1.5
    for _ in range(2):
        with pytest.raises(pipeline.spa.SpaError):
            p.run(*ins)
    p.tau, p.bias = 0.5, None
    with pytest.raises(TypeError):
        p.run(*ins)
    p.bias = torch.zeros((), device="cuda")              # what float() takes, stage by stage
    assert torch.equal(p.run(*ins), want)
    p.bias = 0.0
    assert torch.equal(p.run(*ins), want)


def test_parameters_are_recorded_and_subclasses_are_not(pipeline, recordings):
    class Marked(torch.Tensor):
        pass
    p = _make(pipeline, "forward")
    x, w, qkv = _inputs("forward", 5)
    want = p.run(x, w, qkv).clone()
    for _ in range(3):
        assert torch.equal(p.run(x, torch.nn.Parameter(w, requires_grad=False), qkv), want)
    assert len(recordings) == 1 and recordings[0].runs == 3
    for _ in range(2):
        assert torch.equal(p.run(x, w.as_subclass(Marked), qkv), want)
    assert recordings[0].runs == 3
