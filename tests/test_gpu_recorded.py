"""run() replays a recorded step from the second run on: every run on new tensors, on another
stream, after an attribute changed or with other optional inputs must give what the stages issued
one by one give, bit for bit, and refuse what they refuse."""
import dataclasses

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
            p.bias = ref.bias = 0.75                    # drops the recording
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
