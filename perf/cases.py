"""The work a user of Select-and-Pack Attention has this framework do, as measurable cases.

A case is one step of one of the pass objects of `paper_2410_23608_amd.pipeline`: the forward
pass in its forms, the training step, the block with its projections (forward, forward +
backward), the container-local form and the multi-stage hierarchy.  `launch` says how the
program calls it: "run" hands the step its tensors (each batch in tensors of its own, as a model
does), "prepared" keeps the launches bound to buffers that are filled again for every batch
(serving and benchmark loops).  Shapes are those of `workloads.WORKLOADS` and `HIER_STAGES`,
single images and larger batches of them, and odd grids beside them.
"""
from __future__ import annotations

import math

import torch

from paper_2410_23608_amd import pipeline, workloads

FORWARD = {"packed": {}, "gathered": dict(keep_packed_out=False, gathered=True),
           "selected": dict(keep_packed_out=False, gathered=True, from_mask=True)}


def _case(name, kind, B, h, w, C, H, lo, hi, launch="run", dtype="bf16", mask="disc", **more):
    c = dict(name=name, kind=kind, B=B, h=h, w=w, C=C, H=H, lo=lo, hi=hi, launch=launch, dtype=dtype, mask=mask)
    return {**c, **more}


def listed():
    return [
        # two small images in fp32, every output kept: the smallest call, bound by latency
        _case("tiny_f32", "forward", 2, 14, 14, 64, 2, 0.20, 0.40, dtype="f32", form="packed"),
        # one classification image at a time, as an online service does
        _case("vit_s_one_image", "forward", 1, 14, 14, 384, 6, 0.10, 0.90, form="selected"),
        # a classification batch in the two-launch inference form, launches kept
        _case("vit_s_batch", "forward", 64, 14, 14, 384, 6, 0.10, 0.90, "prepared", form="selected"),
        # a ragged batch just beyond 256 tokens an image; packed rows, output and lse kept (a backward pass elsewhere)
        _case("ragged_keep", "forward", 23, 17, 23, 448, 7, 0.05, 0.95, form="packed"),
        # detection, 800 x 1344 at stride 16: the headline batch, launches kept
        _case("det_batch", "forward", 8, 50, 84, 256, 8, 0.05, 0.40, "prepared", mask="rect", form="gathered"),
        # the same images in a batch of 32: offline inference, the largest forward pass
        _case("det_large", "forward", 32, 50, 84, 256, 8, 0.05, 0.40, mask="rect", form="gathered"),
        # a ViT-B-shaped training step with the selection loss
        _case("vit_b_train", "train", 64, 14, 14, 768, 12, 0.05, 0.95, gumbel=False),
        # four stages of 56^2 .. 7^2 tokens, inference, launches kept
        _case("hierarchy", "hierarchy", 16, 56, 56, 96, 3, 0.10, 0.60, "prepared", stages=4, train=False),
        # the same four stages, training
        _case("hierarchy_train", "hierarchy", 16, 56, 56, 96, 3, 0.10, 0.60, stages=4, train=True),
        # a ViT-S block with its projections, inference
        _case("block", "block", 64, 14, 14, 384, 6, 0.10, 0.90),
        # a ViT-B block with its projections, forward and backward: the largest step
        _case("block_train_large", "block_train", 128, 14, 14, 768, 12, 0.05, 0.95),
        # container-local attention, containers of 7 x 7 tokens on the map shifted by (3, 3)
        _case("container", "container", 64, 14, 14, 384, 6, 0.10, 0.90, L=49, shift=3),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    limit = _cost(next(c for c in listed() if c["name"] == "block_train_large"))
    while True:
        kind = rng.choice(["forward", "forward", "forward", "train", "train", "block", "block_train", "container", "hierarchy"])
        Dh = rng.choice([32, 64])
        launch, dtype, more = rng.choice(["run", "prepared"]), "bf16", {}
        mask = rng.choice(["disc", "rect"])
        lo = round(rng.uniform(0.05, 0.3), 2)
        hi = round(rng.uniform(lo + 0.1, 0.95), 2)
        H = _log_int(rng, 2, 16)
        if kind == "hierarchy":
            stages = rng.choice([2, 3, 4])
            h, w = (2 ** (stages - 1) * rng.randint(3, 9) for _ in range(2))
            B, H, Dh, mask = _log_int(rng, 1, 32), rng.choice([2, 3, 4]), 32, "disc"
            more = dict(stages=stages, train=rng.random() < 0.5)
        else:
            long = kind in ("forward", "train") and rng.random() < 0.5
            h = _log_int(rng, 17, 64) if long else rng.randint(5, 16)
            w = max(17 if long else 5, int(h * rng.uniform(0.7, 1.7)))
            B = _log_int(rng, 1, 128)
            if kind == "forward":
                more = dict(form=rng.choice(["packed", "gathered"] + (["selected", "selected"] if h * w <= 256 else [])))
                if rng.random() < 0.15 and B * h * w <= 4096:
                    dtype = "f32"
            elif kind == "train":
                more = dict(gumbel=rng.random() < 0.3)
            elif kind == "container":
                more = dict(L=rng.choice([25, 49, 64]), shift=rng.randint(0, 3))
        c = _case("", kind, B, h, w, H * Dh, H, lo, hi, launch, dtype, mask, **more)
        del c["name"]
        if H * Dh <= 1024 and B * h * w <= 140_000 and _cost(c) <= limit:
            return c


# ---------------------------------------------------------------------------------- inputs
def _stage_cases(c):
    """The stages of a hierarchy as (h, w, C, H), finest first: the grid halves, the width doubles."""
    return [(c["h"] >> i, c["w"] >> i, c["C"] << i, c["H"] << i) for i in range(c.get("stages", 1))]


def _tokens(g, td, fg, C):
    """Token features whose gate logit under w has the sign of the foreground and a magnitude of at
    least 0.5, so that no selection hangs on the last bit of a sum; w ~ N(0, 1/C)."""
    w = (torch.randn(C, generator=g, device="cuda") / C ** 0.5).to(td)
    z = torch.randn(*fg.shape, C, generator=g, device="cuda")
    mag = 0.5 + torch.randn(fg.shape, generator=g, device="cuda").abs()
    wf = w.float()
    coef = (torch.where(fg, mag, -mag) - z @ wf) / (wf @ wf)
    return (z + coef[..., None] * wf).to(td), w


def _noise(g, x, w):
    """Logistic noise of the stochastic selection, kept away from the threshold as the logits are."""
    u = torch.rand(x.shape[:2], generator=g, device="cuda").clamp_(1e-6, 1 - 1e-6)
    e = torch.log(u) - torch.log1p(-u)
    s = x.float() @ w.float() + e
    return e + torch.where(s >= 0, 0.05, -0.05) * (s.abs() < 0.05)


def prepare(case, seed):
    c = case
    B, N, C, H, dtype = c["B"], c["h"] * c["w"], c["C"], c["H"], c["dtype"]
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    masks = workloads.foreground_masks(
        workloads.Workload("case", B, (c["h"], c["w"]), C, H, dtype, (c["lo"], c["hi"]), c["mask"]), seed)
    fg = torch.from_numpy(masks).cuda().bool()
    flip = lambda f: (f ^ (torch.rand(f.shape, generator=g, device="cuda") < 0.05)).to(torch.uint8)
    kw = {}
    if c["kind"] == "hierarchy":
        cfg, cols = [], []
        for i, (h, w, Ci, Hi) in enumerate(_stage_cases(c)):
            own = fg
            if i > 0:      # the foreground of the 2x coarser map; this stage's own gate finds most of it
                fg = fg.view(B, h, 2, w, 2).amax(4).amax(2).reshape(B, h * w)
                own = fg & (torch.rand(fg.shape, generator=g, device="cuda") < 0.85)
            cfg.append((B, h, w, Ci, Hi, dtype, 0.5, 0.0))
            x, wt = _tokens(g, td, own, Ci)
            cols.append((x, wt, rnd(B, h * w, 2 * Ci).to(td), flip(fg), rnd(B, h * w, Ci).to(td)) if c["train"]
                        else (x, wt, rnd(B, h * w, 3 * Ci).to(td)))
        obj = pipeline.HierarchyTrainPass(cfg) if c["train"] else pipeline.HierarchyPass(cfg, lean=True)
        args = tuple(list(col) for col in zip(*cols))
    else:
        x, w = _tokens(g, td, fg, C)
        if c["kind"] == "forward":
            obj = pipeline.ForwardPass(B, N, C, H, dtype, **FORWARD[c["form"]])
            args = (x, w, rnd(B, N, 3 * C).to(td))
        elif c["kind"] == "container":
            obj = pipeline.ContainerForwardPass(B, c["h"], c["w"], C, H, dtype, c["L"], (c["shift"], c["shift"]))
            args = (x, w, rnd(B, N, 3 * C).to(td))
        elif c["kind"] == "train":
            obj = pipeline.TrainPass(B, N, C, H, dtype)
            args = (x, w, rnd(B, N, 2 * C).to(td), flip(fg), rnd(B, N, C).to(td))
            if c["gumbel"]:
                kw = dict(noise=_noise(g, x, w))
        else:
            weights = tuple((rnd(*s) / C ** 0.5).to(td) for s in ((3 * C, C), (3 * C,), (C, C), (C,)))
            if c["kind"] == "block":
                obj = pipeline.BlockPass(B, N, C, H, dtype)
                args = (x, w, *weights)
            else:
                obj = pipeline.BlockTrainPass(B, N, C, H, dtype)
                args = (x, w, *weights, flip(fg), rnd(B, N, C).to(td))
    launches = [fn for _, fn in obj.stages(*args, **kw)] if c["launch"] == "prepared" else None
    return dict(kind=c["kind"], train=c.get("train"), obj=obj, args=args, kw=kw, launches=launches)


# ---------------------------------------------------------------------------------- the step
RESULTS = {
    "forward": ("y", "scores", "mask"),
    "packed": ("y", "scores", "mask", "cu_seqlens", "gather_idx", "inv_pos", "total", "out", "lse"),
    "gathered": ("y", "scores", "mask", "cu_seqlens", "gather_idx", "inv_pos", "total"),
    "container": ("y", "scores", "mask", "cu_seqlens", "gather_idx", "inv_pos", "total", "seg_cu_seqlens", "n_segments"),
    "block": ("y", "scores", "mask", "cu_seqlens", "gather_idx", "inv_pos", "total"),
    "train": ("y", "loss", "dx", "dqk", "d_rg", "dw", "db", "scores", "mask", "cu_seqlens", "total"),
    "block_train": ("y", "loss", "dx", "d_rg", "dw", "db", "dW_qkv", "db_qkv", "dW_o", "db_o", "scores", "mask", "total"),
}


def _results(kind, obj):
    if kind == "forward" and not obj.from_mask:
        kind = "gathered" if obj.gathered else "packed"
    return {name: getattr(obj, name) for name in RESULTS[kind]}


def run(state):
    obj, kind = state["obj"], state["kind"]
    if state["launches"] is not None:
        for launch in state["launches"]:
            launch()
    elif state["kw"]:      # the stochastic selection is an option of stages()
        for _, launch in obj.stages(*state["args"], **state["kw"]):
            launch()
    else:
        obj.run(*state["args"])
    if kind == "hierarchy":
        return [_results("train" if state["train"] else "forward", p) for p in obj.passes]
    return _results(kind, obj)


# ----------------------------------------------------------------------- what a step cannot do without
def _moments(c):
    """Mean and mean square of the selected fraction, uniform in [lo, hi]."""
    lo, hi = c["lo"], c["hi"]
    return (lo + hi) / 2, (lo * lo + lo * hi + hi * hi) / 3


def work(case):
    c = case
    B, e = c["B"], 2 if c["dtype"] == "bf16" else 4
    f1, f2 = _moments(c)
    nbytes = flops = 0.0
    for h, w, C, H in _stage_cases(c):
        N = h * w
        cap, T, n2 = B * N, B * N * f1, B * N * N * f2
        if c["kind"] == "container":
            n2 = min(n2, T * c["L"])
        full, sel = cap * C * e, T * C * e
        train = c["kind"] in ("train", "block_train") or bool(c.get("train"))
        nbytes += full + full + cap * 5 + C * e                              # x in; y, scores, mask out; w
        flops += 2.0 * cap * C + 4.0 * C * n2                                # gate, attention
        if c["kind"] in ("block", "block_train"):
            nbytes += 4 * C * C * e                                          # projection weights
            flops += 8.0 * T * C * C
        else:
            nbytes += (2 if train else 3) * sel                              # selected rows of q | k | v
        if c.get("form", "gathered") != "selected" and c["kind"] != "hierarchy":
            nbytes += 4 * (B + 1) + 8 * cap                                  # packing index
        if c.get("form") == "packed":
            nbytes += sel + 4 * H * T                                        # packed output, lse
        if train:
            flops += 10.0 * C * n2 + 6.0 * cap * C                           # attention and gate backward
            nbytes += cap + 2 * full                                         # labels in; dx, d_rg out
            if c["kind"] == "block_train":
                flops += 16.0 * T * C * C
                nbytes += full + 16 * C * C                                  # dy of the residual rows; fp32 dW
            else:
                nbytes += sel + 2 * full                                     # dy of the selected rows in; dq | dk out
    return {"bytes": nbytes, "flops": flops}


def _cost(c):
    """Rough seconds of a step, to keep drawn cases within the largest listed one."""
    w = work(c)
    return w["bytes"] / 3e12 + w["flops"] / (20e12 if c["dtype"] == "f32" else 300e12)


def tolerance(case):
    # fp32 sums in another order; bf16 inputs and outputs, probabilities and gradients rounded to bf16 on the way
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
