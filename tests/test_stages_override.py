"""A run issues what stages() lists, also where a subclass or a program puts its own stages() in place of a training pass's."""
import pytest
import torch

from paper_2410_23608_amd import pipeline


def _bare(cls, **attributes):
    p = object.__new__(cls)                        # (no device here: a pass without its buffers)
    p.__dict__.update(attributes)
    return p


@pytest.mark.parametrize("N", [196, 400])
def test_train_pass(N):
    class Own(pipeline.TrainPass):
        def stages(self, x, w, qk, labels, dy):
            return [("own", (x, w, qk, labels, dy))]

    assert _bare(Own, N=N)._steps(1, 2, 3, 4, 5) == [("own", (1, 2, 3, 4, 5))]
    p = _bare(pipeline.TrainPass, N=N)
    p.stages = lambda *a: [("put", a)]
    assert p._steps(1, 2, 3, 4, 5) == [("put", (1, 2, 3, 4, 5))]
    p = _bare(pipeline.TrainPass, N=N)
    p._all_stages = lambda early_d, *a: [(early_d, a)]
    assert p._steps(1, 2, 3, 4, 5) == [(N > 256, (1, 2, 3, 4, 5))]


def test_hierarchy_and_its_passes(monkeypatch):
    seen = []

    class Own(pipeline.TrainPass):
        def stages(self, *inputs, **options):
            seen.append((inputs, options))
            return [(f"stage {i}", None) for i in range(5)]

    class OwnHierarchy(pipeline.HierarchyTrainPass):
        def stages(self, *inputs):
            return [("own", inputs)]

    cfg = [(2, 28 >> i, 28 >> i, 64 << i, 2 << i, "f32", 0.5, 0.0) for i in range(2)]        # (fp32: stage by stage)
    passes = [_bare(Own, N=c[1] * c[2], scores=f"scores {i}", gated=False, pack_pair=True) for i, c in enumerate(cfg)]
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: None)
    t = tuple(range(10))
    for cls, want in ((pipeline.HierarchyTrainPass, None), (OwnHierarchy, [("own", ((0, 1), (2, 3), (4, 5), (6, 7), (8, 9)))])):
        got = _bare(cls, cfg=cfg, passes=passes, concurrent=False)._steps(*t)
        if want is not None:
            assert got == want and len(seen) == 2
        else:
            assert [i for i, _ in seen] == [(0, 2, 4, 6, 8), (1, 3, 5, 7, 9)] and [n for n, _ in got].count("s1.stage 4") == 1
            assert seen[1][1] == dict(s_fine="scores 0", grid=(14, 14))
