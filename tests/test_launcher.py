"""The native program of a recorded step without a GPU: what it compares of its owner on every run, and what it refuses to
be made of.  (A program without calls issues nothing; tensors always fail its check here, as they are not on a device.)"""
import gc
import sys

import pytest
import torch

from paper_2410_23608_amd import spa

Program = spa._launcher.Program


class Owner:
    def __init__(self, **kw):
        self.__dict__.update(kw)


def _program(*places):
    return Program((), (), places)


@pytest.mark.parametrize("value,other", [(3, 4), (0.5, 0.25), (None, 0), ("a", "b"), ((1, 2), (1, 3)), ([1, (2, 3)], [1, (2, 4)]),
                                         (True, False)])
def test_constants_are_compared(value, other):
    o = Owner(a=value)
    p = _program(("constant", 0, "a", -1, value))
    assert p(o) is True and p.runs == 1
    o.a = type(value)(value) if value is not None else None
    assert p(o) is True
    o.a = other
    assert p(o) is False
    del o.a
    assert p(o) is False and p.runs == 2
    assert p() is False and p(o, 1) is False


def test_elements_lengths_and_objects():
    inner = Owner(n=1)
    o = Owner(parts=[None, inner], k=(5, 6))
    p = _program(("length", 0, "parts", 2, None), ("constant", 0, "parts", 0, None), ("object", 0, "parts", 1, Owner),
                 ("constant", 1, "n", -1, 1), ("length", 0, "k", 2, None), ("constant", 0, "k", 1, 6))
    assert p(o) is True
    o.parts[1] = Owner(n=1)                              # another object of the type, in the same state
    assert p(o) is True
    o.parts[1].n = 2
    assert p(o) is False
    o.parts[1] = inner
    o.parts.append(None)
    assert p(o) is False
    o.parts = o.parts[:1]
    assert p(o) is False
    o.parts = [None, type("Sub", (Owner,), {})(n=1)]     # another type may do anything with the same attributes
    assert p(o) is False
    o.parts = (None, inner)
    assert p(o) is True
    o.k = {0: 5, 1: 6}
    assert p(o) is False
    assert p(object()) is False                          # no attributes at all


def test_numbers_are_open_places_of_plain_numbers():
    o = Owner(bias=0.5)
    p = _program(("number", 0, "bias", -1, None))
    for v in (0.5, -1, 0, 1e30, float("nan")):
        o.bias = v
        assert p(o) is True
    for v in (None, "1", True, torch.zeros(()), 10 ** 400):
        o.bias = v
        assert p(o) is False


def test_a_comparison_that_raises_or_is_ambiguous_is_a_mismatch():
    class Bad:
        def __eq__(self, other):
            raise RuntimeError("no")
    o = Owner(a=Bad())
    p = _program(("constant", 0, "a", -1, Bad()))
    assert p(o) is False
    o.a = torch.zeros(3)
    assert _program(("constant", 0, "a", -1, torch.zeros(3)))(o) is False


def test_tensors_that_are_not_device_tensors_do_not_match():
    t = torch.zeros(2, 3)
    p = Program((), (t, None), (("tensor", 0, "y", -1, t),))
    o = Owner(y=t)
    assert p(o, t, None) is False and p(o, t, t) is False and p(o, None, None) is False
    assert Program((), (None,), ())(Owner(), None) is True


def test_what_a_program_is_not_made_of():
    for bad in (((1,), ()), ((), (1,)), ((), ("x",))):
        with pytest.raises(TypeError):
            Program(*bad)
    for places in ([], (1,), (("constant", 0, "a"),), (("constant", 0, 1, -1, None),), (("tensor", 0, "a", -1, 3),)):
        with pytest.raises(TypeError):
            Program((), (), places)
    with pytest.raises(ValueError):
        _program(("constant", 1, "a", -1, 0))            # an object that comes after it
    with pytest.raises(ValueError):
        Program((), (None,) * 600)
    with pytest.raises(TypeError):
        _program()(Owner(), key=1)


def test_references_are_given_back():
    value, t, o = (1, object()), torch.zeros(2), Owner(n=1)
    o.a, o.y = value, t
    gc.collect()
    before = [sys.getrefcount(x) for x in (value, t, o)]
    for _ in range(50):
        p = Program((), (t,), (("constant", 0, "a", -1, value), ("tensor", 0, "y", -1, t)))
        p(o, t)
        with pytest.raises(ValueError):
            Program((), (), (("constant", 0, "a", -1, value), ("constant", 3, "a", -1, value)))
    del p
    gc.collect()
    assert [sys.getrefcount(x) for x in (value, t, o)] == before
