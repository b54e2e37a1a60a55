"""The buffers of a stage as a dictionary (no device needed)."""
import copy
import pickle

import pytest
import torch

from paper_2406_11836_amd import raster


def _pair():
    base = torch.arange(1024, dtype=torch.int64).to(torch.uint8)
    at = {"a": (0, 4, torch.int32), "b": (256, 3, torch.float32), "c": (512, 16, torch.uint8)}
    c = raster.Carved(base, at)
    plain = {k: base[o: o + n * raster._SIZE[d]].view(d) for k, (o, n, d) in at.items()}
    return c, plain


def _same(x, y):
    assert list(x) == list(y)
    for k in y:
        assert x[k].dtype == y[k].dtype and torch.equal(x[k].view(torch.uint8), y[k].view(torch.uint8)), k


READS = {
    "copy()": lambda d: d.copy(),
    "dict()": dict,
    "**": lambda d: {**d},
    "|": lambda d: d | {},
    "| from the right": lambda d: {} | d,
    "items()": lambda d: dict(d.items()),
    "copy.copy": copy.copy,
    "copy.deepcopy": copy.deepcopy,
    "pickle": lambda d: pickle.loads(pickle.dumps(d)),
    "update of another": lambda d: (lambda e: (e.update(d), e)[1])({}),
    "reversed": lambda d: {k: d[k] for k in list(reversed(d))[::-1]},
}


@pytest.mark.parametrize("touched", ["", "b"])
@pytest.mark.parametrize("how", READS)
def test_reads_see_every_buffer(how, touched):
    c, plain = _pair()
    for k in touched:
        c[k]
    _same(READS[how](c), plain)
    _same(c, plain)


def _both(f):
    c, plain = _pair()
    got = []
    for d in (c, plain):
        try:
            got.append(f(d))
        except KeyError as e:
            got.append(("KeyError", e.args))
    return c, plain, got


@pytest.mark.parametrize("f", [
    lambda d: d.pop("b").tolist(),
    lambda d: d.pop("x"),
    lambda d: d.pop("x", 5),
    lambda d: d.popitem()[0],
    lambda d: d["x"],
    lambda d: d.get("x", 7),
    lambda d: d.get("c").tolist(),
    lambda d: d.setdefault("a", None).tolist(),
    lambda d: d.setdefault("x", torch.ones(2)).tolist(),
    lambda d: d.update(x=torch.ones(1), a=torch.zeros(2)),
    lambda d: d.__ior__({"y": torch.ones(1)}) is d,
    lambda d: d.__delitem__("a"),
    lambda d: d.__delitem__("x"),
    lambda d: d.__setitem__("z", torch.ones(3)),
    lambda d: d.clear(),
    lambda d: (len(d), "a" in d, "x" in d, bool(d)),
    lambda d: repr(d),
])
def test_operations_as_on_a_plain_dictionary(f):
    c, plain, got = _both(f)
    assert got[0] == got[1]
    _same(c, plain)
    assert len(c) == len(plain) and bool(c) == bool(plain)


def test_equality_and_pointers():
    c, plain = _pair()
    d, _ = _pair()
    assert c != {} and {} != c and not (c == {}) and not ({"a": 1} == c)
    assert copy.copy(c)["a"] is c["a"] and c.copy()["b"] is c["b"]  # shallow
    assert copy.deepcopy(c)["a"].data_ptr() != c["a"].data_ptr()
    assert len(pickle.dumps(c)) < 2000  # the buffers, not the allocation for each
    for k in plain:
        c[k], d[k] = k, k  # (values that compare)
    assert c == {k: k for k in plain} and {k: k for k in plain} == c and c == d
    c, plain = _pair()
    assert c.ptr("b") == plain["b"].data_ptr()
    t = torch.ones(3)
    c["b"] = t
    assert c.ptr("b") == t.data_ptr() == raster._ptr(c, "b")
    c.update(a=t)
    assert c.ptr("a") == t.data_ptr()
    del c["a"]
    with pytest.raises(KeyError):
        c.ptr("a")
