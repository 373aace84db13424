"""The request array of a pose batch (CPU only): filled by column or one record after the
other, the same requests come out, and what is refused is refused the same way."""
import ctypes
import decimal
from types import SimpleNamespace

import numpy as np
import pytest
import torch


class Floatable:
    def __init__(self, v):
        self.v = v

    def __float__(self):
        return self.v


def _request(rng, n=5):
    q = rng.normal(size=4)
    return SimpleNamespace(K=rng.uniform(300, 600, 4), q0=q / np.linalg.norm(q), t0=rng.normal(size=3),
                           X=rng.normal(size=(n, 3)), uv=rng.uniform(0, 640, (n, 2)))


def _one_by_one(balib, requests, keep):
    arr = (balib.PoseRequest * len(requests))()
    for i, q in enumerate(requests):
        arr[i] = balib._pose_request(q.K, q.q0, q.t0, q.X, q.uv, keep)
    return arr


def _values(arr, n):
    out = []
    for i in range(n):
        r = arr[i]
        X = (ctypes.c_double * (3 * r.n)).from_address(r.X)
        uv = (ctypes.c_double * (2 * r.n)).from_address(r.uv)
        out.append((bytes(r.K), bytes(r.pose0), r.n, bytes(X), bytes(uv)))
    return out


ACCEPTED = {
    "arrays": lambda v: v,
    "float32": lambda v: v.astype(np.float32),
    "lists": lambda v: v.tolist(),
    "tuples": lambda v: tuple(v),
    "integers": lambda v: [int(x) for x in v],
    "texts": lambda v: [repr(float(x)) for x in v],
    "decimals": lambda v: [decimal.Decimal(float(x)) for x in v],
    "floatable": lambda v: [Floatable(float(x)) for x in v],
    "tensors": lambda v: torch.tensor(v),
    "tensors of tensors": lambda v: [torch.tensor(float(x), requires_grad=True) for x in v],
    "dict values": lambda v: dict(enumerate(v)).values(),
    "iterators": lambda v: iter(v.tolist()),
    "one-element arrays": lambda v: [np.array([x]) for x in v][:2] + list(v[2:]),
    "strided": lambda v: np.repeat(v, 2)[::2],
    "masked": lambda v: np.ma.masked_array(v, mask=[i == 1 for i in range(len(v))]),
    "nan": lambda v: np.where(np.arange(len(v)) == 1, np.nan, v),
}


@pytest.mark.filterwarnings("ignore")
@pytest.mark.parametrize("n", [3, 16, 40])
@pytest.mark.parametrize("form", list(ACCEPTED))
@pytest.mark.parametrize("which", ["first", "all"])
def test_what_was_accepted(balib, n, form, which):
    """K, q0 and t0 in every form that float() and iteration take, in one request or in all."""
    def make():
        rs = [_request(np.random.default_rng(i), 3 + i % 4) for i in range(n)]
        for r in rs[:1] if which == "first" else rs:
            for f in ("K", "q0", "t0"):
                setattr(r, f, ACCEPTED[form](getattr(r, f)))
        return rs
    ka, kb = [], []
    a, b = balib._pose_requests(make(), ka), _one_by_one(balib, make(), kb)
    assert _values(a, n) == _values(b, n)


REFUSED = {
    "none": lambda v: [None] + list(v)[1:],
    "none in an array": lambda v: np.array([None] + list(v)[1:], object),
    "complex": lambda v: [1j] + list(v)[1:],
    "word": lambda v: ["x"] + list(v)[1:],
    "too long": lambda v: list(v) + [1.0] * 5,
    "a row": lambda v: [list(v)],
    "a number": lambda v: 1.0,
    "nothing": lambda v: None,
}


@pytest.mark.filterwarnings("ignore")
@pytest.mark.parametrize("form", list(REFUSED))
@pytest.mark.parametrize("field", ["K", "q0", "t0"])
def test_what_was_refused(balib, form, field):
    def make():
        rs = [_request(np.random.default_rng(i)) for i in range(20)]
        setattr(rs[7], field, REFUSED[form](getattr(rs[7], field)))
        return rs
    try:
        want = _values(_one_by_one(balib, make(), kb := []), 20)
    except Exception as e:
        with pytest.raises(type(e)):
            balib._pose_requests(make(), [])
    else:  # a pose longer than it should be may run over into the next field
        assert _values(balib._pose_requests(make(), ka := []), 20) == want


def test_the_first_bad_request_is_the_one_reported(balib):
    """Points of one request that are no numbers, pixels of an earlier one that are none."""
    rs = [_request(np.random.default_rng(i)) for i in range(20)]
    rs[3].uv = [["pixel", 0.0]]
    rs[2].X = [["point", 0.0, 0.0]]
    rs[1].uv = None
    for bad in (1, 2, 3):
        with pytest.raises(Exception) as a:
            balib._pose_requests(rs, [])
        with pytest.raises(Exception) as b:
            _one_by_one(balib, rs, [])
        assert str(a.value) == str(b.value)
        rs[bad] = _request(np.random.default_rng(bad))
