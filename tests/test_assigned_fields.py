"""A tensor that a program assigns to a field of a particle, rate or cotangent
set takes the field's place in the ABI structs, whenever it is assigned (CPU
tensors: addresses and copies only)."""
import copy
import io

import pytest
import torch

from paper_2310_03596_amd.adjoint import Cotangent
from paper_2310_03596_amd.state import Particles, Rates

N = 5
# (set, its field, the struct's member), of one, of several and of 8-byte entries
FIELDS = [("particles", "S", "S"), ("particles", "x", "x"), ("particles", "E", "E"), ("particles", "w", "omega"),
          ("rates", "hi", "hi"), ("rates", "Lhi", "Lhi"), ("cotangent", "x", "x"), ("cotangent", "S", "S"),
          ("cotangent", "w", "omega"), ("cotangent", "c", "c")]


def _make(kind, prec):
    return {"particles": lambda: Particles(N, prec, True, "cpu"), "rates": lambda: Rates(N, prec, True, "cpu"),
            "cotangent": lambda: Cotangent(N, prec, "cpu", True)}[kind]()


def _pointers(struct, member):
    got = getattr(struct, member)
    return list(got) if hasattr(got, "__len__") else [got]


def _rows(t):
    return [row.data_ptr() for row in t] if t.dim() == 2 else [t.data_ptr()]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("after", [False, True], ids=["before a call", "after a call"])
@pytest.mark.parametrize("kind,field,member", FIELDS)
def test_assigned_tensor_is_the_struct_s(kind, field, member, after, prec):
    s = _make(kind, prec)
    if after:
        s.struct()
        if kind == "cotangent":
            s.state_struct()
    t = torch.ones_like(getattr(s, field))
    setattr(s, field, t)
    assert getattr(s, field) is t
    assert _pointers(s.struct(), member) == _rows(t)
    if kind == "cotangent" and field != "c":
        assert _pointers(s.state_struct(), member) == _rows(t)
    # the other fields stay where they were
    other = "v" if kind != "rates" else "lo"
    if getattr(s, other) is not None:
        assert _pointers(s.struct(), other) == _rows(getattr(s, other))
    q = s.clone()
    u = getattr(q, field)
    assert u.data_ptr() != t.data_ptr() and torch.equal(u, t)
    assert _pointers(q.struct(), member) == _rows(u)
    assert _pointers(s.struct(), member) == _rows(t)


def test_fields_that_are_absent():
    r = Rates(N, 1, False, "cpu")           # no velocity gradient
    assert not any(r.struct().Lhi)
    r.Lhi = torch.zeros(9, N)
    assert _pointers(r.struct(), "Lhi") == _rows(r.Lhi)
    c = Cotangent(N, 0, "cpu", True)
    assert all(c.struct().S)
    c.S = None
    assert not any(c.struct().S) and not any(c.state_struct().S)
    p = Particles(N, 0, False, "cpu")       # a fluid: its stress is not part of the struct
    p.S = torch.zeros(6, N, dtype=torch.float64)
    assert not any(p.struct().S)


def test_in_place_operators_keep_the_buffer():
    c = Cotangent(N, 0, "cpu")
    at = _pointers(c.struct(), "x")
    c.x += 2.0
    assert _pointers(c.struct(), "x") == at and (c.clone().x == 2.0).all()
    d = Cotangent(N, 0, "cpu")
    d.copy_from(c)
    assert (d.x == 2.0).all()
    c.v = torch.full_like(c.v, 5.0)
    d.copy_from(c)
    assert (d.v == 5.0).all()


def test_copies_of_a_set_that_was_used():
    """deepcopy and serialisation give a set with its own memory."""
    c = Cotangent(N, 0, "cpu", True)
    c.x.fill_(3.0)
    c.struct(), c.state_struct()
    shallow = copy.copy(c)
    shallow.v = torch.zeros_like(c.v)
    assert _pointers(c.struct(), "v") == _rows(c.v)
    buf = io.BytesIO()
    torch.save(c, buf)
    buf.seek(0)
    for q in (copy.deepcopy(c), torch.load(buf, weights_only=False)):
        assert torch.equal(q.x, c.x) and q.x.data_ptr() != c.x.data_ptr()
        q.x.fill_(4.0)
        assert _pointers(q.struct(), "x") == _rows(q.x)
        assert (q.clone().x == 4.0).all() and (c.x == 3.0).all()
