"""The ABI structs of particle, rate and cotangent sets name the same memory
as the sets' tensors (CPU tensors: addresses only)."""
import pytest

from paper_2310_03596_amd.adjoint import Cotangent
from paper_2310_03596_amd.state import Particles, Rates


def _same(struct, name, tensor):
    got = getattr(struct, name)
    if tensor is None or tensor.numel() == 0:
        assert not any(got) if hasattr(got, "__len__") else not got, name
    elif hasattr(got, "__len__"):
        assert list(got)[:tensor.shape[0]] == [row.data_ptr() for row in tensor], name
    else:
        assert got == tensor.data_ptr(), name


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("solid", [False, True])
@pytest.mark.parametrize("n", [0, 1, 5, 300])
def test_structs_name_the_tensors(n, solid, prec):
    p = Particles(n, prec, solid, "cpu")
    for q in (p, p.clone()):
        for name, field in (("x", q.x), ("v", q.v), ("off", q.off), ("hash", q.hash), ("id", q.id), ("m", q.m),
                            ("omega", q.w), ("rho", q.rho), ("p", q.p), ("c", q.c), ("e", q.e), ("E", q.E),
                            ("S", q.S), ("eps_p", q.ep)):
            _same(q.struct(), name, field)
    r = Rates(n, prec, solid, "cpu")
    for name in ("hi", "lo", "Lhi", "Llo"):
        _same(r.struct(), name, getattr(r, name))
    c = Cotangent(n, prec, "cpu", solid)
    for name, field in (("x", c.x), ("v", c.v), ("m", c.m), ("omega", c.w), ("E", c.E), ("S", c.S), ("eps_p", c.ep)):
        _same(c.struct(), name, field)
        _same(c.state_struct(), name, field)
    for name, field in (("rho", c.rho), ("p", c.p), ("c", c.c), ("e", c.e)):
        _same(c.struct(), name, field)
        assert not getattr(c.state_struct(), name)
    with pytest.raises(AttributeError):
        p.no_such_field
