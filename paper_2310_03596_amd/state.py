"""Device particle arrays and ABI struct builders.

PyTorch serves only as the device allocator and stream provider: every
tensor here is raw device memory handed to libsph by pointer.
"""
from __future__ import annotations

import copy
import functools
import math

import numpy as np
import torch

from . import _lib as L


def real_dtype(prec: int):
    return torch.float64 if prec == L.SPH_FP64 else torch.float32


def grid_struct(grid: dict) -> L.SphGrid:
    g = L.SphGrid()
    for d in range(3):
        g.origin[d] = float(grid["origin"][d])
        g.dims[d] = int(grid["dims"][d])
    g.cell = float(grid["cell"])
    return g


def ncells(grid: dict) -> int:
    d = grid["dims"]
    return int(d[0]) * int(d[1]) * int(d[2])


def params_struct(p: dict, prec: int) -> L.SphParams:
    s = L.SphParams()
    for k in ("h", "rho0", "c0", "gamma", "K", "G", "Y0", "H", "beta", "cfl"):
        setattr(s, k, float(p[k]))
    for d in range(3):
        s.gravity[d] = float(p["gravity"][d])
        s.wall_lo[d] = float(p["wall_lo"][d])
        s.wall_hi[d] = float(p["wall_hi"][d])
    s.wall_mask = int(p["wall_mask"])
    s.material = int(p["material"])
    s.prec = int(prec)
    s.eos = int(p.get("eos", L.SPH_EOS_LINEAR))
    for k in ("mg_s", "mg_gamma0", "p_cut"):
        setattr(s, k, float(p.get(k, 0.0)))
    return s


def _ptr(t):
    return None if t is None else t.data_ptr()


@functools.lru_cache(maxsize=1024)
def _plan(layout):
    """Where each field of a layout, a tuple of (name, shape or None, dtype),
    lies in one flat byte buffer: {name: (offset, bytes, shape, dtype, bytes
    per entry of the first axis)} with 256-byte aligned offsets (None where
    the shape is None), and the buffer's size."""
    out, off = {}, 0
    for name, shape, dt in layout:
        if shape is None:
            out[name] = None
            continue
        nbytes = math.prod(shape) * dt.itemsize
        out[name] = (off, nbytes, shape, dt, math.prod(shape[1:]) * dt.itemsize)
        off += (nbytes + 255) & ~255
    return out, max(off, 256)


class _Flat:
    """Fields that live in one device allocation, so that a copy of the whole
    set (checkpoints, saved states of the reverse pass) is one copy.

    A field's tensor is made when it is first asked for, and the ABI structs
    from the buffer's address and the field's place in it: a rollout and its
    reverse pass make dozens of such sets and read only the structs (a
    27,000-particle gradient of ten steps: 5.1 -> 3.6 ms).  A tensor that a
    program assigns to a field takes the place of the buffer's part, in the
    structs too."""

    def _allocate(self, layout, device, zero=True):
        """zero=False leaves the memory uninitialised (no fill kernel), for
        buffers that a call overwrites completely before anything reads them."""
        fields, nbytes = _plan(tuple(layout))
        alloc = torch.zeros if zero else torch.empty
        self._buf = alloc(nbytes, dtype=torch.uint8, device=device)
        self._fields = fields
        self._bind()

    def _bind(self):
        for k in self._fields:
            self.__dict__.pop(k, None)
        self._assigned = frozenset()   # fields whose tensors are the program's own
        self._forget()

    def _forget(self):
        self._struct = None   # the ABI struct, built on first use

    def __getattr__(self, name):
        fields = self.__dict__.get("_fields")
        if fields is None or name not in fields:
            raise AttributeError(f"{type(self).__name__} has no attribute {name!r}")
        at = fields[name]
        t = None if at is None else self._buf[at[0]:at[0] + at[1]].view(at[3]).view(at[2])
        self.__dict__[name] = t
        return t

    def __setattr__(self, name, value):
        field = name in self.__dict__.get("_fields", ())
        if field and value is self.__dict__.get(name, self):   # p.x += t
            return
        self.__dict__[name] = value
        if field:
            self._assigned |= {name}
            self._forget()

    def __getstate__(self):
        """What a copy or a file holds: no struct, whose addresses are this
        set's, and no view of the buffer."""
        state = {k: v for k, v in self.__dict__.items() if k not in self._fields or k in self._assigned}
        state.update((k, None) for k in ("_struct", "_state") if k in state)
        return state

    def _address(self, name):
        """Device address of a field; None if the set has no such field or it is empty."""
        if name in self._assigned:
            t = self.__dict__[name]
            return None if t is None or t.numel() == 0 else t.data_ptr()
        at = self._fields[name]
        return None if at is None or at[1] == 0 else self._buf.data_ptr() + at[0]

    def _addresses(self, name, count):
        """Device addresses of the first `count` entries of a field's first
        axis; none if the set has no such field or it is empty."""
        base = self._address(name)
        if base is None:
            return ()
        if name in self._assigned:
            t = self.__dict__[name]
            return [t[k].data_ptr() for k in range(count)]
        step = self._fields[name][4]
        return range(base, base + count * step, step)

    def _point(self, struct, arrays, scalars):
        """Point a struct's members at the fields: arrays by their common
        name, scalars as (member, field)."""
        for name in arrays:
            to = getattr(struct, name)
            for k, ptr in enumerate(self._addresses(name, len(to))):
                to[k] = ptr
        for member, name in scalars:
            setattr(struct, member, self._address(name))

    def clone(self):
        """A copy with its own storage (one device copy)."""
        q = copy.copy(self)
        q._buf = self._buf.clone()
        q._bind()
        for name in self._assigned:
            t = self.__dict__[name]
            setattr(q, name, None if t is None else t.clone())
        return q

    def copy_from(self, other):
        """Overwrite every field with other's (same sizes; one device copy)."""
        if not (self._assigned or other._assigned):
            self._buf.copy_(other._buf)
            return
        for name in self._fields:
            to = getattr(self, name)
            if to is not None:
                to.copy_(getattr(other, name))


class Particles(_Flat):
    """One particle array in SoA form on the device."""

    REAL = ("m", "w", "rho", "p", "c", "e")

    def __init__(self, n: int, prec: int, solid: bool, device="cuda", zero: bool = True):
        real = real_dtype(prec)
        self.n, self.prec, self.solid, self.device = n, prec, solid, device
        split = prec == L.SPH_FP32_SPLIT
        layout = [("x", (3, n), torch.float64), ("off", (3, n) if split else None, torch.float32),
                  ("hash", (n,), torch.int32), ("id", (n,), torch.int32), ("v", (3, n), real)]
        layout += [(f, (n,), real) for f in self.REAL]
        layout += [("E", (n,), torch.float64), ("S", (6, n) if solid else None, real),
                   ("ep", (n,) if solid else None, real)]
        self._allocate(layout, device, zero)

    STRUCT = (("hash", "hash"), ("id", "id"), ("m", "m"), ("omega", "w"), ("rho", "rho"), ("p", "p"), ("c", "c"),
              ("e", "e"), ("E", "E"))

    def struct(self) -> L.SphParticles:
        """The ABI struct of this array (kept: the buffers never move)."""
        if self._struct is None:
            self._struct = self._make_struct()
        return self._struct

    def _make_struct(self) -> L.SphParticles:
        s = L.SphParticles()
        s.n = self.n
        s.prec = self.prec
        if self.n == 0:
            return s
        self._point(s, ("x", "off", "v"), self.STRUCT)
        if self.solid:
            self._point(s, ("S",), (("eps_p", "ep"),))
        return s

    @classmethod
    def upload(cls, wl, prec: int, device="cuda") -> "Particles":
        p = cls(wl.n, prec, wl.S is not None, device)
        real = real_dtype(prec)
        p.x.copy_(torch.from_numpy(np.ascontiguousarray(wl.x.T)))
        p.v.copy_(torch.from_numpy(np.ascontiguousarray(wl.v.T)).to(real))
        p.m.copy_(torch.from_numpy(wl.m).to(real))
        p.w.copy_(torch.from_numpy(wl.omega).to(real))
        p.rho.copy_(torch.from_numpy(wl.rho).to(real))
        p.E.copy_(torch.from_numpy(wl.E))
        p.id.copy_(torch.from_numpy(wl.id.astype(np.int64)).to(torch.int32))
        if wl.S is not None:
            p.S.copy_(torch.from_numpy(np.ascontiguousarray(wl.S.T)).to(real))
            p.ep.copy_(torch.from_numpy(wl.eps_p).to(real))
        return p

    def host(self) -> dict:
        """Copy every field to host numpy arrays (array order, positions (n,3))."""
        out = {"x": self.x.T.cpu().numpy().copy(), "v": self.v.T.double().cpu().numpy().copy(),
               "hash": self.hash.cpu().numpy().view(np.uint32).copy(),
               "id": self.id.cpu().numpy().view(np.uint32).copy(), "E": self.E.cpu().numpy().copy()}
        for f in self.REAL:
            out[f] = getattr(self, f).double().cpu().numpy().copy()
        if self.off is not None:
            out["off"] = self.off.T.double().cpu().numpy().copy()
        if self.solid:
            out["S"] = self.S.T.double().cpu().numpy().copy()
            out["ep"] = self.ep.double().cpu().numpy().copy()
        return out


class Rates(_Flat):
    """Pair-sum outputs: FORCE rates and, for solids, the velocity gradient."""

    def __init__(self, n: int, prec: int, gradient: bool, device="cuda", zero: bool = True):
        real = real_dtype(prec)
        split = prec == L.SPH_FP32_SPLIT
        self._allocate([("hi", (6, n), real), ("lo", (6, n) if split else None, real),
                        ("Lhi", (9, n) if gradient else None, real),
                        ("Llo", (9, n) if (gradient and split) else None, real)], device, zero)

    def struct(self) -> L.SphRates:
        if self._struct is None:
            self._struct = self._make_struct()
        return self._struct

    def _make_struct(self) -> L.SphRates:
        r = L.SphRates()
        self._point(r, ("hi", "lo", "Lhi", "Llo"), ())
        return r

    def force(self) -> torch.Tensor:
        """(6, n) rate sums as float64 (hi + lo)."""
        f = self.hi.double()
        return f + self.lo.double() if self.lo is not None else f

    def grad(self) -> torch.Tensor:
        f = self.Lhi.double()
        return f + self.Llo.double() if self.Llo is not None else f


def cells_struct(start: torch.Tensor, nc: int) -> L.SphCells:
    c = L.SphCells()
    c.start = start.data_ptr()
    c.ncells = nc
    return c


def stream_handle() -> int:
    return torch.cuda.current_stream().cuda_stream
