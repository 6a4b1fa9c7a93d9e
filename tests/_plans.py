"""The plans that lbmrv_create makes for the kernels of several steps per launch,
read from the built library (host code, no GPU): which kernel a grid takes
without walls, and with what tile."""
import ctypes

from paper_1312_3297_amd import lbmrv

NAME = {("d2q9", "default"): "d2q9_paper", ("d2q9", "geier"): "d2q9_geier", ("d3q19", "default"): "d3q19",
        ("d3q27", "default"): "d3q27"}
KIND = {"f64": "f64", "f32": "f32", "f32dev": "f32", "f16dev": "f16"}


class TilePlan(ctypes.Structure):
    _fields_ = [("t", ctypes.c_uint32 * 3), ("steps", ctypes.c_uint32), ("threads", ctypes.c_uint32)]


class SlidePlan(ctypes.Structure):
    _fields_ = [("t", ctypes.c_uint32 * 2), ("chunk", ctypes.c_uint32), ("threads", ctypes.c_uint32)]


def _call(which, struct, lattice, storage, shape, basis):
    name = "%s_%s_%s" % (which, NAME[lattice, basis], KIND[storage])
    fn = getattr(lbmrv.library(), "_ZN5lbmrv%d%sEjjj" % (len(name), name))
    fn.restype, fn.argtypes = struct, [ctypes.c_uint32] * 3
    return fn(*(tuple(reversed(shape)) + (1,))[:3])


def route(lattice, storage, shape, basis="default"):
    """("closed",), ("tile", (tx, ty, tz), steps), ("slide", (tx, ty), planes) or
    ("single",) for a grid of the array shape (nz, ny, nx) or (ny, nx)."""
    n = 1
    for e in shape:
        n *= e
    if n <= 512:
        return ("closed",)
    t = _call("plan_tile", TilePlan, lattice, storage, shape, basis)
    if t.steps >= 2:
        return ("tile", tuple(t.t), t.steps)
    s = _call("plan_slide", SlidePlan, lattice, storage, shape, basis)
    return ("slide", tuple(s.t), s.chunk) if s.chunk else ("single",)
