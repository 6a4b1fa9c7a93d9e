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


# Grids (nz, ny, nx) that take a kernel of several steps per launch, with what
# each is there for; the GPU tests compare them with single steps, the CPU test
# holds every one to the route it names.
FUSED = [
    # two steps per launch: few planes, a short last chunk, tiles that divide the
    # extents and that leave a remainder in x, y and z, rows of each number
    ("d3q19", "f32", (5, 230, 232), "slide"), ("d3q19", "f32", (131, 45, 64), "slide"),
    ("d3q19", "f32", (70, 64, 64), "slide"), ("d3q19", "f32", (67, 65, 63), "slide"),
    ("d3q19", "f32", (16, 171, 128), "slide"), ("d3q19", "f64", (5, 161, 193), "slide"),
    ("d3q19", "f64", (70, 64, 64), "slide"), ("d3q19", "f64", (49, 53, 57), "slide"),
    ("d3q27", "f32", (101, 77, 90), "slide"), ("d3q27", "f32", (7, 305, 257), "slide"),
    ("d3q27", "f32", (80, 80, 81), "slide"), ("d3q27", "f64", (102, 101, 103), "slide"),
    ("d3q27", "f64", (4, 513, 520), "slide"), ("d3q27", "f64", (104, 104, 98), "slide"),
    # the larger tiles in space: 12 x 6 x 6 and 16 x 8 x 8
    ("d3q19", "f32", (48, 48, 48), "tile 12 6 6"), ("d3q19", "f32", (47, 46, 48), "tile 12 6 6"),
    ("d3q19", "f64", (48, 48, 48), "tile 12 6 6"), ("d3q19", "f64", (42, 41, 47), "tile 12 6 6"),
    ("d3q19", "f16dev", (48, 48, 48), "tile 12 6 6"), ("d3q19", "f16dev", (47, 46, 48), "tile 12 6 6"),
    ("d3q19", "f32", (64, 64, 61), "tile 16 8 8"), ("d3q19", "f32", (59, 62, 63), "tile 16 8 8"),
]


def is_route(lattice, storage, shape, want):
    """Whether a grid's plan is the kernel (and the tile of at most the sides) named."""
    r = route(lattice, storage, shape)
    kind, *sides = want.split()
    if r[0] != kind:
        return False
    # equal tiles of at most side nodes: -(-n // -(-n // side))
    return all(t == -(-n // -(-n // int(s))) for t, n, s in zip(r[1], reversed(shape), sides))
