"""Several time steps per launch against the single relaxation and transport.

lbmrv_collide followed by lbmrv_transport is the general path: one kernel each,
any grid.  The step call must give the same bits whatever number of steps its
launches fuse, on both sides of every rule that picks a tile (the tolerance is
zero: every node does the same arithmetic and rounds to the storage type at
every step in both).
"""
import numpy as np
import pytest

from paper_1312_3297_amd import workloads
from paper_1312_3297_amd.lbmrv import Lbmrv

from _common import far_state, oracle_lattice, to_storage

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RATES = {"d2q9": workloads.RATES_D2Q9_GROUPED, "d3q19": workloads.RATES_D3Q19, "d3q27": workloads.RATES_D3Q27}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def one_by_one(ctx, f, mode, field, nsteps):
    """nsteps single relaxations and transports; the states after each."""
    out, f = [], f.clone()
    for _ in range(nsteps):
        g = torch.empty_like(f)
        ctx.collide(f, g, mode, 0.7, field)
        ctx.transport(g, f)
        out.append(f.clone())
    return out


def compare(lattice, shape, storage, mode, steps, basis="default", equilibrium="polynomial", rates=None,
            streaming=("pull", "push"), order="auto"):
    print("%s %s %s %s %s steps %s" % (lattice, shape, storage, mode, basis if isinstance(basis, str) else "run-time",
                                      steps), flush=True)
    lat = oracle_lattice(lattice, basis if basis == "geier" else "default")
    st, _ = to_storage(lat, far_state(lat, shape, seed=41, amp=0.02, umax=0.08), storage)
    f0 = torch.from_numpy(st).cuda()
    field = None
    if mode == "field":
        rng = np.random.default_rng(42)
        field = torch.from_numpy(rng.uniform(-0.1, 0.1, (lat.d,) + shape).astype(np.float32)).cuda()
    ctx = Lbmrv(lattice, rates or RATES[lattice], tuple(reversed(shape)), storage, basis)
    ctx.set_equilibrium(equilibrium)
    ctx.set_block_order(order)
    want = one_by_one(ctx, f0, mode, field, max(steps))
    for kind in streaming:
        ctx.set_streaming(kind)
        for n in steps:
            a, b = f0.clone(), torch.full_like(f0, float("nan"))
            ctx.step(a, b, mode, 0.7, field, n)
            torch.cuda.synchronize()
            bits = torch.int16 if storage == "f16dev" else torch.int64 if storage == "f64" else torch.int32
            assert torch.equal(b.view(bits), want[n - 1].view(bits)), (kind, n)


# 2-D grids (ny, nx): around the smallest tiled extent, tiles of each size and of
# unequal sides, remainders, one round of workgroups and more, thin grids
@pytest.mark.parametrize("shape", [(8, 40), (9, 9), (10, 300), (15, 16), (31, 33), (64, 64), (173, 190), (16, 2049),
                                   (300, 301), (429, 458), (440, 450), (601, 590), (33, 6000), (36, 6001)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f32dev", "f16dev"])
def test_tiles_equal_single_steps(shape, storage):
    compare("d2q9", shape, storage, "fluid", (1, 2, 5, 8, 17), streaming=("pull",))


@pytest.mark.parametrize("basis,mode,equilibrium", [("default", "field", "polynomial"), ("geier", "zero", "polynomial"),
                                                    ("geier", "field", "maxwellian"), ("custom", "fluid", "polynomial"),
                                                    ("custom", "field", "maxwellian")])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_tiles_in_every_mode_and_basis(basis, mode, equilibrium, storage):
    b, rates = (workloads.RAW_D2Q9, workloads.RATES_RAW_D2Q9) if basis == "custom" else (basis, None)
    for shape in ((21, 37), (190, 200), (450, 449), (601, 590)):
        compare("d2q9", shape, storage, mode, (2, 7, 12), b, equilibrium, rates)


# 3-D grids (nz, ny, nx): every tile of the rule (up to 256 workgroups of each),
# extents equal to and one above a tile's, the first grid beyond the tiles, and
# extents too small for any
@pytest.mark.parametrize("lattice", ["d3q19", "d3q27"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("shape", [(4, 4, 4), (5, 6, 7), (8, 8, 9), (3, 17, 20), (24, 25, 26), (17, 30, 33),
                                   (47, 48, 49), (64, 64, 61)])
def test_tiles_in_space_equal_single_steps(lattice, storage, shape):
    compare(lattice, shape, storage, "field" if shape[0] % 2 else "fluid", (2, 3, 4, 7), streaming=("pull",))


# two steps per launch on 3-D grids: chunks of one plane count and with a short
# last one, tiles of each number of rows (FP32: 20 with 257 rows), tiles that
# divide an extent and that leave a remainder, few planes; the last of each list
# is below the bound on idle columns (single steps)
PAIRS = {"d3q19": [(70, 64, 64), (5, 161, 193), (131, 31, 64), (16, 97, 128), (8, 257, 250), (301, 17, 33)],
         "d3q27": [(80, 80, 81), (101, 77, 66), (7, 305, 257), (8, 257, 250), (900, 24, 28)]}


@pytest.mark.parametrize("lattice", ["d3q19", "d3q27"])
@pytest.mark.parametrize("storage,mode", [("f64", "field"), ("f32", "fluid"), ("f32dev", "zero")])
def test_pairs_equal_single_steps(lattice, storage, mode):
    for shape in PAIRS[lattice]:
        compare(lattice, shape, storage, mode, (2, 3, 4, 5, 8), streaming=("pull",))


@pytest.mark.parametrize("lattice,storage,shape", [("d3q19", "f32", (40, 64, 64)), ("d3q19", "f64", (6, 9, 20)),
                                                   ("d3q27", "f32", (80, 80, 81)), ("d3q27", "f64", (9, 8, 10))])
def test_run_time_bases_in_space(lattice, storage, shape):
    basis, rates = {"d3q19": (workloads.RAW2_D3Q19, workloads.RATES_RAW2_D3Q19),
                    "d3q27": (workloads.HERMITE_D3Q27, workloads.RATES_HERMITE_D3Q27)}[lattice]
    compare(lattice, shape, storage, "fluid", (2, 5), basis, "maxwellian", rates, streaming=("push",))


@pytest.mark.parametrize("order", ["natural", "xcd"])
@pytest.mark.parametrize("lattice,shape", [("d2q9", (70, 95)), ("d3q19", (20, 21, 40)), ("d3q19", (70, 64, 64))])
def test_every_block_order(lattice, shape, order):
    compare(lattice, shape, "f32", "fluid", (9,), order=order)


@pytest.mark.parametrize("lattice", ["d2q9", "d3q19", "d3q27"])
@pytest.mark.parametrize("storage", ["f64", "f32dev", "f16dev"])
def test_one_step_is_the_relaxation_and_the_transport(lattice, storage):
    compare(lattice, (7, 70) if lattice == "d2q9" else (3, 5, 70), storage, "fluid", (1,))


@pytest.mark.parametrize("shape", [(4, 8, 8), (2, 3, 43), (1, 1, 257), (5, 1, 51), (3, 2, 171)])
@pytest.mark.parametrize("mode", ["fluid", "field"])
def test_reverse_step_over_whole_rows(shape, mode):
    """The reverse step's workgroups take 256 consecutive nodes whatever the
    rows: one full workgroup, one or two nodes in the last one, rows longer and
    shorter than a workgroup, against the FP64 adjoint oracle (1e-10 normwise:
    both sides FP64, different order of operations over a few steps)."""
    from oracle import adjoint as E
    lat = oracle_lattice("d3q19")
    rng = np.random.default_rng(43)
    f0 = far_state(lat, shape, seed=44, amp=0.02, umax=0.05)
    field = rng.uniform(-0.1, 0.1, (3,) + shape).astype(np.float32).astype(np.float64) if mode == "field" else None
    cot = rng.standard_normal(f0.shape)
    _, gf, gs, gu = E.vjp(lat, f0, RATES["d3q19"], 3, cot, field=field, alpha=0.9 if mode == "fluid" else None)
    ctx = Lbmrv("d3q19", RATES["d3q19"], tuple(reversed(shape)), "f64")
    gpu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    _, gfg, gsg, gug = ctx.adjoint(gpu(f0), gpu(cot), 3, 2, mode, None if field is None else gpu(field.astype(np.float32)),
                                   alpha=0.9)
    torch.cuda.synchronize()
    for got, ref in ((gfg, gf), (gsg, gs)) + (((gug, gu),) if mode == "field" else ()):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("shape", [(200, 1), (37, 2), (5, 3), (2, 65), (17, 66), (8, 127)])
def test_reverse_pairs_on_narrow_grids(shape):
    """Two reverse steps per launch where the two-node halo wraps several times
    in x or the last tile holds one or two columns: dJ/df0 and dJ/du~ bit for
    bit those of single steps (K = 1), dJ/ds to the order of FP64 sums."""
    lat = oracle_lattice("d2q9")
    rng = np.random.default_rng(48)
    st, _ = to_storage(lat, far_state(lat, shape, seed=49, amp=0.02, umax=0.05), "f32")
    ctx = Lbmrv("d2q9", RATES["d2q9"], tuple(reversed(shape)), "f32")
    gpu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    cot = gpu(rng.standard_normal((9,) + shape).astype(np.float32))
    field = gpu(rng.uniform(-0.1, 0.1, (2,) + shape).astype(np.float32))
    single, paired = (ctx.adjoint(gpu(st), cot, 7, K, "field", field) for K in (1, 7))
    torch.cuda.synchronize()
    assert torch.equal(single[1], paired[1]) and torch.equal(single[3], paired[3])
    assert torch.allclose(single[2], paired[2], rtol=1e-13, atol=1e-13 * float(single[2].abs().max()))


@pytest.mark.parametrize("shape", [(2049, 2050), (1, 2 ** 22 + 1)])
def test_reverse_pairs_on_large_grids(shape):
    """The first grids beyond 2^22 nodes, in two-step launches again: bit for bit
    single steps, as on narrow grids."""
    test_reverse_pairs_on_narrow_grids(shape)


@pytest.mark.parametrize("lattice,shape", [("d2q9", (1, 1)), ("d2q9", (1, 7)), ("d2q9", (16, 32)), ("d2q9", (19, 27)),
                                           ("d3q19", (1, 2, 3)), ("d3q19", (8, 8, 8)), ("d3q27", (7, 8, 9))])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_small_grids_in_one_workgroup(lattice, shape, storage):
    """Grids of up to 512 nodes (and the first beyond) run whole in one
    workgroup, in place as well as between two arrays."""
    for mode in ("fluid", "field"):
        compare(lattice, shape, storage, mode, (1, 2, 7), streaming=("pull", "push", "aa"))
    lat = oracle_lattice(lattice)
    st, _ = to_storage(lat, far_state(lat, shape, seed=46, amp=0.02, umax=0.05), storage)
    f = torch.from_numpy(st).cuda()
    ctx = Lbmrv(lattice, RATES[lattice], tuple(reversed(shape)), storage)
    ctx.set_streaming("aa")
    for n in (1, 2, 5):
        g = f.clone()
        ctx.step(g, g, "fluid", 0.7, None, n)
        torch.cuda.synchronize()
        assert torch.equal(g, one_by_one(ctx, f, "fluid", None, n)[-1]), n


def test_more_steps_than_one_launch_takes():
    compare("d2q9", (3, 5), "f64", "fluid", (4096, 4097), streaming=("pull",))


# walls on both faces of an axis (moving ones among them); a wall on one face, a z
# wall and other storages keep single steps
@pytest.mark.parametrize("lattice,shape", [("d3q19", (70, 64, 64)), ("d3q19", (16, 97, 257)), ("d3q27", (80, 80, 81))])
@pytest.mark.parametrize("mask", [0b1100, 0b0100, 0b1111, 0b0010, 0b101100])
def test_pairs_with_walls_equal_single_steps(lattice, shape, mask):
    lat = oracle_lattice(lattice)
    storage = "f32dev" if mask & 1 else "f32"
    st, _ = to_storage(lat, far_state(lat, shape, seed=45, amp=0.02, umax=0.05), storage)
    f0 = torch.from_numpy(st).cuda()
    ctx = Lbmrv(lattice, RATES[lattice], tuple(reversed(shape)), storage)
    ctx.set_walls(mask, [[0.0, 0.03, 0.0], [0.0, 0.0, 0.01], [0.02, 0.0, 0.0], [0.05, 0.0, 0.01]] + [[0.0] * 3] * 2, 1.1)
    f = f0.clone()
    for n in range(1, 7):
        g = torch.empty_like(f)
        ctx.collide(f, g, "fluid", 0.7)
        ctx.transport(g, f)
        if n in (2, 3, 5, 6):
            a, b = f0.clone(), torch.full_like(f0, float("nan"))
            ctx.step(a, b, "fluid", 0.7, None, n)
            torch.cuda.synchronize()
            assert torch.equal(b, f), n


@pytest.mark.parametrize("shape", [(1, 1), (32, 64), (3, 683), (257, 255), (513, 512)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_sums_at_the_edges_of_their_rows(shape, storage):
    """One workgroup up to 2048 nodes, a row per 256 nodes, 1024 rows at most.
    Each sum is a chain of at most some 600 FP64 additions of terms up to
    |f|: 1e-13 of the sum of magnitudes."""
    lat = oracle_lattice("d2q9")
    st, f64 = to_storage(lat, far_state(lat, shape, seed=47, amp=0.02, umax=0.05), storage)
    f = torch.from_numpy(st).cuda()
    ctx = Lbmrv("d2q9", RATES["d2q9"], tuple(reversed(shape)), storage)
    mass, mom, finite = ctx.conservation(f)
    tol = 1e-13 * np.abs(f64).sum()
    assert finite and abs(mass - f64.sum()) <= tol
    for a in range(2):
        assert abs(mom[a] - np.tensordot(lat.c[:, a].astype(float), f64, axes=(0, 0)).sum()) <= tol
    ref = np.linspace(0.1, 0.2, 9)
    d2 = ((f64 - ref.reshape(9, 1, 1)) ** 2).sum()
    norm2, finite = ctx.deviation_norm2(f, ref)
    assert finite and abs(norm2 - d2) <= 1e-12 * d2   # the stored reference is rounded once more
    out = torch.zeros(5, dtype=torch.float64, device="cuda")
    flat = f.view(-1)
    flat[0], flat[-1] = float("inf"), float("nan")
    ctx.conservation_noalloc(f, out)
    assert out[4].item() == 2.0
    assert not ctx.conservation(f)[2] and not ctx.deviation_norm2(f, ref)[1]
