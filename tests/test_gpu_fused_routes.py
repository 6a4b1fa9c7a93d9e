"""The kernels of several steps per launch on grids that are known to take them
(_plans.FUSED, held to their routes here and in a CPU test), against single
relaxations and transports, and the adjoint whose forward and recomputed states
they make, against one step per segment (K = 1).  Bit for bit: every node does
the same arithmetic and rounds to the storage type at every step.  Only dJ/ds
sums its rows in another order where reverse steps are paired: FP64 sums of N
terms of random sign differ by about 2^-53 sqrt(N) of the result, 5e-13 for the
largest N here, so 1e-12."""
import numpy as np
import pytest

from paper_1312_3297_amd import workloads
from paper_1312_3297_amd.lbmrv import Lbmrv

from _common import far_state, oracle_lattice, to_storage
from _plans import FUSED, is_route, route
from test_gpu_multistep import RATES, compare

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("lattice,storage,shape,want", FUSED)
def test_fused_steps_equal_single_steps(lattice, storage, shape, want):
    assert is_route(lattice, storage, shape, want)
    compare(lattice, shape, storage, ("field", "fluid", "zero")[sum(shape) % 3], (2, 3, 4, 5, 8), streaming=("pull",))


# kept states: rows of whole sectors; the first grids of each kernel's range
@pytest.mark.parametrize("lattice,storage,shape,kind,basis", [
    ("d3q19", "f32", (72, 64, 64), "slide", "default"), ("d3q19", "f64", (50, 64, 64), "slide", "default"),
    ("d3q27", "f32", (80, 80, 96), "slide", "default"), ("d3q27", "f64", (110, 101, 96), "slide", "default"),
    ("d3q19", "f32", (48, 48, 48), "tile", "default"), ("d3q19", "f16dev", (32, 32, 32), "tile", "default"),
    ("d3q27", "f32", (20, 20, 20), "tile", "default"), ("d2q9", "f32", (513, 1024), "tile", "default"),
    ("d2q9", "f16dev", (700, 768), "tile", "default"), ("d2q9", "f64", (520, 512), "tile", "default"),
    ("d2q9", "f32", (2049, 2048), "tile", "geier"), ("d3q19", "f32", (70, 64, 64), "single", "custom")])
def test_adjoint_over_fused_states_equals_single_steps(lattice, storage, shape, kind, basis):
    print("%s %s %s %s" % (lattice, shape, storage, basis), flush=True)
    if basis != "custom":
        assert route(lattice, storage, shape, basis)[0] == kind
    lat = oracle_lattice(lattice, "geier" if basis == "geier" else "default")
    rng = np.random.default_rng(71)
    st, _ = to_storage(lat, far_state(lat, shape, seed=72, amp=0.02, umax=0.05), storage)
    b, s = (workloads.RAW2_D3Q19, workloads.RATES_RAW2_D3Q19) if basis == "custom" else (basis, RATES[lattice])
    ctx = Lbmrv(lattice, s, tuple(reversed(shape)), storage, b)
    f0 = torch.from_numpy(st).cuda()
    cot = torch.from_numpy(rng.standard_normal((lat.q,) + shape).astype(np.float32)).to("cuda", ctx.compute_dtype)
    field = torch.from_numpy(rng.uniform(-0.1, 0.1, (lat.d,) + shape).astype(np.float32)).cuda()
    for mode, n in (("field", 7), ("fluid", 6)):
        args = (mode, field if mode == "field" else None, True)
        one = ctx.adjoint(f0, cot, n, 1, *args, alpha=0.9)
        # one segment (kept states only), two and three, of odd and even counts
        for K in (n, 5, 4, 3, 2):
            got = ctx.adjoint(f0, cot, n, K, *args, alpha=0.9)
            torch.cuda.synchronize()
            for i in (0, 1, 3):
                assert one[i] is None or torch.equal(one[i], got[i]), (mode, K, i)
            assert torch.allclose(one[2], got[2], rtol=1e-12, atol=1e-12 * float(one[2].abs().max())), (mode, K)
