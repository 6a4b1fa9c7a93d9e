"""The kernels of several steps per launch on grids that are known to take them
(_plans.FUSED, held to their routes here and in a CPU test), against single
relaxations and transports, bit for bit."""
import pytest

from _plans import FUSED, is_route
from test_gpu_multistep import compare

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

