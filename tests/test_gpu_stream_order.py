"""lbmrv_adjoint right behind the work that makes its inputs: f0 and u~ are
written by kernels still queued on the same stream, and two calls share one
workspace without a synchronisation in between.  In two segments (K < N <= 2 K)
the first one is recomputed on the context's own stream from the call's start,
in three also from a snapshot.  K = N uses one stream only; f_N, dJ/df0 and
dJ/du~ do not depend on K (bit for bit), dJ/ds to the order of FP64 sums."""
import numpy as np
import pytest

from paper_1312_3297_amd import workloads
from paper_1312_3297_amd.lbmrv import Lbmrv

from _common import far_state, oracle_lattice, to_storage

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RATES = {"d2q9": workloads.RATES_D2Q9_GROUPED, "d3q19": workloads.RATES_D3Q19}


@pytest.mark.parametrize("lattice,shape,storage", [("d2q9", (300, 310), "f32"), ("d2q9", (16, 20), "f64"),
                                                   ("d3q19", (40, 30, 32), "f32")])
@pytest.mark.parametrize("nsteps,K", [(12, 11), (12, 6), (13, 5)])
def test_adjoint_follows_the_work_that_makes_its_inputs(lattice, shape, storage, nsteps, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lat = oracle_lattice(lattice)
    rng = np.random.default_rng(61)
    st, _ = to_storage(lat, far_state(lat, shape, seed=62, amp=0.02, umax=0.05), storage)
    start = torch.from_numpy(st).cuda()
    cdt = torch.float64 if storage == "f64" else torch.float32
    cot = torch.from_numpy(rng.standard_normal((lat.q,) + shape)).to("cuda", cdt)
    fields = torch.from_numpy(rng.uniform(-0.1, 0.1, (2, lat.d) + shape).astype(np.float32)).cuda()
    ctx = Lbmrv(lattice, RATES[lattice], tuple(reversed(shape)), storage)
    f0, tmp, field = torch.zeros_like(start), torch.empty_like(start), torch.zeros_like(fields[0])
    work = torch.zeros(max(ctx.adjoint_workspace_bytes(nsteps, k) for k in (K, nsteps)), dtype=torch.uint8, device="cuda")

    def inputs(i):  # some milliseconds of queued steps end in f0
        tmp.copy_(start)
        ctx.step(tmp, f0, "zero", 1.0, None, 2001 + 2 * i)
        field.copy_(fields[i])

    def call(k):
        return ctx.adjoint(f0, cot, nsteps, k, "field", field, want_fN=True, workspace=work)

    want = []
    for i in (0, 1):
        inputs(i)
        torch.cuda.synchronize()
        want.append(call(nsteps))
        torch.cuda.synchronize()
    got = []
    f0.zero_()
    torch.cuda.synchronize()
    for i in (0, 1):
        inputs(i)
        got.append(call(K))
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        for i in (0, 1, 3):
            assert torch.equal(a[i], b[i]), i
        assert torch.allclose(a[2], b[2], rtol=1e-13, atol=1e-13 * float(a[2].abs().max()))
