"""The two-step sweeps of untuned calls against the one-step ones: forward-only
calls, illumination, captured series and the gradient, with tiles that the
wavefield has not reached yet left out, records of odd and even lengths, and
snapshot restarts on either step of a reverse launch (odd spacings).

A sponge wider than the LDS-resident sweeps hold makes untuned calls take the
two-step sweeps at a small size.  Both forms make the same operations in the
same order per cell: same bits.  The extended image adds its windows of 64
instead of 32 steps (FP32): a few roundings of its largest partial sums,
1e-5 relative L2 allows for 16 windows' worth.
"""
import numpy as np
import pytest

from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid, gaussian_anomaly, random_traces, ricker

from helpers import rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ONE_STEP = dict(tile_rows=16, graph_steps=-1)


def problem(nts, nx=301, nz=58, N=130):
    ns, nt = len(nts), max(nts)
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 20.0, iz0=nz // 2, ix0=nx // 3)
    rec = [(1, x) for x in range(0, nx, 2)] + [(z, nx - 1) for z in range(2, nz, 3)]
    iz = np.array([r[0] for r in rec] * ns, np.int32)
    ix = np.array([r[1] for r in rec] * ns, np.int32)
    six = np.linspace(3, nx - 1, ns).astype(np.int32)
    geom = Geometry(np.full(ns, 2, np.int32), six, np.arange(ns + 1, dtype=np.int32) * len(rec), iz, ix,
                    np.array(nts, np.int32))
    return grid, geom, v, ricker(14.0, 1e-3, nt).astype(np.float32)


@pytest.mark.parametrize("nts", [(120, 119, 64), (2, 3), (230,), (145, 50, 99, 101, 10)])
def test_untuned_two_step_calls_have_the_one_step_bits(nts):
    grid, geom, v, wav = problem(nts)
    q = B.fwi_exec_query(grid, geom, None, B.WS_GRADIENT)
    assert (q["forward_steps"], q["reverse_steps"]) == (2, 2)
    d = random_traces(geom, grid.nt_max, seed=8, scale=1e-2)

    def calls(ex):
        return {"forward": (B.forward(v, wav, grid, geom, ex),),
                "misfit": (B.misfit_value(v, wav, grid, geom, d, "l2", ex),),
                "hessian": (B.hessian_diag(v, wav, grid, geom, B.HESS_OFFSET, hmax=2, exec_=ex),),
                "gradient": B.gradient(v, wav, grid, geom, d, "l2", ex, hmax=2),
                "image": B.extended_image(v, wav, grid, geom, d, 2, "l2", ex)}
    a, b = calls(None), calls(B.make_exec(**ONE_STEP))
    for name in a:
        for k, (x, y) in enumerate(zip(a[name], b[name])):
            assert bool(torch.isfinite(x).all())
            if name == "image" and k == 2:
                if float(y.abs().max()) > 0:
                    assert rel(x.cpu().numpy(), y.cpu().numpy()) < 1e-5
            else:
                assert torch.equal(x, y), (name, k)


def test_untuned_two_step_capture_has_the_one_step_bits():
    grid, geom, v, wav = problem((150, 150))
    small = geom.subset([0, 1])
    keep = np.arange(0, small.rec_ptr[1], 40)
    geom = Geometry(small.src_iz, small.src_ix, np.array([0, len(keep), 2 * len(keep)], np.int32),
                    np.tile(small.rec_iz[keep], 2), np.tile(small.rec_ix[keep], 2), small.nt)
    a = B.offset_diag_exact(v, wav, grid, geom, 3, 60.0, B.make_exec(shots_in_flight=64))   # chunks of 128 updates
    b = B.offset_diag_exact(v, wav, grid, geom, 3, 60.0, B.make_exec(shots_in_flight=64, tile_rows=16))
    assert torch.equal(a, b) and float(a.abs().max()) > 0
