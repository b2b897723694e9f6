"""The LDS-resident forward sweep in the shapes of launches of many tiles,
against the one-step z sweeps bit for bit: four rows per thread (over 1024
tiles), the arrival map with captured series, and an LDS-resident forward
sweep followed by the two-step reverse sweep at odd snapshot spacings.
"""
import numpy as np
import pytest

from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid, gaussian_anomaly, random_traces, ricker

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

Z_SWEEP = dict(tile_rows=16, graph_steps=-1)


def problem(nx, nz, N, nts, step):
    ns, nt = len(nts), max(nts)
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, nx / 12, iz0=nz // 2, ix0=nx // 3)
    ix = np.arange(0, nx, step, dtype=np.int32)
    geom = Geometry((5 + 37 * np.arange(ns, dtype=np.int32)) % nz, np.linspace(0, nx - 1, ns).astype(np.int32),
                    np.arange(ns + 1, dtype=np.int32) * len(ix), np.full(ns * len(ix), nz // 2, np.int32),
                    np.tile(ix, ns), np.array(nts, np.int32))
    return grid, geom, v, ricker(25.0, 1e-3, nt).astype(np.float32)


@pytest.mark.parametrize("nts", [(47, 41, 46, 2, 45, 38, 47, 30), (50, 37) * 5])
def test_four_rows_per_thread_and_a_two_step_reverse(nts):
    """601 x 301 cells: 190 tiles a shot, 1.6 to 8 M cells a step."""
    grid, geom, v, wav = problem(601, 301, 12, nts, 7)
    q = B.fwi_exec_query(grid, geom, None, B.WS_GRADIENT)
    assert (q["forward_steps"], q["reverse_steps"]) == (0, 2)    # LDS-resident, two steps
    d = random_traces(geom, grid.nt_max, seed=3, scale=1e-2)

    def calls(ex):
        return {"forward": (B.forward(v, wav, grid, geom, ex),),
                "misfit": (B.misfit_value(v, wav, grid, geom, d, "int", ex),),
                "hessian": (B.hessian_diag(v, wav, grid, geom, B.HESS_EQ1, exec_=ex),),
                "gradient": B.gradient(v, wav, grid, geom, d, "l2", ex, hmax=2),
                "image": B.extended_image(v, wav, grid, geom, d, 2, "l2", ex)}
    a, b = calls(None), calls(B.make_exec(**Z_SWEEP))
    for name in a:
        for k, (x, y) in enumerate(zip(a[name], b[name])):
            assert bool(torch.isfinite(x).all()) and float(x.abs().max()) > 0, (name, k)
            assert torch.equal(x, y), (name, k)


@pytest.mark.parametrize("nx,nz,N,runs,nt", [
    (301, 150, 20, 16, 70),     # 50 tiles a run, two rows per thread
    (601, 301, 12, 8, 45),      # four rows per thread
])
def test_captured_series_with_an_arrival_map(nx, nz, N, runs, nt):
    grid, geom, v, wav = problem(nx, nz, N, (nt,) * runs, nx // runs + 1)
    assert geom.ntrace // geom.nshot == runs
    a = B.offset_diag_exact(v, wav, grid, geom, 2, 60.0, B.make_exec(shots_in_flight=runs))
    b = B.offset_diag_exact(v, wav, grid, geom, 2, 60.0, B.make_exec(shots_in_flight=runs, tile_rows=16))
    assert torch.equal(a, b) and float(a.abs().max()) > 0


@pytest.mark.parametrize("nts", [(120, 119, 64), (145, 50, 99)])
def test_untuned_two_step_image_has_the_one_step_bits(nts):
    """Untuned calls fold the extended image over windows of the same steps
    whatever form runs the reverse sweep."""
    grid, geom, v, wav = problem(301, 58, 130, nts, 4)
    assert B.fwi_exec_query(grid, geom, None, B.WS_EXTIMAGE)["reverse_steps"] == 2
    d = random_traces(geom, grid.nt_max, seed=8, scale=1e-2)
    a = B.extended_image(v, wav, grid, geom, d, 3, "l2")
    b = B.extended_image(v, wav, grid, geom, d, 3, "l2", B.make_exec(**Z_SWEEP))
    assert float(a[2].abs().max()) > 0 and all(torch.equal(x, y) for x, y in zip(a, b))
