"""The LDS-resident sweeps on models a few cells wide or high: the boundary
ring on both sides of the model then lies within reach of one thread's patch
of 4 columns, or of 4 rows where launches of many tiles take that shape.

Same bits as the one-step z sweeps, which index the ring cell by cell.
"""
import numpy as np
import pytest

from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid, gaussian_anomaly, random_traces, ricker

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

Z_SWEEP = dict(tile_rows=16, graph_steps=-1)


def problem(nx, nz, N, ns, nt):
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 3.0, iz0=nz // 2, ix0=nx // 3)
    rec = sorted({(z, x) for z in (0, nz - 1) for x in range(0, nx, max(1, nx // 60))})
    siz = np.arange(ns, dtype=np.int32) % nz
    six = np.linspace(0, nx - 1, ns).astype(np.int32)
    geom = Geometry(siz, six, np.arange(ns + 1, dtype=np.int32) * len(rec),
                    np.array([r[0] for r in rec] * ns, np.int32), np.array([r[1] for r in rec] * ns, np.int32),
                    np.array([nt - s % 3 for s in range(ns)], np.int32))
    return grid, geom, v, ricker(20.0, 1e-3, nt).astype(np.float32)


def calls(grid, geom, v, wav, ex):
    d = random_traces(geom, grid.nt_max, seed=3, scale=1e-2)
    dv = np.random.default_rng(4).standard_normal((grid.nz, grid.nx)).astype(np.float32) * 30.0
    out = {"forward": (B.forward(v, wav, grid, geom, ex),),
           "gradient": B.gradient(v, wav, grid, geom, d, "int", ex, hmax=0),
           "hessian": (B.hessian_diag(v, wav, grid, geom, B.HESS_EQ1, exec_=ex),),
           "born": (B.born(v, wav, grid, geom, dv, ex),),
           "gn": B.gn_hvp(v, wav, grid, geom, dv, "int", ex),
           "image": B.extended_image(v, wav, grid, geom, d, 0, "int", ex)}
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("nx,nz,N,ns,nt", [
    (1, 1, 4, 1, 60), (2, 5, 5, 2, 60), (3, 6, 4, 2, 60), (3, 1, 9, 2, 60), (4, 2, 6, 2, 60),  # one tile
    (3, 60, 7, 2, 50),                                # rows in several tiles
    (410, 1, 4, 26, 40), (410, 2, 5, 26, 40), (410, 3, 6, 26, 40), (410, 4, 7, 26, 40),  # Born: four rows a thread
    (3001, 2, 4, 12, 40), (3001, 4, 5, 12, 40),       # four rows a thread in every forward sweep, but for two rows
])
def test_same_bits_as_the_z_sweeps(nx, nz, N, ns, nt):
    grid, geom, v, wav = problem(nx, nz, N, ns, nt)
    a = calls(grid, geom, v, wav, None)
    b = calls(grid, geom, v, wav, B.make_exec(**Z_SWEEP))
    for name in a:
        for k, (x, y) in enumerate(zip(a[name], b[name])):
            assert (x is None) == (y is None)
            if x is not None:
                assert bool(torch.isfinite(x).all()), (name, k)
                assert torch.equal(x, y), (name, k)
    assert float(a["gradient"][1].abs().max()) > 0 and float(a["born"][0].abs().max()) > 0
