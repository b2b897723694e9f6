"""The misfit of a few traces around the edges of its workgroups (16 traces)
and of its tiles (128 samples), and the extended image's fold at widths that
its float4 updates do and do not take.

J is one FP64 sum per trace and a fixed-order sum over traces: against NumPy's
FP64 on the same traces, 1e-12 relative allows for 600 samples' roundings in
another order.  Gradients and images: against the FP64 oracle, relative L2 1e-3;
the image's h = 0 slice against the gradient, same products in another order, 1e-5.
"""
import numpy as np
import pytest

import oracle
from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid, gaussian_anomaly, random_traces, ricker

from helpers import GRAD_TOL, rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def problem(nts, nrecs, nx=45, nz=17):
    nt = max(nts)
    grid = Grid(nz, nx, 10.0, 1e-3, nt, 8, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 20.0, iz0=nz // 2, ix0=nx // 3)
    iz = np.concatenate([np.full(n, 1 + i, np.int32) for i, n in enumerate(nrecs)])
    ix = np.concatenate([np.arange(n, dtype=np.int32) % nx for n in nrecs])
    ptr = np.concatenate([[0], np.cumsum(nrecs)]).astype(np.int32)
    six = np.linspace(3, nx - 4, len(nts)).astype(np.int32)
    geom = Geometry(np.full(len(nts), nz // 2, np.int32), six, ptr, iz, ix, np.array(nts, np.int32))
    return grid, geom, v, ricker(25.0, 1e-3, nt).astype(np.float32)


@pytest.mark.parametrize("nts,nrecs", [((127, 128, 129), (1, 15, 16)), ((2, 257, 256), (17, 33, 32)), ((600,), (45,))])
@pytest.mark.parametrize("kind", ["l2", "int"])
def test_misfit_tiles(nts, nrecs, kind):
    grid, geom, v, wav = problem(nts, nrecs)
    d = random_traces(geom, grid.nt_max, seed=3, scale=1e-2)
    syn = B.forward(v, wav, grid, geom).cpu().numpy().astype(np.float64)
    J = 0.0
    for s, nt in enumerate(nts):
        for tr in range(geom.rec_ptr[s], geom.rec_ptr[s + 1]):
            r = syn[tr, :nt] - d[tr, :nt].astype(np.float64)
            r[0] = -float(d[tr, 0])
            J += 0.5 * np.sum((grid.dt * np.cumsum(r) if kind == "int" else r) ** 2)
    got = float(B.misfit_value(v, wav, grid, geom, d, kind))
    assert abs(got - J) <= 1e-12 * J
    Jg, g = B.gradient(v, wav, grid, geom, d, kind)[:2]
    assert float(Jg) == got
    ref = oracle.gradient(v, grid, geom, wav, d, kind)
    assert rel(g.cpu().numpy(), ref[1]) < GRAD_TOL


@pytest.mark.parametrize("nx", [45, 47, 60, 258])
@pytest.mark.parametrize("hmax", [3, 8, 16])
def test_fold_widths(nx, hmax):
    grid, geom, v, wav = problem((140, 90, 33), (20, 31, 9), nx=nx)
    d = random_traces(geom, grid.nt_max, seed=4, scale=1e-2)
    _, ref = oracle.extended_image(v, grid, geom, wav, d, "l2", hmax)
    _, g, image = B.extended_image(v, wav, grid, geom, d, hmax, "l2")
    image = image.cpu().numpy()
    for h in range(2 * hmax + 1):
        assert rel(image[h], ref[h]) < GRAD_TOL, h - hmax
    assert rel(image[hmax], g.cpu().numpy()) < 1e-5
