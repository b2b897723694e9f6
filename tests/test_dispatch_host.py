"""Host checks of the rules that choose a call's sweeps (no GPU needed)."""
import re

import numpy as np
import pytest

from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid


def problem(nx, nz, N, ns, nrec, nt=64, fs=False):
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0, fs)
    iz, ix = np.divmod(np.arange(nrec, dtype=np.int32), nx)
    geom = Geometry(np.zeros(ns, np.int32), (np.arange(ns, dtype=np.int32) * 7) % nx,
                    np.arange(ns + 1, dtype=np.int32) * nrec, np.tile(iz, ns), np.tile(ix, ns), np.full(ns, nt, np.int32))
    return grid, geom


@pytest.mark.parametrize("N,nrec", [(20, 1025), (129, 30)])
def test_tuned_calls_keep_two_steps_past_the_lds_tables(N, nrec):
    """A shot with more receivers, or a sponge wider, than the LDS-resident
    sweeps hold: a tuned call keeps the two-step sweeps' levels, as an untuned
    one does, however few its cells."""
    grid, geom = problem(300, 150, N, 2, nrec)
    for what in (B.WS_FORWARD, B.WS_HESSIAN, B.WS_GRADIENT, B.WS_AUTOGRAD):
        tuned = B.fwi_workspace_bytes(grid, geom, B.make_exec(autotune=1), what)
        untuned = B.fwi_workspace_bytes(grid, geom, None, what)
        assert tuned >= untuned, what


# Sizes that the library reported for these calls, and accepted, while it had
# only the z sweeps and no arrival map: 3 shots of 130 x 90 cells, sponge 11,
# 100 receivers, 110 samples.
Z_SIZES = {
    "none": dict(forward=1466880, hessian=1607424, gradient=7401216, autograd=7401216, image=17650432, born=2793984,
                 gn=8728320, exact=160110080),
    "two": dict(forward=1466880, hessian=1607424, gradient=9368576, autograd=9368576, image=28603392, born=2793984,
                gn=10302464, exact=160110080),
    "tuned": dict(forward=1466880, hessian=1607424, gradient=9368576, autograd=9368576, image=28603392, born=2793984,
                  gn=10302464, exact=160110080),
}
EXEC = {"none": {}, "two": dict(forward_steps=2, reverse_steps=2), "tuned": dict(autotune=1)}


def needed(call):
    """The bytes that a call refused for its workspace says it needs: the
    least it accepts (raised before any HIP call)."""
    with pytest.raises(B.FwiError) as e:
        call()
    assert e.value.code == B.FWI_ERR_WORKSPACE
    return int(re.search(r"need (\d+)", str(e.value)).group(1))


@pytest.mark.parametrize("ex", sorted(EXEC))
def test_workspaces_of_the_z_sweeps_sizes_are_accepted(ex):
    grid, geom = problem(130, 90, 11, 3, 100, nt=110)
    p = 0x1000
    a = (grid, geom, B.make_exec(**EXEC[ex]), p, p, 0)
    calls = {
        "forward": lambda: B.fwi_forward(*a, p, p, 16, stream=0),
        "hessian": lambda: B.fwi_hessian_diag(*a, B.HESS_EQ1, 0, "pm", p, p, 16, stream=0),
        "gradient": lambda: B.fwi_gradient(*a, p, "int", p, p, None, 0, "pm", None, p, 16, stream=0),
        "autograd": lambda: B.fwi_misfit_forward(*a, p, "int", p, p, 16, stream=0),
        "image": lambda: B.fwi_extended_image(*a, p, "int", p, None, 4, p, p, 16, stream=0),
        "born": lambda: B.fwi_born(*a, p, p, p, 16, stream=0),
        "gn": lambda: B.fwi_gn_hvp(*a, p, "int", p, p, p, 16, stream=0),
        "exact": lambda: B.fwi_offset_diag_exact(*a, 4, 30.0, 0, p, p, 16, stream=0),
    }
    for name, call in calls.items():
        assert needed(call) <= Z_SIZES[ex][name], name


def test_tuned_image_is_sized_for_two_steps_per_launch():
    """Tuned extended images of over 1.6 M cells a step run the two-step reverse
    sweep, whose windows hold twice the steps."""
    grid, geom = problem(1000, 400, 20, 4, 50)
    two = B.fwi_workspace_bytes(grid, geom, B.make_exec(forward_steps=2, reverse_steps=2), B.WS_EXTIMAGE, 3)
    assert B.fwi_workspace_bytes(grid, geom, B.make_exec(autotune=1), B.WS_EXTIMAGE, 3) >= two
