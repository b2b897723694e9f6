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


@pytest.mark.parametrize("nx,nz,N,ns,nrec,fs,what,steps,shots", [
    (300, 150, 20, 9, 1024, False, B.WS_GRADIENT, (0, 0), 8),
    (300, 150, 20, 9, 1025, False, B.WS_GRADIENT, (2, 2), 8),    # receivers of a shot
    (300, 150, 128, 2, 30, False, B.WS_GRADIENT, (0, 0), 2),
    (300, 150, 129, 2, 30, False, B.WS_GRADIENT, (2, 2), 2),     # sponge cells
    (960, 360, 20, 4, 30, False, B.WS_GRADIENT, (0, 0), 4),      # 1.6 M cells a step
    (961, 360, 20, 4, 30, False, B.WS_GRADIENT, (0, 2), 4),
    (961, 360, 20, 4, 30, False, B.WS_GNHVP, (0, 2), 4),
    (961, 360, 20, 4, 30, True, B.WS_GRADIENT, (0, 1), 4),       # no two steps with a free surface
    (960, 360, 20, 20, 30, False, B.WS_FORWARD, (0, 1), 16),
    (961, 360, 20, 24, 30, False, B.WS_FORWARD, (2, 1), 24),     # 8 M cells a step
    (961, 360, 20, 24, 30, False, B.WS_HESSIAN, (2, 1), 24),
    (961, 360, 20, 24, 30, False, B.WS_BORN, (1, 1), 24),
    (961, 360, 20, 24, 30, False, B.WS_AUTOGRAD, (2, 2), 24),
])
def test_query_reports_the_sweeps_that_run(nx, nz, N, ns, nrec, fs, what, steps, shots):
    """Steps per launch on both sides of each limit (0: LDS-resident); the
    settings passed back in choose the same sweeps."""
    grid, geom = problem(nx, nz, N, ns, nrec, fs=fs)
    q = B.fwi_exec_query(grid, geom, None, what)
    assert (q["forward_steps"], q["reverse_steps"], q["shots_in_flight"]) == (*steps, shots)
    # rows and prefetch: 0 where naming them would choose another sweep
    free = steps[0] == 0 or (steps[0] == 2 and what in (B.WS_FORWARD, B.WS_HESSIAN))
    assert (q["tile_rows"] == 0) == free and (q["prefetch"] == 0) == free
    assert (q["tile_rows_reverse"] == 0) == (steps[1] == 0) and (q["prefetch_reverse"] == 0) == (steps[1] == 0)
    assert B.fwi_exec_query(grid, geom, B.make_exec(**q), what) == q


def test_query_of_tuned_calls_takes_every_shot_where_lds_resident():
    """Without a tuning entry: what is fixed by the sizes alone."""
    tuned = B.make_exec(autotune=1)
    grid, geom = problem(130, 90, 11, 40, 30)
    for what in (B.WS_FORWARD, B.WS_GRADIENT, B.WS_AUTOGRAD):
        q = B.fwi_exec_query(grid, geom, tuned, what)
        assert q["shots_in_flight"] == 40 and q["forward_steps"] == 0, what
    assert q["reverse_steps"] == 0 and q["shots_in_flight_reverse"] == 40
    grid, geom = problem(130, 90, 11, 40, 1025)
    q = B.fwi_exec_query(grid, geom, tuned, B.WS_GRADIENT)
    assert q["shots_in_flight"] == 32 and q["forward_steps"] > 0 and q["reverse_steps"] > 0


def test_forward_steps_are_the_gradient_calls_alone():
    """Calls that do not use the field choose their sweeps as if it were 0,
    tuned or not."""
    for nx, ns, nrec in ((130, 3, 30), (961, 24, 30), (300, 2, 1025)):
        grid, geom = problem(nx, 360, 20, ns, nrec)
        for what in (B.WS_FORWARD, B.WS_HESSIAN, B.WS_BORN, B.WS_GNHVP):
            for steps in (1, 2):
                for tuned in (0, 1):
                    a = B.fwi_workspace_bytes(grid, geom, B.make_exec(autotune=tuned, forward_steps=steps), what)
                    assert a == B.fwi_workspace_bytes(grid, geom, B.make_exec(autotune=tuned), what)
