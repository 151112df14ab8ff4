"""Team relaxation kernels (one workgroup, several starts in step) against the
oracle, start by start, at the edges of their shapes: half volumes of one site
more than a wavefront holds, the first and last of each wavefront count's
range, two sites per thread, three, five and seven colours, and launches with
more starts than the workgroups hold, so that places are refilled."""
import numpy as np
import pytest

import gribov_inputs as GI
import paper_1403_0555_amd as gc
from oracle import oracle as O

from tests.test_gpu_parity import compare_starts, oracle_params, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with gc.Context(0) as c:
        yield c


@pytest.mark.parametrize("extent", [
    (132,), (2, 66), (16, 16), (2, 130), (2, 258), (32, 32), (2, 1024),      # 1D and 2D, 2 to 16 wavefronts
    (2, 4, 18), (4, 6, 6), (8, 8, 8), (2, 2, 130), (2, 2, 258), (12, 12, 12), (8, 16, 16),
    (2, 2, 2, 18), (4, 4, 4, 4), (2, 4, 8, 8), (2, 2, 2, 66), (4, 6, 6, 6), (2, 2, 2, 130), (6, 6, 6, 6),
    (4, 6, 8, 8), (2, 4, 10, 20), (8, 8, 8, 4),                              # 4D, two sites per thread in the last
    (3, 3), (9, 15), (3, 3, 3, 3), (3, 6, 9), (9, 9, 9), (3, 21, 21), (3, 3, 9, 9),
    (5, 5), (5, 5, 5), (5, 5, 5, 5), (7, 7), (7, 7, 7),
])
@pytest.mark.parametrize("kw", [{"omega": 1.7}, {"omega": 1.0, "max_sweeps": 40, "stop_norm": "max_abs", "eps64": 1e-3},
                                {"omega": 1.6, "check_every": 3}])
def test_team_kernels_match_the_oracle(ctx, extent, kw):
    n = 24 if GI.volume(extent) > 600 else 48
    phi = GI.orbit_angles(extent, 3, 1)
    p = gc.SolveParams(first_start=5, **{"max_sweeps": 150, **kw})
    h, _, starts, _ = run_gpu(ctx, extent, phi, n, p, orbit_index=1)
    rec, _, _ = O.solve(extent, phi, 5 + np.arange(n), oracle_params(p, 1))
    compare_starts(extent, starts, rec)
    ctx.gc_release(h)


@pytest.mark.parametrize("extent,n", [((16, 16), 6000), ((2, 2, 2, 18), 6000), ((6, 6, 6), 6000), ((3, 3, 3), 6000)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_refilled_places_do_not_depend_on_the_launch(ctx, extent, n, precision):
    """A start's record is the same in a launch of many starts (places are
    refilled many times over) and in one of few."""
    phi = GI.orbit_angles(extent, 4, 2)
    h, _, many, prog = run_gpu(ctx, extent, phi, n, gc.SolveParams(omega=1.7, precision=precision), orbit_index=2)
    assert prog["starts_done"] == n and np.all(many["status"] == 1)
    few = n - 37
    h2, _, last, _ = run_gpu(ctx, extent, phi, 37, gc.SolveParams(omega=1.7, precision=precision, first_start=few),
                             orbit_index=2)
    for f in ("status", "sweeps32", "sweeps64", "F", "D", "key_hi", "key_lo"):
        assert np.array_equal(many[f][few:], last[f]), f
    ctx.gc_release(h)
    ctx.gc_release(h2)


@pytest.mark.parametrize("extent", [(16, 16), (32, 32), (8, 8, 8), (4, 4, 4, 4), (4, 6, 6, 6), (9, 15), (3, 3, 3, 3),
                                    (9, 9, 9), (5, 5, 5)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_a_start_on_its_own_stops_at_its_sweep(ctx, extent, precision):
    """A start that a workgroup holds alone runs several sweeps between looks
    at its norms: every cap, and every sweep that converges, is found."""
    phi = GI.orbit_angles(extent, 6, 0)
    for k, kw in enumerate([{"max_sweeps": c} for c in range(1, 9)] +
                           [{"eps64": e, "eps32": 10 * e} for e in (3e-2, 1e-2, 3e-3, 1e-3, 3e-4, 1e-5)]):
        p = gc.SolveParams(omega=1.7, precision=precision, first_start=11 * k, **kw)
        h, _, starts, _ = run_gpu(ctx, extent, phi, 3, p)
        rec, _, _ = O.solve(extent, phi, 11 * k + np.arange(3), oracle_params(p))
        assert np.array_equal(starts["status"], rec["status"])
        assert np.max(np.abs(starts["sweeps32"].astype(np.int64) - rec["sweeps32"])) <= (precision == "mixed")
        if precision == "fp64":
            assert np.array_equal(starts["sweeps64"], rec["sweeps64"])
        ctx.gc_release(h)


@pytest.mark.parametrize("extent,precision", [
    ((16, 16), "fp64"), ((32, 32), "fp64"), ((6, 6, 6), "fp64"), ((4, 4, 4, 4), "fp64"), ((4, 4, 6, 6), "fp64"),
    ((10, 10, 10), "mixed"), ((4, 6, 6, 6), "mixed")])
def test_starts_that_end_beside_the_last_one(ctx, extent, precision):
    """The end of a launch, where workgroups go from several starts in step to
    one on its own: every record, and the final states of the last starts to
    be claimed, as from launches that give each workgroup a single start."""
    n, single = 7000 if GI.volume(extent) <= 256 else 3000, 250
    phi = GI.orbit_angles(extent, 9, 1)
    h, _, many, _ = run_gpu(ctx, extent, phi, n, gc.SolveParams(omega=1.7, precision=precision), orbit_index=1)
    last = range(n - single, n)
    states = [ctx.gc_fetch_start_state(h, k) for k in last]
    for first in range(0, n, single):
        p = gc.SolveParams(omega=1.7, precision=precision, first_start=first)
        h2, _, few, _ = run_gpu(ctx, extent, phi, single, p, orbit_index=1)
        for f in ("status", "sweeps32", "sweeps64", "F", "D", "key_hi", "key_lo"):
            assert np.array_equal(many[f][first:first + single], few[f]), f
        if first == last[0]:
            for k, state in zip(last, states):
                assert np.array_equal(state, ctx.gc_fetch_start_state(h2, k)), k
        ctx.gc_release(h2)
    ctx.gc_release(h)


@pytest.mark.parametrize("extent", [(4, 4, 8, 8), (2, 8, 8, 8), (2, 2, 2, 114), (2, 2, 2, 128)])
@pytest.mark.parametrize("kw", [{"omega": 1.7}, {"omega": 1.0, "max_sweeps": 40, "stop_norm": "max_abs", "eps64": 1e-3},
                                {"omega": 1.6, "check_every": 3}])
def test_eight_wavefronts_in_four_dimensions(ctx, extent, kw):
    """449 to 512 sites a colour, five starts in step: against the oracle, and
    in a launch of more starts than the workgroups hold at once."""
    test_team_kernels_match_the_oracle(ctx, extent, kw)
    phi = GI.orbit_angles(extent, 3, 1)
    p = gc.SolveParams(**{"max_sweeps": 150, **kw})
    h, _, many, _ = run_gpu(ctx, extent, phi, 2000, p, orbit_index=1)
    h2, _, few, _ = run_gpu(ctx, extent, phi, 24, p, orbit_index=1)
    for f in ("status", "sweeps64", "F", "D", "key_hi", "key_lo"):
        assert np.array_equal(many[f][:24], few[f], equal_nan=many[f].dtype.kind == "f"), f
    ctx.gc_release(h)
    ctx.gc_release(h2)


def test_relax_time_counts_the_start_states(ctx):
    """With a single sweep per start, drawing the start states is a large part
    of a launch: its device times add up to nearly all of it."""
    extent, n = (6, 6, 6, 6), 400000
    h = ctx.gc_orbit_load(extent, GI.orbit_angles(extent, 2, 0), 0)
    for _ in range(3):
        ctx.gc_launch(h, n, gc.SolveParams(omega=1.7, max_sweeps=1))
        assert ctx.gc_wait(h, 60_000) == gc.GC_OK
        prog = ctx.gc_poll(h)
    assert prog["nonconverged"] == n
    device = prog["device_ms"] + prog["post_ms"] + prog["filter_ms"]
    assert device > 0.85 * prog["submit_to_done_ms"], prog
    ctx.gc_release(h)
