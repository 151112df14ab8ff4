"""Counters and claims: totals that workgroups keep to themselves for a while
arrive complete, and every start is relaxed and keyed exactly once, whatever
share of them is dealt out and whatever is claimed."""
import numpy as np
import pytest

import gribov_inputs as GI
import paper_1403_0555_amd as gc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with gc.Context(0) as c:
        yield c


def check(prog, starts, copies, n):
    conv = starts["status"] == 1
    assert prog["starts_done"] == n and prog["converged"] == conv.sum()
    assert prog["sweeps_total"] == int(starts["sweeps64"].astype(np.int64).sum())
    assert prog["distinct"] == len(copies) == len(np.unique(starts["key_lo"][conv]))
    assert int(copies["hits"].sum()) == conv.sum()
    assert prog["lanczos_iters"] == int(copies["lanczos_iters"].sum())
    # bounds that are only written where they change
    for c in copies[:: max(1, len(copies) // 50)]:
        mine = np.flatnonzero((starts["key_lo"] == c["key_lo"]) & (starts["key_hi"] == c["key_hi"]) & conv)
        assert c["first_start"] == mine[0] and c["hits"] == len(mine)
        assert abs(c["F"] - starts["F"][mine].min()) <= 1e-9


@pytest.mark.parametrize("extent,n", [
    ((4, 4), 1), ((4, 4), 5000), ((8, 8), 4097), ((8, 8), 40000), ((3, 3), 3000), ((16, 16), 9000), ((8, 8, 8), 5000),
    ((4, 4, 4, 4), 6001), ((10, 10, 10), 1500), ((8, 8, 8, 8), 40),
])
def test_totals_are_complete(ctx, extent, n):
    h = ctx.gc_orbit_load(extent, GI.orbit_angles(extent, 2, 0), 0)
    # a cap on the sweeps leaves some starts unconverged
    ctx.gc_launch(h, n, gc.SolveParams(omega=1.7, max_sweeps=60 if len(extent) == 2 else 300))
    assert ctx.gc_wait(h, 600_000) == gc.GC_OK
    check(ctx.gc_poll(h), ctx.gc_fetch_starts(h, n), ctx.gc_fetch(h), n)
    ctx.gc_release(h)
