"""The largest lattices, a workgroup of 16 wavefronts per start: slots full
and partly idle, coefficients of one colour or both in registers (single
precision) and from memory, against the oracle."""
import numpy as np
import pytest

import gribov_inputs as GI
import paper_1403_0555_amd as gc
from oracle import oracle as O

from tests.test_gpu_parity import F_TOL_PER_SITE, oracle_params, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with gc.Context(0) as c:
        yield c


@pytest.mark.parametrize("extent", [(32, 66), (50, 50), (64, 64), (14, 14, 14), (16, 16, 16), (6, 6, 8, 8), (8, 8, 8, 8)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_workgroup_starts_match_the_oracle(ctx, extent, precision):
    n, V = 3, GI.volume(extent)
    phi = GI.orbit_angles(extent, 7, 0)
    p = gc.SolveParams(omega=1.7, precision=precision, max_sweeps=3000)
    h, _, starts, _ = run_gpu(ctx, extent, phi, n, p)
    rec, _, _ = O.solve(extent, phi, np.arange(n), oracle_params(p))
    assert np.array_equal(starts["status"], rec["status"])
    for f in ("sweeps32", "sweeps64"):
        assert np.max(np.abs(starts[f].astype(np.int64) - rec[f])) <= 1
    conv = rec["status"] == O.CONVERGED
    assert np.array_equal(starts["key_lo"][conv], rec["key_lo"][conv])
    same = conv & (starts["sweeps32"] == rec["sweeps32"]) & (starts["sweeps64"] == rec["sweeps64"])
    if same.any():
        tol = F_TOL_PER_SITE if precision == "fp64" else 1e-8   # |div| reaches 1e-7 on average
        assert np.max(np.abs(starts["F"][same] - rec["F"][same])) / V < tol
    ctx.gc_release(h)
