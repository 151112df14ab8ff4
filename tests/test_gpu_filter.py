"""The line-segment FP filter against the dense spectrum at the edges of its
shapes: one to eight wavefronts, segments of every length, whole lines and
parts of them, an odd last site, idle threads, Krylov spaces shorter than a
block of Sturm rows, and iterations stopped at their cap."""
import numpy as np
import pytest

import gribov_inputs as GI
import paper_1403_0555_amd as gc
from oracle import oracle as O

from tests.test_gpu_parity import LAMBDA_TOL, compare_tables, oracle_params, run_gpu

pytestmark = pytest.mark.gpu

EXTENTS = [
    (5,), (3, 3), (4, 4), (6, 6), (9, 9), (12, 12), (16, 16), (14, 14), (20, 20), (10, 26), (128, 4), (2, 64),
    (6, 6, 6), (5, 5, 5), (7, 7, 7), (8, 8, 8), (9, 9, 9), (10, 10, 10), (10, 12, 12), (12, 12, 12), (3, 21, 21),
    (4, 4, 4, 4), (3, 3, 3, 3), (6, 6, 6, 6), (6, 6, 6, 8), (8, 8, 8, 4),
]


@pytest.fixture(scope="module")
def ctx():
    with gc.Context(0) as c:
        yield c


@pytest.mark.parametrize("extent", EXTENTS)
def test_filter_matches_the_dense_spectrum(ctx, extent):
    n = 2 if GI.volume(extent) > 600 else 6
    phi = GI.orbit_angles(extent, 5, 1)
    p = gc.SolveParams(omega=1.7)
    h, copies, _, _ = run_gpu(ctx, extent, phi, n, p, orbit_index=1)
    o = O.enumerate_copies(extent, phi, np.arange(n), oracle_params(p, 1))
    compare_tables(extent, phi, copies, o, p)
    ctx.gc_release(h)


@pytest.mark.parametrize("extent", [(4, 4), (9, 9), (5, 5, 5), (9, 9, 9), (4, 4, 4, 4), (6, 6, 6, 8)])
def test_capped_iterations_bound_the_spectrum_from_above(ctx, extent):
    """A Ritz value is an upper bound of lambda_2 that never rises with the
    iteration count; a capped run says so in its flags."""
    phi = GI.orbit_angles(extent, 5, 1)
    h, ref, _, _ = run_gpu(ctx, extent, phi, 2, gc.SolveParams(omega=1.7), orbit_index=1)
    ctx.gc_release(h)
    last = np.full(len(ref), np.inf)
    for cap in (1, 2, 7, 8, 9, 15, 16):
        h, c, _, _ = run_gpu(ctx, extent, phi, 2, gc.SolveParams(omega=1.7, lanczos_max_iter=cap), orbit_index=1)
        ctx.gc_release(h)
        assert np.array_equal(c["key_lo"], ref["key_lo"])
        capped = (c["flags"] & gc.GC_FLAG_LANCZOS_CAP) != 0
        assert np.all(c["lanczos_iters"][capped] == cap) and np.all(c["lanczos_iters"] <= cap)
        if cap < 8:
            assert capped.all()
        assert np.all(c["lambda2"] >= ref["lambda2"] - LAMBDA_TOL)
        assert np.all(c["lambda2"] <= last + LAMBDA_TOL)
        last = c["lambda2"]


def start_vector(V):
    """The filter's start vector: mixed site indices as fractions, less their mean, normalised."""
    m = (1 << 64) - 1
    x = np.empty(V)
    for i in range(V):
        z = (i + 0x5851F42D4C957F2D) & m
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
        x[i] = ((z ^ (z >> 31)) >> 11) * 2.0 ** -53 - 0.5
    x -= x.mean()
    return x / np.linalg.norm(x)


@pytest.mark.parametrize("extent", [(4, 4), (5, 5), (10, 26), (6, 8, 10), (10, 12, 12), (3, 21, 21), (14, 14, 14),
                                    (6, 6, 6, 6), (6, 6, 6, 8)])
def test_one_iteration_is_the_start_vectors_quotient(ctx, extent):
    """Stopped after one iteration, the filter returns q.(M q) of its start
    vector: threads without sites of their own, up to an eighth of the
    workgroup past the arrays' stride, have no part in it."""
    phi, V = GI.orbit_angles(extent, 5, 1), GI.volume(extent)
    p = gc.SolveParams(omega=1.7, lanczos_max_iter=1)
    h, copies, _, _ = run_gpu(ctx, extent, phi, 2, p, orbit_index=1)
    q = start_vector(V)
    for c in copies:
        theta = ctx.gc_fetch_start_state(h, int(c["rep_start"]))
        _, _, _, w = O.observe(extent, phi, theta)
        assert abs(c["lambda2"] - q @ (O.fp_operator(extent, w) @ q)) < LAMBDA_TOL
        assert int(c["flags"]) & gc.GC_FLAG_LANCZOS_CAP and c["lanczos_iters"] == 1
    ctx.gc_release(h)
