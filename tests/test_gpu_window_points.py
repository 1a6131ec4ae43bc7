"""Scattered targets on grids small enough for the window spread: widths, grids
of one window's size and just beyond, degenerate extents, and rules whose
order is not known (which keep the tiled spread), against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def targets(M, r, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    return g.uniform(-r, r, M) + 0.1 * r, g.uniform(-r, r, M)


@pytest.mark.parametrize("prec,tol", [("fp64", 10.0 ** -k) for k in (2, 5, 9, 11, 13)] + [("mixed", 10.0 ** -k) for k in (3, 5)])
@pytest.mark.parametrize("r", [1e-6, 0.02, 0.2, 0.35, 0.6, 1.2])
@pytest.mark.parametrize("M", [1, 300])
def test_grids_about_a_window(prec, tol, r, M):
    import paper_2010_05978_amd as fh
    ctx = fh.Context(prec, tol=tol)
    lz = 0.3
    xi, eta = targets(M, r, 3)
    args = (1.0, [0.05, 0.1], [0.0, 0.05], 5, 12, 24)
    ref_rule = oracle.quad_radial(*args)
    ref = oracle.fresnel_direct(*ref_rule, lz, 1.0, xi, eta)
    txi, teta = torch.tensor(xi, device="cuda"), torch.tensor(eta, device="cuda")
    print(f"window points: {prec} tol={tol} r={r} M={M}", flush=True)
    q = ctx.quad_radial(*args)
    u = ctx.field_points(q, lz, 1.0, txi, teta).cpu().numpy()
    tiled = fh.Context(prec, tol=tol, options=fh.fh_options(sigma=0, kernel_width=0, beta=0.0, tile=0,
                                                            max_subproblem=0, spread_method=2, deterministic=0))
    v = tiled.field_points(tiled.quad_radial(*args), lz, 1.0, txi, teta).cpu().numpy()
    tiled.close()
    # the nodes as a user's own, in an order that is not known: tiled, too
    q2 = ctx.quad_from_nodes(*(torch.tensor(a, device="cuda") for a in ref_rule))
    v2 = ctx.field_points(q2, lz, 1.0, txi, teta).cpu().numpy()
    assert np.linalg.norm(v2 - ref) / np.linalg.norm(ref) <= tol
    assert np.linalg.norm(u - ref) / np.linalg.norm(ref) <= tol
    assert np.linalg.norm(v - ref) / np.linalg.norm(ref) <= tol
    # the tiled spread sums the same kernel values: the difference is rounding,
    # of sums of 1440 strengths of size area/(lambda z) = 11, which the
    # corrections by 1/Phi raise by at most a hundred at the grid's edge
    if prec == "fp64":
        assert np.abs(u - v).max() <= 11.0 * 100.0 * 100.0 * 2.3e-16
    ctx.close()
