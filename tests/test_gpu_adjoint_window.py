"""The adjoint's Fourier sums over small windows: window sizes about the edges
of the 16-cell blocks and past the path's limit, ragged grids, both
precisions and both outputs (written, and added over wavelengths), against the
oracle's direct gradient."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# R h nf/lz cells to a side: windows of 16 to past 48 cells, narrow ones among
# them
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("fp64", 1e-4), ("mixed", 1e-5)])
@pytest.mark.parametrize("hx,hy", [(0.0005, 0.0005), (0.004, 0.0005), (0.008, 0.009), (0.014, 0.004), (0.016, 0.016), (0.02, 0.03)])
@pytest.mark.parametrize("n1,n2", [(64, 64), (66, 34), (18, 130), (200, 98)])
def test_windows(prec, tol, hx, hy, n1, n2):
    import paper_2010_05978_amd as fh
    ctx = fh.Context(prec, tol=tol)
    args = (1.0, [0.1, 0.05], [0.0, 0.1], 4, 9, 11)
    q, (x, y, w) = ctx.quad_radial(*args), oracle.quad_radial(*args)
    g = np.random.Generator(np.random.PCG64([n1, n2]))
    lams, zs = np.array([0.25, 0.31]), np.array([1.0, 1.2])
    gu = (g.normal(size=(2, n2, n1)) + 1j * g.normal(size=(2, n2, n1))).astype(np.complex128)
    t = torch.tensor(gu, device="cuda").to(ctx.cdtype)
    xc, yc = 0.1, -0.05
    xi, eta = oracle.grid_targets(n1, n2, hx, hy, xc, yc)
    refs = [oracle.fresnel_direct_vjp(x, y, w, lams[i], zs[i], xi, eta, gu[i].ravel(), occulter=True) for i in range(2)]
    print(f"adjoint window: {prec} {tol} {n1} x {n2} h = {hx}, {hy}", flush=True)
    one = [v.cpu().numpy() for v in ctx.field_grid_vjp(q, lams[0], zs[0], n1, n2, hx, hy, t[0], xc=xc, yc=yc, occulter=True)]
    both = [v.cpu().numpy() for v in ctx.field_grid_vjp_sum(q, lams, zs, n1, n2, hx, hy, t, xc=xc, yc=yc, occulter=True)]
    # the context's tolerance is that of the field; the node gradients are
    # differences x G - H of two such sums, at most |x - xi|/min(1, ..) of
    # them: within 20 times it here (targets reach 3 radii)
    for got, ref in ((one, refs[0]), (both, [a + b for a, b in zip(*refs)])):
        for a, b in zip(got, ref):
            assert np.linalg.norm(a - b) / np.linalg.norm(b) <= 20 * tol
    ctx.close()
