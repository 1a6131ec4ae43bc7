"""Grids whose length leaves the six-cell tile a remainder that the tile
reduce cannot follow: the automatic choice falls back to 16-cell tiles there.
Against the oracle, below and from the node count that takes the matrix-core
spread, on grids that fall back and on neighbours that do not, with the last
tile row full and the nodes spread out and crowded into one tile."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("fp64", 1e-6), ("mixed", 1e-5)])
@pytest.mark.parametrize("N", [(1 << 18) - 1, 1 << 18, (1 << 18) + 777])
@pytest.mark.parametrize("n1,n2", [(256, 256), (250, 256), (256, 1000), (254, 258), (500, 250)])
@pytest.mark.parametrize("size", [1.0, 0.02])
def test_field(prec, tol, N, n1, n2, size):
    import paper_2010_05978_amd as fh
    ctx = fh.Context(prec, tol=tol)
    g = np.random.Generator(np.random.PCG64(N + n1 * 7 + n2))
    x, y = size * g.uniform(-1, 1, N), size * g.uniform(-1, 1, N)
    w = g.random(N) / N
    q = ctx.quad_from_nodes(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"), torch.tensor(w, device="cuda"))
    h, lz = 3.0 / max(n1, n2), 0.05
    print(f"fallback: {prec} tol={tol} N={N} {n1}x{n2} size={size}", flush=True)
    u = ctx.field_grid(q, lz, 1.0, n1, n2, h, h).cpu().numpy().ravel()
    xi, eta = oracle.grid_targets(n1, n2, h, h)
    k = g.choice(n1 * n2, 40, replace=False)
    ref = oracle.fresnel_direct(x, y, w, lz, 1.0, xi[k], eta[k])
    # an error of tol in L2 over the whole grid, spread evenly, is tol times
    # the grid's root mean square at a target; a sample of 40 of it stays
    # within three times that
    rms = np.linalg.norm(u) / np.sqrt(u.size)
    assert np.linalg.norm(u[k] - ref) / np.sqrt(len(k)) <= 3 * tol * rms
    ctx.close()
