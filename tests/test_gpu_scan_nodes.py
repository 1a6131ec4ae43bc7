"""Either side of the node count from which the tile scan is a launch of its
own again, on few and on many tiles, against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("mixed", 1e-5)])
@pytest.mark.parametrize("N", [(1 << 19) - 1, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("n,h", [(64, 0.0007), (500, 0.011)])
def test_node_counts_about_the_limit(prec, tol, N, n, h):
    import paper_2010_05978_amd as fh
    ctx = fh.Context(prec, tol=tol)
    g = np.random.Generator(np.random.PCG64([N, n]))
    x, y, w = g.uniform(-1, 1, N), g.uniform(-1, 1, N), g.random(N) / N
    q = ctx.quad_from_nodes(*(torch.tensor(v, device="cuda") for v in (x, y, w)))
    lz = 0.05
    xi, eta = oracle.grid_targets(n, n, h, h)
    # the targets nearest the axis, where the terms add up
    idx = np.argsort(xi ** 2 + eta ** 2)[:60]
    ref = oracle.fresnel_direct(x, y, w, lz, 1.0, xi[idx], eta[idx])
    print(f"scan: {prec} N = {N}, {n} x {n}", flush=True)
    for rep in range(2):  # the counters are back at zero
        u = ctx.field_grid(q, lz, 1.0, n, n, h, h).cpu().numpy().ravel()[idx]
        assert np.linalg.norm(u - ref) / np.linalg.norm(ref) <= tol
    ctx.close()
