"""Merging crowded tiles in one launch: tiles with as many work items as the
reduce takes unmerged and one more, several crowded tiles among one block's
items, fewer elements than threads and more, against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# items of one node each (P = 1) make a crowded tile out of few nodes; 2048
# items per tile is the cap, beyond which items grow
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("mixed", 1e-5)])
@pytest.mark.parametrize("P", [1, 7])
@pytest.mark.parametrize("n_in_tile", [16, 17, 33, 40, 129, 2047, 2049, 5000])
@pytest.mark.parametrize("tile,method", [(4, 2), (16, 2), (32, 2), (0, 5), (16, 5)])
def test_crowded_tiles(prec, tol, P, n_in_tile, tile, method):
    import paper_2010_05978_amd as fh
    ctx = fh.Context(prec, tol=tol, options=fh.fh_options(sigma=0, kernel_width=0 if tile != 4 else 5, beta=0.0, tile=tile,
                                                          max_subproblem=P, spread_method=method, deterministic=0))
    if tile == 4:
        tol = 2e-3  # a five-cell kernel, so that a 4-cell tile reaches one tile on
    g = np.random.Generator(np.random.PCG64(n_in_tile + P))
    # three clusters inside one cell each (two in neighbouring tiles) and a
    # sprinkle of single nodes
    ctr = np.array([[0.013, 0.021], [0.21, 0.022], [-0.5, 0.6]])
    x = np.concatenate([c[0] + 1e-4 * g.random(n_in_tile) for c in ctr] + [g.uniform(-1, 1, 50)])
    y = np.concatenate([c[1] + 1e-4 * g.random(n_in_tile) for c in ctr] + [g.uniform(-1, 1, 50)])
    w = g.random(len(x))
    q = ctx.quad_from_nodes(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"), torch.tensor(w, device="cuda"))
    n, h, lz = 64, 0.03, 0.1
    print(f"crowded tiles: {prec} P={P} n={n_in_tile} tile={tile} method={method}", flush=True)
    u = ctx.field_grid(q, lz, 1.0, n, n, h, h).cpu().numpy().ravel()
    xi, eta = oracle.grid_targets(n, n, h, h)
    ref = oracle.fresnel_direct(x, y, w, lz, 1.0, xi, eta)
    # the field is of the size of its terms' sum (the strengths are random and
    # positive, clustered): the context's tolerance holds as it is
    assert np.linalg.norm(u - ref) / np.linalg.norm(ref) <= tol
    ctx.close()
