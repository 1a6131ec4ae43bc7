"""A single rule's blocks: node counts about those at which a block takes more
nodes (262,144 and its multiples on 256 CUs, 2,097,152), few and many nodes a
ray, against the oracle's rules."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("panels,q,m", [(8191, 16, 2), (8192, 16, 2), (8193, 16, 2), (512, 16, 32), (64, 16, 257),
                                        (8, 16, 2049), (1024, 16, 33), (4096, 16, 32), (8193, 16, 17), (131072, 16, 1),
                                        (131073, 16, 1)])
@pytest.mark.parametrize("K", [0, 3, 20])
def test_radial_rules(panels, q, m, K):
    import paper_2010_05978_amd as fh
    ctx = fh.Context("fp64")
    g = np.random.Generator(np.random.PCG64([panels, m, K]))
    a, b = 0.04 * g.normal(size=K), 0.04 * g.normal(size=K)
    print(f"rule of {panels * q * m} nodes, {m} a ray, {K} harmonics", flush=True)
    rule = ctx.quad_radial(1.0, a if K else None, b if K else None, panels, q, m)
    # angle rounding (4 2^-53 2 pi), times k in the k-th harmonic, and a few
    # roundings of coordinates of order 1
    tol = 1e-14 + 2.8e-15 * (np.arange(1, K + 1) * (np.abs(a) + np.abs(b))).sum()
    for got, want in zip(rule.export(), oracle.quad_radial(1.0, a if K else None, b if K else None, panels, q, m)):
        assert np.abs(got.cpu().numpy() - want).max() <= tol
    ctx.close()


@pytest.mark.parametrize("nv,q,m", [(7, 200, 187), (7, 200, 188), (128, 16, 128), (128, 128, 128), (128, 128, 129)])
def test_polygon_rules(nv, q, m):
    import paper_2010_05978_amd as fh
    ctx = fh.Context("fp64")
    t = 2.0 * np.pi * np.arange(nv) / nv
    rule = ctx.quad_polygon(np.cos(t), 0.7 * np.sin(t), q, m)
    for got, want in zip(rule.export(), oracle.quad_polygon(np.cos(t), 0.7 * np.sin(t), q, m)):
        assert np.abs(got.cpu().numpy() - want).max() <= 1e-14
    ctx.close()
