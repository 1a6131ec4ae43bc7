"""The window path's last kernel at the largest windows, on grids that ask for
its largest chunks of output rows (128), against the tiled path."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# windows of (2 R h1-cells + 14) x (2 R h2-cells + 14) cells: in FP64 49 to 52 x
# 33 to 47 (52 padded columns and 48 rows, where 128 rows' factors no longer
# fit beside the window in 64 KB), and its neighbours
@pytest.mark.parametrize("c1,c2", [(18.4, 10.5), (18.9, 13.0), (18.4, 16.4), (17.0, 16.4), (16.4, 18.4), (10.0, 24.4)])
def test_largest_windows_on_large_grids(c1, c2):
    import paper_2010_05978_amd as fh
    lam, z, n = 0.25, 1.2, 2048
    ctx = fh.Context("fp64")
    tiled = fh.Context("fp64", options=fh.fh_options(sigma=0, kernel_width=0, beta=0.0, tile=0, max_subproblem=0,
                                                     spread_method=2, deterministic=0))
    q = ctx.quad_radial(1.0, None, None, 0, 300, 400)
    h1, h2 = (c * lam * z / (2 * n) for c in (c1, c2))
    print(f"window of some {2 * c1 + 14:.0f} x {2 * c2 + 14:.0f} cells", flush=True)
    u, v = (c.field_grid(q, lam, z, n, n, h1, h2) for c in (ctx, tiled))
    # rounding of 120,000 terms of total size pi/(lambda z) = 10.5
    assert float((u - v).abs().max()) <= 10.5 * 100.0 * 2.3e-16
    tiled.close()
    ctx.close()
