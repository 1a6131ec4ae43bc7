"""Small grid calls evaluated as the quadrature sum itself: sizes at the edges
of the kernel's stages, tiles and splits, either side of the work limit, and
every option of the call, against the oracle and the transform."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rule(n, seed):
    g = np.random.Generator(np.random.PCG64([7, n, seed]))
    return g.uniform(-1, 1, n), g.uniform(-1, 1, n), g.uniform(0.0, 1.0, n)


def quad(ctx, r):
    return ctx.quad_from_nodes(*(torch.tensor(v, device="cuda") for v in r))


def reference(r, lz, grid, src=None, D=0.0):
    xi, eta = oracle.grid_targets(*grid)
    return oracle.fresnel_direct_src(*r, lz, 1.0, xi, eta, src=src, D=D)


# the sum has no truncation: with N strengths below 1 and phases of at most
# (4^2 + 4^2)/(2 lz) = 160 turns, rounded to 2 pi 160 2^-53 = 1.1e-13 each, a
# value's error stays below 1e-12 of sum |w|/lz in FP64, whatever the order; in
# mixed precision each operand carries 2^-24 and the FP32 sums N 2^-24 at worst
def bound(prec, r, lz):
    n = len(r[0])
    return np.abs(r[2]).sum() / lz * (1e-12 if prec == "fp64" else (4 + n / 16) * 6e-8)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("N", [1, 3, 15, 16, 17, 33, 500, 4800])
@pytest.mark.parametrize("n1,n2", [(2, 2), (16, 64), (18, 62), (64, 66), (130, 34), (100, 100)])
def test_sizes(prec, N, n1, n2):
    import paper_2010_05978_amd as fh
    ctx = fh.Context(prec)
    r, lz, grid = rule(N, n1), 0.1, (n1, n2, 0.03, 0.025)
    print(f"direct sum: {prec} N={N} {n1} x {n2}", flush=True)
    u = ctx.field_grid(quad(ctx, r), lz, 1.0, *grid).cpu().numpy().ravel()
    assert np.abs(u - reference(r, lz, grid)).max() <= bound(prec, r, lz)
    ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("lit", [False, True])
def test_options_of_the_call(prec, lit):
    import paper_2010_05978_amd as fh
    ctx = fh.Context(prec)
    r, lz, grid = rule(700, 1), 0.13, (70, 44, 0.03, 0.025, 0.3, -0.2)
    q = quad(ctx, r)
    src, D = None, 0.0
    if lit:
        src, D = (1.0 + 0.3 * np.cos(r[0])) * np.exp(1j * r[1]), 4.0
        q.set_illumination(torch.tensor(src, device="cuda"), D)
    ref = reference(r, lz, grid, src, D)
    u = ctx.field_grid(q, lz, 1.0, *grid[:4], xc=grid[4], yc=grid[5], occulter=True)
    assert np.abs(u.cpu().numpy().ravel() - (1.0 - ref)).max() <= 2.0 * bound(prec, r, lz)
    # a host array; again: the same bits
    host = torch.empty_like(u, device="cpu")
    ctx.field_grid(q, lz, 1.0, *grid[:4], xc=grid[4], yc=grid[5], occulter=True, out=host)
    assert torch.equal(host, u.cpu())
    ctx.close()


# just inside and just outside the work limit, and inside it with options that
# keep the transform: the two agree to the context's tolerance
@pytest.mark.parametrize("prec,work", [("fp64", 1.0e8), ("mixed", 1.5e8)])
def test_both_sides_of_the_limit(prec, work):
    import paper_2010_05978_amd as fh
    ctx, tol = fh.Context(prec), 1e-9 if prec == "fp64" else 1e-5
    opt = fh.fh_options(sigma=2.0, kernel_width=0, beta=0.0, tile=0, max_subproblem=0, spread_method=0, deterministic=0)
    tiled = fh.Context(prec, options=opt)
    n, lz = 160, 0.1
    for N in (int(work / n ** 2), int(work / n ** 2) + 1):
        r, grid = rule(N, 5), (n, n, 0.02, 0.02)
        u = ctx.field_grid(quad(ctx, r), lz, 1.0, *grid).cpu().numpy().ravel()
        v = tiled.field_grid(quad(tiled, r), lz, 1.0, *grid).cpu().numpy().ravel()
        print(f"direct sum and transform at N = {N}: {np.linalg.norm(u - v) / np.linalg.norm(v):.1e}", flush=True)
        assert np.linalg.norm(u - v) / np.linalg.norm(v) <= 2 * tol
    ctx.close()
    tiled.close()


def test_capped_workspace_falls_back(monkeypatch):
    import paper_2010_05978_amd as fh
    monkeypatch.setenv("FH_ALLOC_CAP_BYTES", str(8 << 20))
    ctx = fh.Context("fp64")
    monkeypatch.delenv("FH_ALLOC_CAP_BYTES")
    r, grid = rule(4000, 9), (100, 100, 0.03, 0.03)
    u = ctx.field_grid(quad(ctx, r), 0.1, 1.0, *grid).cpu().numpy().ravel()
    ref = reference(r, 0.1, grid)
    assert np.linalg.norm(u - ref) / np.linalg.norm(ref) <= 1e-9
    ctx.close()
