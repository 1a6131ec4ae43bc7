"""The window spread's split of a batch into workgroups: rules of very
different sizes in one batch, rules at the edges of a run of nodes, and the
rounding of long rules in mixed precision."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LAM, Z, RADIUS = 0.25, 1.0, 8  # the rules' radius in fine-grid cells


@pytest.fixture(scope="module")
def fh():
    import paper_2010_05978_amd as fh
    return fh


def tiled(fh, prec, **kw):
    return fh.Context(prec, options=fh.fh_options(sigma=0, kernel_width=0, beta=0.0, tile=0, max_subproblem=0,
                                                  spread_method=2, deterministic=0), **kw)


def test_largest_rule_of_an_uneven_batch_keeps_the_tolerance(fh):
    ctx = fh.Context("mixed", tol=1e-5)
    shapes = [(1.0, None, None, 2000, 20, 100)] + [(1.0, None, None, 2, 15, 100)] * 255
    quads = [ctx.quad_radial(*s) for s in shapes]
    n = 64
    h = RADIUS * LAM * Z / (2 * n)
    lams = np.full(len(quads), LAM)
    u = ctx.field_grid_batch(quads, lams, np.full(len(quads), Z), n, n, h, h)
    xi, eta = oracle.grid_targets(n, n, h, h)
    idx = np.random.Generator(np.random.PCG64(21)).choice(n * n, 24, replace=False)
    for b in (0, 200):
        ref = oracle.fresnel_direct(*oracle.quad_radial(*shapes[b]), LAM, Z, xi[idx], eta[idx])
        got = u[b].cpu().numpy().ravel()[idx]
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"  rule {b} of {quads[b].N} nodes: {err:.1e}", flush=True)
        assert err <= 1e-5
    ctx.close()


# 2e7 nodes in one rule: the error of the window path and of the tiled path,
# whose items hold some 800 nodes each
@pytest.mark.parametrize("points", [False, True], ids=["grid", "points"])
def test_long_rules_round_as_the_tiled_path(fh, points):
    n = 256
    h = RADIUS * LAM * Z / (2 * n)
    exact, ctx, other = tiled(fh, "fp64", tol=1e-12), fh.Context("mixed", tol=1e-5), tiled(fh, "mixed", tol=1e-5)
    q = ctx.quad_radial(1.0, [0.05], [0.1], 0, 100_000, 200)
    g = np.random.Generator(np.random.PCG64(22))
    xi, eta = (torch.tensor(g.uniform(-0.5, 0.5, 3000), device="cuda") for _ in range(2))

    def call(c):
        u = c.field_points(q, 2 * LAM, Z, xi, eta) if points else c.field_grid(q, LAM, Z, n, n, h, h)
        return u.to(torch.complex128)

    want = call(exact)
    err, base = (float((call(c) - want).norm() / want.norm()) for c in (ctx, other))
    print(f"  window {err:.2e}, tiled {base:.2e}", flush=True)
    assert err <= 1.25 * base
    for c in (exact, ctx, other):
        c.close()


# an uneven batch takes no longer than its nodes do in equal rules (a factor
# of three in hand; it was 24)
def test_uneven_batch_is_not_slower(fh):
    ctx = fh.Context("fp64")
    n, B, rays = 128, 64, 40_000
    h = RADIUS * LAM * Z / (2 * n)
    ms = []
    for sizes in ([rays // B] * B, [rays * 9 // 10] + [rays // 10 // B] * (B - 1)):
        quads = [ctx.quad_radial(1.0, None, None, 0, s, 100) for s in sizes]
        call = lambda: ctx.field_grid_batch(quads, np.full(B, LAM), np.full(B, Z), n, n, h, h)
        call(), call()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            call()
        b.record()
        b.synchronize()
        ms.append(a.elapsed_time(b) / 5)
    print(f"  equal {ms[0]:.3f} ms, uneven {ms[1]:.3f} ms", flush=True)
    assert ms[1] <= 3.0 * ms[0]
    ctx.close()


# rules of one node, of runs of 64, 128 and 512 nodes per wavefront and of four
# wavefronts' runs, a node more and fewer, and enough others that a run is long
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("count", [1, 40])
def test_edges_of_runs_and_workgroups(fh, prec, count):
    sizes = [1, 63, 64, 65, 128, 511, 512, 513, 2047, 2048, 2049, 4097, 60_000] * count
    ctx, other = fh.Context(prec), tiled(fh, prec)
    quads = [ctx.quad_radial(1.0, None, None, 0, k, 1) for k in sizes]
    n = 32
    # (1 cell in radius: any order is close enough)
    h = LAM * Z / (2 * n)
    lams = LAM * np.linspace(1.0, 1.2, len(sizes))
    zs = np.full(len(sizes), Z)
    u = ctx.field_grid_batch(quads, lams, zs, n, n, h, h)
    v = other.field_grid_batch(quads, lams, zs, n, n, h, h)
    # both paths sum the same kernel values: rounding of terms of total size
    # area/(lambda z) = 13
    assert float((u - v).abs().max()) <= 13.0 * 100.0 * (2.3e-16 if prec == "fp64" else 1.2e-7)
    ctx.close()
    other.close()
