"""Which calls the window spread takes: rules whose consecutive nodes lie close
together in fine-grid cells.  Others, whose nodes it would take one by one at
several times the cost, stay on the tiled path, for both transform types.  The
path shows in the stage times: the window spread has no binning stage (two
event marks, 5 to 8 us), a tiled call of a million nodes spends 36 us or more
there."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 1_000_000
BIN_MS = 0.018  # between the two


@pytest.fixture(scope="module")
def fh():
    import paper_2010_05978_amd as fh
    return fh


def rule(ctx, kind, m):
    if kind == "radial":
        return ctx.quad_radial(1.0, None, None, 0, N // m, m)
    if kind == "polygon":
        t = np.arange(8) * np.pi / 4
        return ctx.quad_polygon(np.cos(t), np.sin(t), N // m // 8, m)
    if kind == "kite":
        return ctx.quad_fourier([0.0, 0.5, 0.5], None, [0.0, 0.0, 0.0], [0.0, 1.0, 0.0], 0, N // m, m)
    if kind == "starshade":
        return ctx.quad_starshade(20, 0.5, 1.0, 0.5, 6.0, m, int(0.8 * N) // 20 // m, int(0.2 * N) // m, m)
    if kind == "koch":
        return ctx.quad_koch(9, [20] * 5 + [2] * 5)
    B = ctx.boundary_radial(1.0, None, None, 0, N // m)
    if kind == "shuffled":
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        B = B[:, torch.randperm(B.shape[1], device="cuda", generator=g)].contiguous()
    q = ctx.quad_from_boundary(B[0], B[1], B[2], B[3], m)
    if kind == "nodes":
        q = ctx.quad_from_nodes(*(torch.as_tensor(v, device="cuda") for v in q.export()))
    return q


# (rule, radial nodes, radius in cells, window path in FP64, in mixed)
CASES = [("radial", 200, 10, True, True), ("radial", 1, 10, True, True), ("radial", 2, 10, False, True),
         ("radial", 4, 8, False, True), ("radial", 12, 11, False, False), ("radial", 24, 10, False, True),
         ("radial", 24, 5, True, True), ("radial", 4, 4, True, True),
         ("polygon", 12, 11, False, False), ("polygon", 100, 11, True, True),
         ("kite", 12, 11, False, False), ("kite", 100, 11, True, True),
         ("starshade", 8, 12, False, True), ("starshade", 80, 12, True, True),
         ("koch", 0, 12, True, True),
         ("boundary", 100, 11, True, True), ("boundary", 4, 11, False, False),
         ("shuffled", 100, 11, True, True), ("shuffled", 4, 11, False, False), ("shuffled", 1, 11, False, False),
         ("nodes", 100, 4, False, False)]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("kind,m,R,w64,w32", CASES, ids=[f"{c[0]}-{c[1]}-{c[2]}" for c in CASES])
def test_path_by_order(fh, prec, kind, m, R, w64, w32):
    ctx = fh.Context(prec)
    q = rule(ctx, kind, m)
    lam, z, n = 0.25, 1.0, 256
    h = R * lam * z / (2 * n)
    for _ in range(3):
        u = ctx.field_grid(q, lam, z, n, n, h, h)
    ctx.set_timing(True)
    ctx.field_grid(q, lam, z, n, n, h, h)
    torch.cuda.synchronize()
    t = ctx.last_timing()
    print(f"  {prec} {kind} m {m} R {R}: binning {t[0]:.4f} of {t[4]:.4f} ms", flush=True)
    assert (t[0] < BIN_MS) == (w64 if prec == "fp64" else w32)
    ctx.set_timing(False)
    # both paths sum the same kernel values: rounding of a million terms of
    # total size area/(lambda z) = 13
    ctx.set_options(fh.fh_options(sigma=0, kernel_width=0, beta=0.0, tile=0, max_subproblem=0, spread_method=2,
                                  deterministic=0))
    v = ctx.field_grid(q, lam, z, n, n, h, h)
    assert float((u - v).abs().max()) <= 13.0 * 100.0 * (2.3e-16 if prec == "fp64" else 1.2e-7)
    ctx.close()


# type 3: a grid of one window (32 cells a side, the rule 10 cells in radius)
@pytest.mark.parametrize("prec,m,kind,window", [
    ("fp64", 100, "radial", True), ("fp64", 2, "radial", False), ("fp64", 1, "shuffled", False),
    ("mixed", 100, "radial", True), ("mixed", 2, "radial", True), ("mixed", 8, "radial", False),
    ("mixed", 1, "shuffled", False)])
def test_points_path_by_order(fh, prec, m, kind, window):
    ctx = fh.Context(prec)
    q = rule(ctx, kind, m)
    g = np.random.Generator(np.random.PCG64(4))
    xi, eta = (torch.tensor(g.uniform(-0.5, 0.5, 500), device="cuda") for _ in range(2))
    t = ctx.targets(xi, eta, box=(-0.5, 0.5, -0.5, 0.5))
    for _ in range(3):
        ctx.field_targets(q, 0.2, 1.0, t)
    ctx.set_timing(True)
    ctx.field_targets(q, 0.2, 1.0, t)
    torch.cuda.synchronize()
    ms = ctx.last_timing()
    print(f"  {prec} {kind} m {m}: binning {ms[0]:.4f} of {ms[4]:.4f} ms", flush=True)
    assert (ms[0] < BIN_MS) == window
    ctx.close()
