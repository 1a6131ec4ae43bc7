"""The window path on both sides of its limits, read from the binning stage's
time (none on the window path, two event marks of 5 to 8 us; 30 us and more for
a million nodes on the tiled path): window sizes, options that name a spread,
batches, and contexts whose autotuner found the automatic choice the fastest."""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LAM, Z, N, BIN_MS = 0.25, 1.0, 256, 0.018


@pytest.fixture(scope="module")
def fh():
    import paper_2010_05978_amd as fh
    return fh


def binned(ctx, call):
    """Whether the call bins its nodes."""
    for _ in range(2):
        call()
    ctx.set_timing(True)
    call()
    torch.cuda.synchronize()
    t = ctx.last_timing()[0]
    ctx.set_timing(False)
    print(f"  binning {t:.4f} ms", flush=True)
    return t > BIN_MS


def spacing(cells):
    return cells * LAM * Z / (2 * N)


def rule(ctx):
    return ctx.quad_radial(1.0, None, None, 0, 2500, 400)


# 2 c + 14 cells a side; 64 KB of LDS hold some 47 of them in FP64, 39 in FP32
@pytest.mark.parametrize("prec,cells,window", [("fp64", 1, True), ("fp64", 15.5, True), ("fp64", 19, False),
                                               ("mixed", 1, True), ("mixed", 13, True), ("mixed", 17, False)])
def test_window_size(fh, prec, cells, window):
    ctx = fh.Context(prec)
    q, h = rule(ctx), spacing(cells)
    assert binned(ctx, lambda: ctx.field_grid(q, LAM, Z, N, N, h, h)) != window
    ctx.close()


@pytest.mark.parametrize("name,value,window", [("sigma", 2.0, True), ("tile", 16, False), ("max_subproblem", 64, False),
                                               ("spread_method", 5, False), ("deterministic", 1, False)])
def test_named_options(fh, name, value, window):
    o = dict(sigma=0.0, kernel_width=0, beta=0.0, tile=0, max_subproblem=0, spread_method=0, deterministic=0)
    ctx = fh.Context("fp64", options=fh.fh_options(**dict(o, **{name: value})))
    q, h = rule(ctx), spacing(6)
    assert binned(ctx, lambda: ctx.field_grid(q, LAM, Z, N, N, h, h)) != window
    ctx.close()


# one rule too large for a window keeps its batch on the tiled path
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("radius,window", [(1.2, True), (5.0, False)])
def test_batches(fh, prec, radius, window):
    ctx = fh.Context(prec)
    quads, h = [rule(ctx), ctx.quad_radial(radius, None, None, 0, 250, 400)], spacing(6)
    lams, zs = np.full(2, LAM), np.full(2, Z)
    assert binned(ctx, lambda: ctx.field_grid_batch(quads, lams, zs, N, N, h, h)) != window
    ctx.close()


@pytest.mark.parametrize("sigma", [2.0, 1.25])
def test_autotuned(fh, tmp_path, sigma):
    q, h, path = None, spacing(6), tmp_path / "tune.jsonl"
    first = fh.Context("fp64")
    q = rule(first)
    first.autotune_grid(q, LAM, Z, N, N, h, h, cache_path=str(path))
    line = json.loads(path.read_text())
    for automatic in (0, 1):
        path.write_text(json.dumps(dict(line, automatic=automatic, sigma=sigma)) + "\n")
        ctx = fh.Context("fp64")
        ctx.autotune_grid(q, LAM, Z, N, N, h, h, cache_path=str(path))
        assert binned(ctx, lambda: ctx.field_grid(q, LAM, Z, N, N, h, h)) != bool(automatic)
        ctx.close()
    first.close()


# every kernel width that the matrix-core tile holds, on the window path (a
# width that is named, not chosen by the tolerance, may have no polynomial table)
@pytest.mark.parametrize("prec,digits", [("fp64", d) for d in range(1, 14)] + [("mixed", d) for d in range(2, 6)])
def test_kernel_widths(fh, prec, digits):
    o = dict(sigma=2.0, kernel_width=0, beta=0.0, tile=0, max_subproblem=0, deterministic=0)
    ctx = fh.Context(prec, tol=10.0 ** -digits, options=fh.fh_options(spread_method=0, **o))
    tiled = fh.Context(prec, tol=10.0 ** -digits, options=fh.fh_options(spread_method=2, **o))
    q, h, ctx_tol = rule(ctx), spacing(2), 10.0 ** -digits
    print(f"  width {ctx.query_params(N)['width']}", flush=True)
    assert not binned(ctx, lambda: ctx.field_grid(q, LAM, Z, N, N, h, h))
    u, v = (c.field_grid(q, LAM, Z, N, N, h, h) for c in (ctx, tiled))
    # rounding of a million terms of total size pi/(lambda z) = 13, and the
    # kernel's polynomials, whose error is a small part of the tolerance (the
    # wavefront spread evaluates them per cell, the window spread in pairs)
    assert float((u - v).abs().max()) <= 13.0 * (100.0 * (2.3e-16 if prec == "fp64" else 1.2e-7) + 1e-3 * ctx_tol)
    tiled.close()
    ctx.close()
