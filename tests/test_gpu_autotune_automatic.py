"""An autotuned context whose automatic choice was the fastest goes on to
choose its path by itself: it gives, bit for bit, what a context without
options gives (the direct sum, and the window path and type 3 in mixed
precision, add in a fixed order), and not what the named options give."""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RADIAL = (1.0, [0.02, 0.0, 0.1], [0.0, 0.05, 0.0], 0, 500, 40)
# a call for each path: rule, grid (the last one's reach is three cells a side)
CALLS = [("fp64", "direct", (1.0, None, None, 6, 20, 40), (100, 100, 0.03, 0.03)),
         ("mixed", "direct", (1.0, None, None, 6, 20, 40), (100, 100, 0.03, 0.03)),
         ("mixed", "window", RADIAL, (512, 512, 0.0005, 0.0005)),
         ("mixed", "points", RADIAL, (512, 512, 0.0005, 0.0005))]


@pytest.fixture(scope="module")
def fh():
    import paper_2010_05978_amd as fh
    return fh


@pytest.mark.parametrize("prec,path,shape,grid", CALLS, ids=[f"{c[0]}-{c[1]}" for c in CALLS])
def test_automatic_winner_keeps_the_automatic_path(fh, tmp_path, prec, path, shape, grid):
    lam, z = 0.25, 1.0
    g = np.random.Generator(np.random.PCG64(11))
    xi, eta = (torch.tensor(g.uniform(-0.5, 0.5, 300), device="cuda") for _ in range(2))

    def call(ctx, q):
        if path == "points":
            return ctx.field_points(q, lam, z, xi, eta)
        return ctx.field_grid(q, lam, z, *grid)

    plain = fh.Context(prec)
    q = plain.quad_radial(*shape)
    want = call(plain, q)
    cache = tmp_path / "tune.jsonl"
    tuned = fh.Context(prec)
    best = tuned.autotune_grid(q, lam, z, *grid, cache_path=str(cache))
    line = json.loads(cache.read_text())
    if line["automatic"]:
        assert torch.equal(call(tuned, q), want)
    # the same line, with each of the two winners, read by a new context; the
    # named options' upsampling factor must not stay behind
    for automatic in (1, 0):
        cache.write_text(json.dumps(dict(line, automatic=automatic, sigma=2.0 if automatic == 0 else 1.25)) + "\n")
        ctx = fh.Context(prec)
        got = ctx.autotune_grid(q, lam, z, *grid, cache_path=str(cache))
        assert (got.tile, got.max_subproblem, got.spread_method) == (best.tile, best.max_subproblem, best.spread_method)
        same = torch.equal(call(ctx, q), want)
        print(f"  {prec} {path}: automatic {automatic}, same bits {same}", flush=True)
        assert same == bool(automatic)
        ctx.close()
    tuned.close()
    plain.close()
