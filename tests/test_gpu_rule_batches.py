"""Many rules computed again in one launch inside a batched call: block and
search edges of the launch, and rules exchanged for others of the same sizes."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fh():
    import paper_2010_05978_amd as fh
    return fh


def cpu(t):
    return t.detach().cpu().numpy()


def radial(K, panels, q, m, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    return ("radial", 0.04 * g.normal(size=K), 0.04 * g.normal(size=K), panels, q, m)


def polygon(nv, q, m, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    th = 2.0 * np.pi * np.arange(nv) / nv
    r = 1.0 + 0.1 * g.random(nv)
    return ("polygon", r * np.cos(th), r * np.sin(th), q, m)


def make(ctx, s):
    return ctx.quad_radial(1.0, *s[1:]) if s[0] == "radial" else ctx.quad_polygon(*s[1:])


def reference(s):
    if s[0] == "radial" and s[3] == 0:
        n, (a,), (b,) = s[4], s[1], s[2]  # one harmonic: eq. ptr written out
        t = 2.0 * np.pi * np.arange(1, n + 1) / n
        r, dr = 1.0 + a * np.cos(t) + b * np.sin(t), b * np.cos(t) - a * np.sin(t)
        om = 2.0 * np.pi / n
        return oracle.dilation(r * np.cos(t), r * np.sin(t), om * (dr * np.cos(t) - r * np.sin(t)),
                               om * (dr * np.sin(t) + r * np.cos(t)), s[5])
    return oracle.quad_radial(1.0, *s[1:]) if s[0] == "radial" else oracle.quad_polygon(*s[1:])


# one radial node (as many boundary nodes as areal ones, several batches of
# 256), exactly one block of 2048 and one node more, few and many harmonics,
# the trapezoid rule, the fewest and the most vertices
EDGES = [radial(5, 128, 16, 1, 1), radial(64, 8, 16, 16, 2), radial(64, 3, 683, 1, 3), radial(1, 0, 33, 63, 4),
         radial(0, 4, 16, 333, 5), polygon(3, 2, 3, 6), polygon(128, 16, 1, 7), polygon(17, 5, 241, 8),
         radial(20, 37, 16, 150, 9), radial(3, 1, 1, 5000, 10)]


@pytest.mark.parametrize("count", [len(EDGES), 65, 130])
def test_rules_again_in_one_launch(fh, count):
    shapes = [EDGES[i % len(EDGES)][:-1] + (EDGES[i % len(EDGES)][-1] + i // len(EDGES),) for i in range(count)]
    ctx = fh.Context("mixed")
    n, h = 32, 3.0 / 32
    lams, zs = np.full(count + 1, 5e-7), np.full(count + 1, 2e5)
    out = torch.empty((count + 1, n, n), dtype=ctx.cdtype, device="cuda")
    for change in (0.0, 0.01):  # the second set has the sizes of the first, whose graph may be replayed
        cur = [(s[0], s[1] * (1.0 + change), s[2] * (1.0 + change)) + s[3:] for s in shapes]
        quads = [make(ctx, s) for s in cur]
        made = [[cpu(v).copy() for v in q.export()] for q in quads]
        print(f"rules in one launch: {count} rules, change {change}", flush=True)
        ctx.field_grid_batch_rebuild(quads + quads[:1], lams, zs, n, n, h, h, out=out)  # one rule twice
        for q, s, before in zip(quads, cur, made):
            # the constructor runs the same sums: a few roundings of
            # coordinates of order 1.  The oracle rounds the angle t < 2 pi on
            # its own (two roundings a side, 4 2^-53 2 pi = 2.8e-15), which
            # the k-th harmonic multiplies by k.
            tol = 1e-14
            if s[0] == "radial":
                tol += 2.8e-15 * (np.arange(1, len(s[1]) + 1) * (np.abs(s[1]) + np.abs(s[2]))).sum()
            for a, b, o in zip((cpu(v) for v in q.export()), before, reference(s)):
                assert np.abs(a - b).max() <= 1e-15, s
                assert np.abs(a - o).max() <= tol, s
        for q in quads:
            q.close()
    ctx.close()
