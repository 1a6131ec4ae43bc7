"""The direct sum's second limit: many nodes on few outputs, where it would
stage more than it multiplies, keep the transform, and its FP32 sums are as
accurate as the transform's on the side it takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LZ = 0.25


@pytest.fixture(scope="module")
def fh():
    import paper_2010_05978_amd as fh
    return fh


def tiled(fh, prec, **kw):
    return fh.Context(prec, options=fh.fh_options(sigma=0, kernel_width=0, beta=0.0, tile=0, max_subproblem=0,
                                                  spread_method=2, deterministic=0), **kw)


def lit(q):
    x, y, _ = (torch.as_tensor(v, device="cuda") for v in q.export())
    q.set_illumination(torch.polar(1.0 + 0.1 * x, 0.3 * y), 3.0)


# (outputs, rays of 100 nodes, lit, direct): the kernel truncation of the
# transform (1e-11 and more on these grids) tells the two apart, whose rounding
# agrees to 1e-13
@pytest.mark.parametrize("n1,n2,rays,src,direct", [
    (16, 16, 1000, False, True), (16, 16, 1050, False, False), (16, 16, 600, True, True), (16, 16, 700, True, False),
    (16, 16, 3900, False, False), (2, 400, 140, False, True), (2, 400, 150, False, False), (400, 2, 140, False, True),
    (400, 2, 150, False, False)])
def test_path_by_staged_work(fh, n1, n2, rays, src, direct):
    ctx, other = fh.Context("fp64"), tiled(fh, "fp64")
    q = ctx.quad_radial(1.0, [0.05], [0.1], 0, rays, 100)
    if src:
        lit(q)
    h = 0.01
    u, v = (c.field_grid(q, LZ, 1.0, n1, n2, h, h) for c in (ctx, other))
    d = float((u - v).norm() / v.norm())
    print(f"  {n1} x {n2}, {q.N} nodes, lit {src}: {d:.1e}", flush=True)
    assert (d > 2e-12) == direct
    ctx.close()
    other.close()


@pytest.mark.parametrize("n1,n2", [(2, 2), (4, 4), (16, 16), (2, 40)])
@pytest.mark.parametrize("rays", [40, 200, 400, 680, 1000, 4000])
def test_fp32_sums_are_as_accurate(fh, n1, n2, rays):
    exact, ctx, other = tiled(fh, "fp64", tol=1e-13), fh.Context("mixed"), tiled(fh, "mixed")
    q = ctx.quad_radial(1.0, [0.05], [0.1], 0, rays, 100)
    # eight calls at different wavelengths: the root mean square of their errors
    lzs = LZ * np.linspace(0.8, 1.2, 8)
    ms = {}
    for name, c in (("call", ctx), ("transform", other)):
        e = []
        for lz in lzs:
            want = exact.field_grid(q, lz, 1.0, n1, n2, 0.01, 0.01)
            e.append(float((c.field_grid(q, lz, 1.0, n1, n2, 0.01, 0.01).to(want.dtype) - want).norm() / want.norm()))
        ms[name] = float(np.sqrt(np.mean(np.square(e))))
    print(f"  {n1} x {n2}, {q.N} nodes: {ms['call']:.2e}, transform {ms['transform']:.2e}", flush=True)
    assert ms["call"] <= 1.25 * ms["transform"]
    for c in (exact, ctx, other):
        c.close()
