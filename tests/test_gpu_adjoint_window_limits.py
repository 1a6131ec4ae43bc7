"""The adjoint's dense window sums at their limits: a context whose capped
memory holds the transforms' workspace only."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_capped_workspace_falls_back_to_the_transforms(monkeypatch):
    import paper_2010_05978_amd as fh
    # 2 x 32768 outputs: 512 workgroups' windows of some 22 x 47 cells take 25
    # MB, the transforms 7
    n1, n2, lz = 2, 32768, 0.25
    h1, h2 = 4 * lz / 24, 17 * lz / 65536
    monkeypatch.setenv("FH_ALLOC_CAP_BYTES", str(16 << 20))
    ctx = fh.Context("fp64")
    monkeypatch.delenv("FH_ALLOC_CAP_BYTES")
    free = fh.Context("fp64")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    gu = torch.randn((n2, n1), dtype=torch.complex128, device="cuda", generator=g)
    got, want = ([x.cpu().numpy() for x in c.field_grid_vjp(c.quad_radial(1.0, None, None, 0, 60, 40), lz, 1.0, n1, n2,
                                                           h1, h2, gu)] for c in (ctx, free))
    for a, b in zip(got, want):
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        print(f"  capped against free: {err:.1e}", flush=True)
        assert err <= 1e-9
    ctx.close()
    free.close()
