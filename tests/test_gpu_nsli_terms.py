"""The edge integral's terms where their evaluation could go wrong: phases at
the ends of the reduced interval, targets on and almost on a node, with and
without the deep-shadow sums, in one and in several node groups."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 200])
@pytest.mark.parametrize("far", [0.0, 0.05])
def test_terms_at_the_ends_of_the_phase(n, far):
    import paper_2010_05978_amd as fh
    ctx = fh.Context("fp64")
    lz = 0.1
    t = 2.0 * np.pi * np.arange(n) / n
    X, Y = np.cos(t), np.sin(t)
    W, V = -np.sin(t) * (2 * np.pi / n), np.cos(t) * (2 * np.pi / n)
    # distances from node 0 whose phase t = r^2/(2 lz) is k/4 of a turn, and
    # one rounding to either side; on the node; as near as 1e-3 ... 1e-160
    r = np.sqrt(2.0 * lz * 0.25 * np.arange(1, 41))
    r = np.concatenate([r, np.nextafter(r, 9), np.nextafter(r, 0), [0.0], 10.0 ** -np.arange(3.0, 161.0, 12.0)])
    xi, eta = 1.0 + np.concatenate([r, 0 * r]), np.concatenate([0 * r, r])
    B = torch.tensor(np.stack([X, Y, W, V]), device="cuda")
    print(f"edge-integral terms: n = {n}, far = {far}", flush=True)
    u = ctx.field_nsli(B, 1.0, lz, torch.tensor(xi, device="cuda"), torch.tensor(eta, device="cuda"), far=far)
    ref = oracle.nsli(X, Y, W, V, 1.0, lz, xi, eta, far=far)
    # each term |1 - e| |r x ds|/r^2/(2 pi) <= min(2/r, pi r/lz) |ds|/(2 pi) < 1 here and carries the rounding of
    # its phase (up to 13 turns: 2 pi 13 2^-53) and of about ten operations; the oracle's carry the same
    assert np.abs(u.cpu().numpy() - ref).max() <= 4e-14
    ctx.close()
