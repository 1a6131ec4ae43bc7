"""Every node of every rule is written by the launch that computes a batch's
rules again: nodes and weights are overwritten with NaN first, so that a block
or a rule left out shows, in the rules and in the batch's fields."""
import numpy as np
import pytest

from test_gpu_rule_batches import EDGES, cpu, make

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class _DeviceArray:
    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<f8", "data": (ptr, False), "version": 3}


@pytest.mark.parametrize("count", [len(EDGES), 64, 65, 130])
def test_every_node_is_written(count):
    import paper_2010_05978_amd as fh
    ctx = fh.Context("mixed")
    shapes = [EDGES[i % len(EDGES)][:-1] + (EDGES[i % len(EDGES)][-1] + i // len(EDGES),) for i in range(count)]
    quads = [make(ctx, s) for s in shapes]
    n, h = 32, 3.0 / 32
    lams, zs = np.full(count, 5e-7), np.full(count, 2e5)
    made = [[cpu(v).copy() for v in q.export()] for q in quads]
    fields = ctx.field_grid_batch(quads, lams, zs, n, n, h, h)
    for rep in range(2):
        for q in quads:
            for p in fh._binding.fh_quad_device_ptrs(q.handle):
                torch.as_tensor(_DeviceArray(p, q.N), device="cuda").fill_(float("nan"))
        torch.cuda.synchronize()
        u = ctx.field_grid_batch_rebuild(quads, lams, zs, n, n, h, h)
        for q, s, before in zip(quads, shapes, made):
            for a, b in zip((cpu(v) for v in q.export()), before):
                assert np.abs(a - b).max() <= 1e-15, s  # (NaN fails)
        # each field to the context's tolerance twice
        err = ((u - fields).flatten(1).norm(dim=1) / fields.flatten(1).norm(dim=1)).max()
        print(f"rules overwritten: {count} rules, fields differ by {float(err):.1e}", flush=True)
        assert float(err) <= 2e-5
    ctx.close()
