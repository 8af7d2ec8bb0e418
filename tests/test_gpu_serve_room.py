"""Requests run in the smaller workspace give the bits of the full one, and their solves take it as it is."""

import pytest

from gpu_util import needs_gpu, note

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_plain_requests_give_the_same_bits(prec):
    import torch
    from dataclasses import replace
    from paper_1103_6031_amd import mgic, serve
    reqs = [serve.Request(0, 0.0, 96, [((64,) * 3, (30,) * 3)], 2, 0.98), serve.Request(1, 0.0, 64, [], 1, 1.02)]
    fields = serve.device_fields(serve.host_fields(reqs, workers=1))
    ex = serve.GpuExecutor(fields, 1, prec=prec, keep=[0, 1, 10, 11])
    for r in reqs:
        note("serve: request %d, full and plain, %s" % (r.id, prec))
        ex(r, 0)
        ex(replace(r, id=10 + r.id, plain=True), 0)
        for a, b in zip(ex.outputs[r.id], ex.outputs[10 + r.id]):
            for x, y in zip(a, b):
                assert torch.equal(x, y)
        H = serve.hier_of(r)
        if mgic.mg_plain_workspace_bytes(H, ex.opts) < mgic.mg_workspace_bytes(H, ex.opts):
            ws = mgic.Workspace(mgic.mg_plain_workspace_bytes(H, ex.opts))
            assert mgic._solve_ws(ws, H, ex.opts) is ws
