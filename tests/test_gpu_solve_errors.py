"""A solve that ends in an error leaves nothing on its stream (a mixed-precision
one enqueues iterations ahead and may then lack the workspace of its first
reliable update): the context can go on at once on another stream."""
import numpy as np
import pytest

from helpers import CSW, KAPPA, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (16, 16, 16, 16)


@pytest.mark.parametrize("kind", [1, 2])
def test_stream_is_drained(kind, monkeypatch):
    import torch

    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu solve errors] kind {kind}", flush=True)
    U = synth.gauge_links(DIMS, 0.3, 3)
    o = Oracle(DIMS, U, KAPPA, CSW, mu=0.05)
    b = synth.gaussian_cb_spinor(DIMS, 6, 0)
    x, db = to_dev(np.zeros_like(b)), to_dev(b)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    field = o.Vh * 24 * 8  # one FP64 odd field
    # the largest cap that fails: the iterations run, the first reliable update has no room
    for cap in range(12 * field, 4 * field, -field // 8):
        monkeypatch.setenv("TMX_WS_LIMIT", str(cap))
        ctx = tmx.Context(DIMS, stream=s1.cuda_stream)
        ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, 0.0, 0.0, -1))
        ctx.load_gauge(U, 1.0)
        torch.cuda.synchronize()
        try:
            assert ctx.solve(x, db, 1, kind=kind, op=1)[0] == tmx.TMX_OK
            code = 0
        except tmx.TmxError as e:
            idle, code = s1.query(), e.code
            ctx.set_stream(s2.cuda_stream)
        ctx.close()
        if code:
            break
    assert cap < 12 * field and code == tmx.TMX_ENOMEM and idle
    monkeypatch.delenv("TMX_WS_LIMIT")
    # a non-finite residual (a NaN among the links), then a good field on another stream
    bad = U.copy()
    bad.reshape(-1)[5] = np.nan
    ctx = tmx.Context(DIMS, stream=s1.cuda_stream)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, 0.0, 0.0, -1))
    ctx.load_gauge(bad, 10.0)
    rc, _ = ctx.solve(x, db, 1, kind=kind, op=1)
    idle = s1.query()
    assert rc == tmx.TMX_ENOCONV and idle
    ctx.set_stream(s2.cuda_stream)
    ctx.load_gauge(U, 20.0)
    rc, _ = ctx.solve(x, db, 1, kind=kind, op=1)
    assert rc == tmx.TMX_OK and o.residual(b, to_host(x, b.shape)) <= 1e-10
    ctx.close()
