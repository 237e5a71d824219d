"""Site data that a captured call has to build (another number of right-hand
sides than the call before it, new parameters, FP16 after a solve only) is built
by the graph: eager calls before and between the replays build their own, and
every replay gives the eager result."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, to_dev
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 8, 8)


@pytest.mark.parametrize("op,prec,nrhs,how", [(1, 0, 3, "rhs"), (1, 2, 2, "solve"), (2, 0, 2, "params"),
                                              (1, 1, 1, "params"), (1, 0, 3, "params")])
def test_captured_build(op, prec, nrhs, how):
    import torch

    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu capture builds] op {op} prec {prec} nrhs {nrhs} after {how}", flush=True)
    kind = 1 if op == 2 else 0
    U = synth.gauge_links(DIMS, 0.3, 51)
    v = to_dev(np.stack([synth.gaussian_cb_spinor(DIMS, 52, k, kind + 1) for k in range(nrhs)]))
    p0, p1 = (tmx.Params(KAPPA, CSW, mu, MUBAR, eb, -1) for mu, eb in ((0.05, EPSBAR), (0.2, 0.2)))
    par = p1 if how == "params" else p0

    # the eager result, from a context of its own
    ref_ctx = tmx.Context(DIMS)
    ref_ctx.set_params(par)
    ref_ctx.load_gauge(U, 1.0)
    src = ref_ctx.pack(v, kind, prec, nrhs)
    ref = ref_ctx.empty(kind, prec, nrhs)
    ref_ctx.apply_mhat(ref, src, op, prec, 0, nrhs)
    torch.cuda.synchronize()

    ctx = tmx.Context(DIMS)
    ctx.set_params(p0)
    ctx.load_gauge(U, 1.0)
    one, out = ctx.empty(kind, prec), ctx.empty(kind, prec, nrhs)
    if how == "solve":
        b = v.reshape(nrhs, -1)[0].contiguous()
        assert ctx.solve(b * 0, b, 1, kind=tmx.TMX_SOLVER_MPCG_F16, op=op)[0] == tmx.TMX_OK
    else:
        ctx.apply_mhat(one, ctx.pack(v.reshape(nrhs, -1)[0].contiguous(), kind, prec), op, prec)
    ctx.set_params(par)
    torch.cuda.synchronize()
    graph, eager = torch.cuda.CUDAGraph(), torch.empty_like(out)
    with torch.cuda.graph(graph):
        ctx.set_stream()
        ctx.apply_mhat_noalloc(out, src, op, prec, 0, nrhs)
    ctx.set_stream()
    # nothing of the graph has run: an eager call finds nothing built
    ctx.apply_mhat(eager, src, op, prec, 0, nrhs)
    torch.cuda.synchronize()
    assert torch.equal(eager, ref)
    for k in range(3):
        out.fill_(0xAB)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref), k
        eager.zero_()
        ctx.apply_mhat(eager, src, op, prec, 0, nrhs)
        torch.cuda.synchronize()
        assert torch.equal(eager, ref), k
    ctx.close()
    ref_ctx.close()
