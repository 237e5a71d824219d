"""A call that does without memory it would have liked reports no error: the
gradient with room for 64 partial sums only, the multishift solve without its
spare fields."""
import numpy as np
import pytest

from helpers import CSW, KAPPA, to_dev
from oracle import nn_oracle as nn
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 8, 16)


@pytest.mark.parametrize("call", ["gradient", "multishift"])
def test_no_error_left_behind(call, monkeypatch):
    import paper_2212_06635_amd.tmx as tmx

    U = synth.gauge_links(DIMS, 0.3, 61)
    bs, xs = (np.stack([synth.gaussian_cb_spinor(DIMS, s, k) for k in range(2)]) for s in (63, 64))
    worked = 0
    for cap in np.geomspace(5e6, 200e6, 24):
        monkeypatch.setenv("TMX_WS_LIMIT", str(int(cap)))
        ctx = tmx.Context(DIMS)
        ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, 0.0, 0.0, -1))
        ctx.load_gauge(U, 61.0)
        ctx.pc_set_weights(nn.identity_init(np.random.default_rng(62), 0.1).astype(np.float32))
        try:
            if call == "gradient":
                ctx.pc_loss_grad(to_dev(bs), to_dev(xs), 2, 0, 1)
            else:
                ctx.multishift_solve(to_dev(np.zeros((6,) + bs[0].shape)), to_dev(bs[0]), np.geomspace(1e-3, 1.0, 6), op=1)
            worked += 1
            assert tmx.lib.tmx_last_error(ctx.h) == b"", int(cap)
        except tmx.TmxError as e:
            assert e.code == tmx.TMX_ENOMEM and worked == 0
        ctx.close()
    assert worked > 3
