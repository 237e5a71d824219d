"""The weight-gradient kernel (all paths per tile, two groups per workgroup) at
the edges of its range: fewer sites than a tile, tiles that no second group has,
ragged tails, and the size from which one workgroup per CU is used; every layer
shape and loss against the network oracle, and the result independent of the
workgroup count a workspace cap leaves."""
import numpy as np
import pytest

from helpers import CSW, KAPPA, rel_l2, to_dev
from oracle import Oracle
from oracle import nn_oracle as nn
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu


def _setup(dims):
    import paper_2212_06635_amd.tmx as tmx

    U = synth.gauge_links(dims, 0.3, 61)
    ctx = tmx.Context(dims)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, 0.0, 0.0, -1))
    ctx.load_gauge(U, 61.0)
    w = nn.identity_init(np.random.default_rng(62), 0.1).astype(np.float32)
    ctx.pc_set_weights(w)
    bs, xs = (np.stack([synth.gaussian_cb_spinor(dims, s, k) for k in range(2)]) for s in (63, 64))
    return ctx, U, w.astype(np.float64), bs, xs


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 2, 10), (4, 4, 6, 14), (8, 8, 8, 16)])
@pytest.mark.parametrize("loss", [0, 2, 3])
def test_gradient(dims, loss):
    print(f"\n[gpu wgrad] {dims} loss {loss}", flush=True)
    ctx, U, w, bs, xs = _setup(dims)
    o = Oracle(dims, U, KAPPA, CSW, mu=0.05)
    mh = lambda v: o.mhat(v.reshape(-1, 1, 4, 3)).reshape(-1, 4, 3)
    mhd = lambda v: o.mhat(v.reshape(-1, 1, 4, 3), dagger=True).reshape(-1, 4, 3)
    args = (nn.Lattice(dims, U), w, [b[:, 0] for b in bs], [x[:, 0] for x in xs], mh, mhd)
    L, ref = nn.loss_and_grad(*args) if loss == 0 else nn.sym_loss_and_grad(*args, depth=2 if loss == 2 else 1)
    got_l, got = ctx.pc_loss_grad(to_dev(bs), to_dev(xs), 2, loss, 1)
    ctx.close()
    # BF16 activations, weights and links (2^-9 each) through up to nine roundings
    assert abs(got_l - L) / L < 2e-2 and rel_l2(got, ref) < 5e-2


def test_workgroup_count(monkeypatch):
    """With room for 64 partials only, the gradient is the same to the order of the sums."""
    import paper_2212_06635_amd.tmx as tmx

    dims = (8, 8, 8, 16)
    ctx, _, _, bs, xs = _setup(dims)
    _, full = ctx.pc_loss_grad(to_dev(bs), to_dev(xs), 2, 0, 1)
    ctx.close()
    got = 0
    for cap in (30e6, 50e6, 70e6, 90e6, 110e6, 140e6):
        monkeypatch.setenv("TMX_WS_LIMIT", str(int(cap)))
        ctx, _, _, bs, xs = _setup(dims)
        try:
            _, g = ctx.pc_loss_grad(to_dev(bs), to_dev(xs), 2, 0, 1)
            got += 1
            assert rel_l2(g, full) < 1e-5  # FP32 sums of some 10^5 terms in another order
        except tmx.TmxError as e:
            assert e.code == tmx.TMX_ENOMEM and got == 0
        ctx.close()
    assert got >= 3
