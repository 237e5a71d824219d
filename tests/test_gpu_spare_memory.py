"""Buffers that only make a call faster give way to those a later call cannot
do without, whoever asks for them: under an allocator with a budget that a
multishift solve has used up, a new gauge field, a clover term, the network's
state and a solve of several right-hand sides still find room."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, oracle_T_to_blocks, to_dev, to_host
from oracle import Oracle
from oracle import nn_oracle as nn
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 8, 8)
SHIFTS = np.geomspace(1e-3, 1.0, 8)


class Capped:
    """A context's allocator with a budget in bytes (None: none)."""

    def __init__(self, tmx, ctx):
        import torch

        self.cap, self.live = None, {}

        def alloc(n, user):
            if self.cap is not None and self.bytes() + n > self.cap:
                return None
            t = torch.empty(int(n), dtype=torch.uint8, device="cuda")
            self.live[t.data_ptr()] = t
            return t.data_ptr()

        def release(p, user):
            del self.live[p]

        self.fns = tmx.ALLOC_FN(alloc), tmx.RELEASE_FN(release)
        ctx.check(tmx.lib.tmx_set_allocator(ctx.h, *self.fns, None))

    def bytes(self):
        return sum(t.numel() for t in self.live.values())


def _ctx(tmx, U):
    ctx = tmx.Context(DIMS, allocator="hip")
    A = Capped(tmx, ctx)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, MUBAR, EPSBAR, -1))
    ctx.load_gauge(U, 1.0)
    return ctx, A


def _multishift(ctx, o, inner):
    b = synth.gaussian_cb_spinor(DIMS, 5, 0)
    x = to_dev(np.zeros((len(SHIFTS),) + b.shape))
    rc, _ = ctx.multishift_solve(x, to_dev(b), SHIFTS, op=1, inner_prec=inner)
    assert rc == 0
    got = to_host(x, (len(SHIFTS),) + b.shape)
    for k, s in enumerate(SHIFTS):
        assert np.linalg.norm(b - o.mdagm(got[k], shift=s)) <= 1e-10 * np.linalg.norm(b)


# fields short of what the FP64 stage takes: none, or its last ones (the stage then runs in low precision)
@pytest.mark.parametrize("short", [0, 3])
@pytest.mark.parametrize("inner", [1, 2])
def test_required_buffers_take_the_place_of_spare_ones(short, inner):
    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu spare memory] {short} fields short, inner {inner}", flush=True)
    U, U2 = synth.gauge_links(DIMS, 0.3, 1), synth.gauge_links(DIMS, 0.3, 2)
    par = dict(mu=0.05, mubar=MUBAR, epsbar=EPSBAR)
    o, o2 = Oracle(DIMS, U, KAPPA, CSW, **par), Oracle(DIMS, U2, KAPPA, CSW, **par)
    ctx, A = _ctx(tmx, U)
    _multishift(ctx, o, inner)
    used = A.bytes()
    ctx.close()
    assert not A.live

    ctx, A = _ctx(tmx, U)
    A.cap = used - short * o.Vh * 192
    _multishift(ctx, o, inner)
    ctx.load_gauge(U2, 2.0)
    ctx.load_clover(oracle_T_to_blocks(o2.T))
    assert ctx.get_clover().shape == (o2.V, 2, 6, 6)
    ctx.load_clover(None)
    b = np.stack([synth.gaussian_cb_spinor(DIMS, 6, k) for k in range(2)])
    x = to_dev(np.zeros_like(b))
    rc, _ = ctx.solve(x, to_dev(b), 2, kind=tmx.TMX_SOLVER_CG, op=1)
    got = to_host(x, b.shape)
    assert rc == 0 and all(o2.residual(b[k], got[k]) <= 1e-10 for k in range(2))
    ctx.pc_set_weights(nn.identity_init(np.random.default_rng(3), 1e-2))
    assert A.bytes() <= A.cap
    # and back: the spare buffers fit again or the call does without them
    ctx.load_gauge(U, 3.0)
    _multishift(ctx, o, inner)
    ctx.close()
    assert not A.live
