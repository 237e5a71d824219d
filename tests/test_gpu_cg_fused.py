"""CG with the residual update inside the operator's last kernel: around the
size where the per-slot norms are summed in one pass (8192 sites of one parity)
and with columns that converge at different times, start converged or are zero;
every column accepted by the oracle's residual."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (16, 16, 8, 8), (16, 16, 8, 10)])
@pytest.mark.parametrize("nf,kind", [(1, 0), (1, 1), (1, 2), (2, 0), (2, 1)])
def test_columns(dims, nf, kind):
    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu fused cg] {dims} nf {nf} kind {kind}", flush=True)
    U = synth.gauge_links(dims, 0.3, 5)
    o = Oracle(dims, U, KAPPA, CSW, mu=0.05, mubar=MUBAR, epsbar=EPSBAR)
    ctx = tmx.Context(dims)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, MUBAR, EPSBAR, -1))
    ctx.load_gauge(U, 5.0)
    b = np.stack([synth.gaussian_cb_spinor(dims, 6, k, nf) for k in range(3)])
    b[1] = 0.0  # solved by zero
    op = 2 if nf == 2 else 1
    x = to_dev(np.zeros_like(b))
    rc, _ = ctx.solve(x, to_dev(b), 3, kind=kind, op=op, tol=1e-10)
    got = to_host(x, b.shape)
    assert rc == 0 and not np.any(got[1])
    assert o.residual(b[0], got[0], nf=nf) <= 1e-10 and o.residual(b[2], got[2], nf=nf) <= 1e-10
    # column 0 starts converged, column 2 from zero
    guess = got.copy()
    guess[2] = 0.0
    x = to_dev(guess)
    rc, info = ctx.solve(x, to_dev(b), 3, kind=kind, op=op, tol=1e-10, use_initial_guess=1)
    got = to_host(x, b.shape)
    assert rc == 0 and info[0]["iters"] == 0 and info[2]["iters"] > 0
    assert o.residual(b[0], got[0], nf=nf) <= 1e-10 and o.residual(b[2], got[2], nf=nf) <= 1e-10
    ctx.close()
