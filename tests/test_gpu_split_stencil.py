"""The stencils' split form (four waves per 64 slots, few sites) on lattices
from one partly filled workgroup upwards: every operator, precision and
right-hand-side count against the oracle, and the solvers' fused epilogues."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, oracle_T_to_blocks, rel_l2, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

TOL = {0: 1e-13, 1: 1e-6, 2: 5e-3}  # of the operators in the three storage precisions
RHO = 0.3


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 4, 2, 8), (6, 2, 4, 6), (6, 4, 2, 10), (8, 8, 12, 16)])
@pytest.mark.parametrize("host_clover", [False, True])
def test_operators(dims, host_clover):
    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu split] {dims} host clover {host_clover}", flush=True)
    U = synth.gauge_links(dims, 0.3, 31)
    o = Oracle(dims, U, KAPPA, CSW, mu=0.05, mubar=MUBAR, epsbar=EPSBAR)
    ctx = tmx.Context(dims)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, MUBAR, EPSBAR, -1, RHO))
    ctx.load_gauge(U, 31.0)
    if host_clover:
        ctx.load_clover(oracle_T_to_blocks(o.T))
    for op in (1, -1, 2, 3):
        nf = 2 if op == 2 else 1
        sgn = -1 if op == -1 else 1
        for nrhs in (1, 3):
            v = np.stack([synth.gaussian_cb_spinor(dims, 32, k, nf) for k in range(nrhs)])
            if op == 3:
                ref = {0: [o.w_hat(x, 1, RHO) for x in v], 1: [o.w_hat(x, 1, RHO, dagger=True) for x in v]}
            else:
                ref = {d: [o.mhat(x, nf=nf, sgn=sgn, dagger=bool(d)) for x in v] for d in (0, 1)}
            for prec in (0, 1, 2):
                src = ctx.pack(to_dev(v), nf - 1, prec, nrhs)
                for dag in (0, 1):
                    out = ctx.empty(nf - 1, prec, nrhs)
                    ctx.apply_mhat(out, src, op, prec, dag, nrhs)
                    got = to_host(ctx.unpack(out, nf - 1, prec, nrhs), v.shape)
                    assert rel_l2(got, np.stack(ref[dag])) < TOL[prec], (op, nrhs, prec, dag)
    for kind, op, nf in ((0, 1, 1), (2, -1, 1), (1, 2, 2), (2, 2, 2)):
        b = np.stack([synth.gaussian_cb_spinor(dims, 33, k, nf) for k in range(2)])
        x = to_dev(np.zeros_like(b))
        rc, _ = ctx.solve(x, to_dev(b), 2, kind=kind, op=op, tol=1e-10)
        got = to_host(x, b.shape)
        assert rc == 0
        for k in range(2):
            assert o.residual(b[k], got[k], nf=nf, sgn=-1 if op == -1 else 1) <= 1e-10
    ctx.close()
