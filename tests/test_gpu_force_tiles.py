"""The force kernels' 64-site workgroups at their edges (fewer sites than one
workgroup, a partly filled last one) and the paired first halves (more sites
than the split stencil takes) against the oracle: one and two flavours, both
signs, accumulating and not, site blocks solved in the kernel and inverted."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, oracle_T_to_blocks, rel_l2, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

TOL = 1e-13  # FP64, the tolerance of the force tests on other lattices


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 2, 2, 34), (10, 10, 18, 28)])
@pytest.mark.parametrize("op", [1, -1, 2])
def test_force(dims, op):
    import torch

    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu force tiles] {dims} op {op}", flush=True)
    nf, sgn = (2, 1) if op == 2 else (1, op)
    U = synth.gauge_links(dims, 0.3, 71)
    o = Oracle(dims, U, KAPPA, CSW, mu=0.05, mubar=MUBAR, epsbar=EPSBAR)
    X, Y = (synth.gaussian_cb_spinor(dims, 72, k, nf) for k in range(2))
    hop = o.hop_force(X, Y, sgn, nf=nf)
    clov = o.clover_force(X, Y, sgn, nf=nf)
    for host_clover in (False, True):
        ctx = tmx.Context(dims)
        ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, MUBAR, EPSBAR, -1))
        ctx.load_gauge(U, 71.0)
        if host_clover:  # general blocks, inverted
            ctx.load_clover(oracle_T_to_blocks(o.T))
        F = torch.full((hop.size,), complex(np.nan, np.nan), dtype=torch.complex128, device="cuda")
        ctx.hop_force(F, to_dev(X), to_dev(Y), op=op)
        assert rel_l2(to_host(F, hop.shape), hop) < TOL
        if not host_clover:
            ctx.clover_force(F, to_dev(X), to_dev(Y), op=op, coeff=-2.0, accumulate=1)
            assert rel_l2(to_host(F, hop.shape), hop - 2.0 * clov) < TOL
            ctx.clover_force(F, to_dev(X), to_dev(Y), op=op)
            assert rel_l2(to_host(F, hop.shape), clov) < TOL
        ctx.close()
