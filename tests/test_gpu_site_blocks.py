"""Site blocks inverted inside K1 (structured clover blocks): the eliminated
blocks against the oracle on smooth fields (no pivoting anywhere) and on rough
ones (some or all blocks indefinite, so their threads pivot)."""
import numpy as np
import pytest

from helpers import KAPPA, rel_l2, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

U = {0: 2.0 ** -53, 1: 2.0 ** -24}  # unit roundoff per precision


def _pivots_ok(A):
    """Whether elimination on the Hermitian block A keeps every pivot at 1/8 or more."""
    A = A.copy()
    for k in range(6):
        if not A[k, k].real >= 0.125:
            return False
        for i in range(k + 1, 6):
            A[i, k + 1:] -= A[i, k] / A[k, k] * A[k, k + 1:]
    return True


@pytest.mark.parametrize("dims,eps,csw,rough", [((8, 8, 8, 8), 0.3, 1.69, False), ((6, 4, 2, 10), 0.3, 1.0, False),
                                                ((6, 4, 2, 10), 2.0, 8.0, True), ((2, 2, 2, 2), 2.0, 8.0, True)])
@pytest.mark.parametrize("sgn,mu", [(1, 0.05), (-1, 0.2)])
def test_eliminated_blocks(dims, eps, csw, rough, sgn, mu):
    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu site blocks] {dims} eps {eps} csw {csw} sgn {sgn}", flush=True)
    links = synth.gauge_links(dims, eps, 17)
    o = Oracle(dims, links, KAPPA, csw, mu=mu)
    even = np.setdiff1d(np.arange(o.V), synth.odd_sites(dims, 1))
    A = np.stack([o.T[even][:, 6 * c:6 * c + 6, 6 * c:6 * c + 6] for c in (0, 1)], 1).reshape(-1, 6, 6) + np.eye(6)
    fast = np.array([_pivots_ok(a) for a in A])
    assert fast.all() != rough
    # elimination's error: the blocks' condition number times the roundoff (a
    # small multiple for the sums over neighbours and the products' length)
    cond = np.linalg.cond(A + 2j * KAPPA * mu * np.eye(6)).max()
    ctx = tmx.Context(dims)
    ctx.set_params(tmx.Params(KAPPA, csw, mu, 0.0, 0.0, -1))
    ctx.load_gauge(links, 17.0)
    v = synth.gaussian_cb_spinor(dims, 18, 0)
    ref = o.mhat(v, sgn=sgn)
    for prec in (0, 1):
        src = ctx.pack(to_dev(v), 0, prec)
        out = ctx.empty(0, prec)
        ctx.apply_mhat(out, src, sgn, prec)
        got = to_host(ctx.unpack(out, 0, prec), v.shape)
        tol = 20 * U[prec] * cond
        assert rel_l2(got, ref) < tol, (prec, rel_l2(got, ref), tol)
    ctx.close()
