"""Two-flavour site blocks whose A^2 + nubar^2 - epsbar^2 is not positive, in
every form of their inverse (stored, or eliminated in the kernel) against the
oracle.  The lattice repeats a small one chosen so that no block is close to
singular: the bounds stay small, and a wrong block cannot hide."""
import numpy as np
import pytest

from helpers import KAPPA, rel_l2, tile_cb, tile_links, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

BASE = (2, 2, 2, 4)
U = {0: 2.0 ** -53, 1: 2.0 ** -24}  # unit roundoff per precision


@pytest.mark.parametrize("rep", [(1, 1, 1), (28, 28, 8)])  # 16 sites a parity; 100352, past the in-kernel form's line
@pytest.mark.parametrize("eps,csw,mubar,epsbar,seed", [(2.0, 8.0, 0.1, 0.3, 174), (0.6, 1.69, 0.0, 3.0, 169),
                                                       (1.0, 5.0, 0.05, 0.3, 241)])
def test_against_oracle(rep, eps, csw, mubar, epsbar, seed):
    import paper_2212_06635_amd.tmx as tmx

    dims = (BASE[0] * rep[0], BASE[1] * rep[1], BASE[2] * rep[2], BASE[3])
    print(f"\n[gpu indefinite blocks] {dims} eps {eps} csw {csw} mubar {mubar} epsbar {epsbar}", flush=True)
    links = synth.gauge_links(BASE, eps, seed)
    o = Oracle(BASE, links, KAPPA, csw, mubar=mubar, epsbar=epsbar)
    even = np.setdiff1d(np.arange(o.V), synth.odd_sites(BASE, 1))
    A = np.stack([o.T[even][:, 6 * c:6 * c + 6, 6 * c:6 * c + 6] for c in (0, 1)], 1).reshape(-1, 6, 6) + np.eye(6)
    ev = np.abs(np.linalg.eigvalsh(A))
    d = 2 * KAPPA * np.sqrt(epsbar ** 2 - mubar ** 2)
    assert (ev < d).any(1).sum() >= 5  # blocks of either sign
    # the worst condition number of the factors A -+ del; of their product
    # where that is inverted as a whole
    cond = ((ev.max(1) + d) / np.abs(ev - d).min(1)).max()
    ctx = tmx.Context(dims)
    ctx.set_params(tmx.Params(KAPPA, csw, 0.0, mubar, epsbar, -1))
    ctx.load_gauge(tile_links(links, rep), 27.0)
    v0 = [synth.gaussian_cb_spinor(BASE, 28, k, 2) for k in range(2)]
    v = np.stack([tile_cb(x, BASE, rep) for x in v0])
    for dagger in (0, 1):
        ref = np.stack([tile_cb(o.mhat(x, nf=2, dagger=bool(dagger)), BASE, rep) for x in v0])
        for prec in (0, 1):
            for nrhs in (1, 2):
                src = ctx.pack(to_dev(v[:nrhs]), 1, prec, nrhs)
                out = ctx.empty(1, prec, nrhs)
                ctx.apply_mhat(out, src, 2, prec, dagger, nrhs)
                got = to_host(ctx.unpack(out, 1, prec, nrhs), v[:nrhs].shape)
                whole = prec == 0 and (nrhs > 1 or rep[0] == 1)
                tol = 20 * U[prec] * cond ** (2 if whole else 1)
                assert tol < 1e-3
                assert rel_l2(got, ref[:nrhs]) < tol, (prec, dagger, nrhs, rel_l2(got, ref[:nrhs]), tol)
    ctx.close()
