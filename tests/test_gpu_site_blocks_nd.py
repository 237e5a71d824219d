"""Two-flavour site blocks inverted inside K1 (many sites, nubar <= epsbar)
against the oracle: smooth fields, rough ones whose blocks need pivoting, a
shift large enough to bring the pivots of A - del below the bound, and the
stored inverse on the other side of the rule; the paired first halves of the
force with them."""
import numpy as np
import pytest

from helpers import KAPPA, rel_l2, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (10, 10, 28, 72)  # 100800 sites a parity: past the line, not a multiple of 64
U = {0: 2.0 ** -53, 1: 2.0 ** -24}  # unit roundoff per precision


@pytest.mark.parametrize("eps,csw,mubar,epsbar", [(0.3, 1.69, 0.1246, 0.1315), (0.3, 1.69, 0.2, 0.2),
                                                  (2.0, 8.0, 0.1, 0.3), (0.3, 1.0, 0.0, 3.3),
                                                  (0.3, 1.69, 0.2, 0.1)])
def test_two_flavour_blocks(eps, csw, mubar, epsbar):
    import torch

    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu nd site blocks] eps {eps} csw {csw} mubar {mubar} epsbar {epsbar}", flush=True)
    links = synth.gauge_links(DIMS, eps, 27)
    o = Oracle(DIMS, links, KAPPA, csw, mubar=mubar, epsbar=epsbar)
    even = np.setdiff1d(np.arange(o.V), synth.odd_sites(DIMS, 1))
    A = np.stack([o.T[even][:, 6 * c:6 * c + 6, 6 * c:6 * c + 6] for c in (0, 1)], 1).reshape(-1, 6, 6) + np.eye(6)
    ev = np.linalg.eigvalsh(A)
    sq = (2 * KAPPA) ** 2 * (epsbar ** 2 - mubar ** 2)
    d = np.sqrt(abs(sq))
    # elimination's error: the condition number of the worse of the factors
    # A -+ del (of A^2 + nubar^2 - epsbar^2 where that is inverted as a whole),
    # times the roundoff and a small multiple
    gap = np.abs(np.abs(ev) - d).min(1) if sq >= 0 else np.sqrt(ev ** 2 + d ** 2).min(1)
    cond = ((np.abs(ev).max(1) + d) / gap).max() ** (1 if sq >= 0 else 2)
    ctx = tmx.Context(DIMS)
    ctx.set_params(tmx.Params(KAPPA, csw, 0.0, mubar, epsbar, -1))
    ctx.load_gauge(links, 27.0)
    v = synth.gaussian_cb_spinor(DIMS, 28, 0, 2)
    for dagger in (0, 1):
        ref = o.mhat(v, nf=2, dagger=bool(dagger))
        for prec in (0, 1):
            src = ctx.pack(to_dev(v), 1, prec)
            out = ctx.empty(1, prec)
            ctx.apply_mhat(out, src, 2, prec, dagger)
            got = to_host(ctx.unpack(out, 1, prec), v.shape)
            tol = 20 * U[prec] * cond
            assert rel_l2(got, ref) < tol, (prec, dagger, rel_l2(got, ref), tol)
    if csw == 1.69:
        w = synth.gaussian_cb_spinor(DIMS, 28, 1, 2)
        hop = o.hop_force(v, w, nf=2)
        F = torch.full((hop.size,), complex(np.nan, np.nan), dtype=torch.complex128, device="cuda")
        ctx.hop_force(F, to_dev(v), to_dev(w), op=2)
        assert rel_l2(to_host(F, hop.shape), hop) < 200 * U[0] * cond
    ctx.close()
