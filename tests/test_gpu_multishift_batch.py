"""Batched multishift updates: few and many shifts (more than one launch takes),
iteration counts off the batch length, equal shifts, and workspace caps that
leave no room for the batch; every shift by the oracle's residual."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, to_dev, to_host
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu
DIMS = (4, 6, 4, 8)


@pytest.fixture(scope="module")
def field():
    U = synth.gauge_links(DIMS, 0.3, 8)
    return U, Oracle(DIMS, U, KAPPA, CSW, mu=0.05, mubar=MUBAR, epsbar=EPSBAR)


def _solve(U, o, nf, shifts, inner, **kw):
    import paper_2212_06635_amd.tmx as tmx

    ctx = tmx.Context(DIMS)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, MUBAR, EPSBAR, -1))
    ctx.load_gauge(U, 8.0)
    b = synth.gaussian_cb_spinor(DIMS, 9, 0, nf)
    x = to_dev(np.zeros((len(shifts),) + b.shape))
    try:
        rc, _ = ctx.multishift_solve(x, to_dev(b), shifts, op=2 if nf == 2 else 1, inner_prec=inner, tol=1e-10, **kw)
    finally:
        got = to_host(x, (len(shifts),) + b.shape)
        ctx.close()
    assert rc == 0
    for k, s in enumerate(shifts):
        assert o.residual(b, got[k], nf=nf) > 0 and np.all(np.isfinite(got[k]))
        r = b - o.mdagm(got[k], nf=nf, shift=s)
        assert np.linalg.norm(r) <= 1e-10 * np.linalg.norm(b), (k, s)


@pytest.mark.parametrize("ns", [1, 2, 17, 32])
@pytest.mark.parametrize("nf,inner", [(1, 0), (1, 1), (1, 2), (2, 0), (2, 1), (2, 2)])
@pytest.mark.parametrize("inner_tol", [0.0, 1e-3])  # a stage tolerance of the caller's keeps the stage in its precision
def test_shift_counts(field, ns, nf, inner, inner_tol):
    print(f"\n[gpu multishift batch] ns {ns} nf {nf} inner {inner} inner_tol {inner_tol}", flush=True)
    _solve(*field, nf, np.geomspace(1e-4, 10.0, ns), inner, inner_tol=inner_tol)


@pytest.mark.parametrize("inner", [0, 1, 2])
def test_equal_shifts(field, inner):
    _solve(*field, 1, np.array([0.0, 0.0, 0.01, 0.01, 3.0]), inner)


@pytest.mark.parametrize("inner_tol", [0.0, 1e-3])
def test_caps(field, inner_tol, monkeypatch):
    """From the smallest cap that works upwards, the call works at every cap."""
    import paper_2212_06635_amd.tmx as tmx

    worked = 0
    for cap in range(400_000, 3_000_000, 200_000):
        monkeypatch.setenv("TMX_WS_LIMIT", str(cap))
        try:
            _solve(*field, 1, np.geomspace(1e-3, 1.0, 5), 1, inner_tol=inner_tol)
            worked += 1
        except tmx.TmxError as e:
            assert e.code == tmx.TMX_ENOMEM and worked == 0
    assert worked > 3
