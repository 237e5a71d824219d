"""What the allocation-free Schur operator finds resident: after any call that
prepared a precision and sector it gives tmx_apply_mhat's result bit for bit,
without a device allocation -- for another number of right-hand sides, after a
solve only, with a clover term given later, and after parameters under which
the site blocks are no longer inverted in the kernel."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, oracle_T_to_blocks, to_dev
from oracle import Oracle
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu


def _ctx(tmx, dims, mubar=MUBAR, epsbar=EPSBAR):
    ctx = tmx.Context(dims, allocator="torch")
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, mubar, epsbar, -1))
    ctx.load_gauge(synth.gauge_links(dims, 0.3, 41), 41.0)
    return ctx


def _field(ctx, dims, op, prec, nrhs):
    kind = 1 if op == 2 else 0
    v = np.stack([synth.gaussian_cb_spinor(dims, 42, k, kind + 1) for k in range(nrhs)])
    return ctx.pack(to_dev(v), kind, prec, nrhs), ctx.empty(kind, prec, nrhs)


def _check(ctx, dims, op, prec, nrhs):
    import torch

    src, got = _field(ctx, dims, op, prec, nrhs)
    n = ctx.allocator.n_alloc
    ctx.apply_mhat_noalloc(got, src, op, prec, 0, nrhs)
    assert ctx.allocator.n_alloc == n
    ref = torch.empty_like(got)
    ctx.apply_mhat(ref, src, op, prec, 0, nrhs)
    assert torch.equal(got, ref), (dims, op, prec, nrhs)


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (16, 16, 16, 32)])
@pytest.mark.parametrize("op,prec", [(1, 0), (1, 1), (1, 2), (2, 0), (2, 1)])
def test_after_one_right_hand_side(dims, op, prec):
    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu no-alloc resident] {dims} op {op} prec {prec}", flush=True)
    ctx = _ctx(tmx, dims)
    src, out = _field(ctx, dims, op, prec, 1)
    ctx.apply_mhat(out, src, op, prec)
    _check(ctx, dims, op, prec, 2 if dims[0] == 16 else 3)
    ctx.close()


@pytest.mark.parametrize("op", [1, 2])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_after_a_solve(op, nrhs):
    import paper_2212_06635_amd.tmx as tmx

    dims = (8, 8, 8, 8)
    print(f"\n[gpu no-alloc resident] after an FP16 solve, op {op} nrhs {nrhs}", flush=True)
    ctx = _ctx(tmx, dims)
    b = to_dev(synth.gaussian_cb_spinor(dims, 43, 0, 2 if op == 2 else 1))
    rc, _ = ctx.solve(b * 0, b, 1, kind=tmx.TMX_SOLVER_MPCG_F16, op=op)
    assert rc == tmx.TMX_OK
    _check(ctx, dims, op, 2, nrhs)
    ctx.close()


@pytest.mark.parametrize("op,prec", [(1, 0), (1, 2), (2, 0)])
@pytest.mark.parametrize("solve", [False, True])
def test_after_a_clover_term_of_the_callers(op, prec, solve):
    import paper_2212_06635_amd.tmx as tmx

    dims = (8, 8, 8, 8)
    print(f"\n[gpu no-alloc resident] load_clover, op {op} prec {prec} solve {solve}", flush=True)
    ctx = _ctx(tmx, dims)
    if solve:
        b = to_dev(synth.gaussian_cb_spinor(dims, 43, 0, 2 if op == 2 else 1))
        assert ctx.solve(b * 0, b, 1, kind=tmx.TMX_SOLVER_MPCG_F16 if prec == 2 else tmx.TMX_SOLVER_CG, op=op)[0] == 0
    else:
        src, out = _field(ctx, dims, op, prec, 1)
        ctx.apply_mhat(out, src, op, prec)
    T = oracle_T_to_blocks(Oracle(dims, synth.gauge_links(dims, 0.3, 44), KAPPA, CSW).T)
    ctx.load_clover(T)
    _check(ctx, dims, op, prec, 1)
    ctx.load_clover(None)
    _check(ctx, dims, op, prec, 2)
    ctx.close()


def test_after_parameters_that_need_the_inverse():
    import paper_2212_06635_amd.tmx as tmx

    dims = (10, 10, 28, 72)  # two-flavour blocks inverted in the kernel while mubar <= epsbar
    print(f"\n[gpu no-alloc resident] new parameters {dims}", flush=True)
    ctx = _ctx(tmx, dims)
    src, out = _field(ctx, dims, 2, 0, 1)
    ctx.apply_mhat(out, src, 2, 0)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, 0.2, 0.1, -1))
    _check(ctx, dims, 2, 0, 1)
    ctx.close()
