"""FP32 operators read the site-block inverse that was formed in FP64 and
rounded once, in every launch: one right-hand side gives, bit for bit, what it
gives among several (on both sides of the split form's line, and past the line
from which FP64 inverts two-flavour blocks in the kernel)."""
import numpy as np
import pytest

from helpers import CSW, EPSBAR, KAPPA, MUBAR, to_dev
from paper_2212_06635_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(6, 4, 2, 10), (10, 10, 28, 72)])
@pytest.mark.parametrize("op", [1, -1, 2, 3])
def test_same_bits_as_one_of_several(dims, op):
    import torch

    import paper_2212_06635_amd.tmx as tmx

    print(f"\n[gpu f32 blocks] {dims} op {op}", flush=True)
    ctx = tmx.Context(dims)
    ctx.set_params(tmx.Params(KAPPA, CSW, 0.05, MUBAR, EPSBAR, -1, 0.3))
    ctx.load_gauge(synth.gauge_links(dims, 0.3, 31), 31.0)
    kind = 1 if op == 2 else 0
    v = to_dev(np.stack([synth.gaussian_cb_spinor(dims, 32, k, kind + 1) for k in range(2)])).reshape(2, -1)
    one, two = ctx.empty(kind, 1), ctx.empty(kind, 1, 2)
    for dagger in (0, 1):
        ctx.apply_mhat(one, ctx.pack(v[0].contiguous(), kind, 1), op, 1, dagger)
        ctx.apply_mhat(two, ctx.pack(v.reshape(-1), kind, 1, 2), op, 1, dagger, 2)
        assert torch.equal(ctx.unpack(one, kind, 1).reshape(-1), ctx.unpack(two, kind, 1, 2).reshape(2, -1)[0])
    ctx.close()
