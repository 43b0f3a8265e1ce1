"""GPU checks of the VJP's face-state pass with its layers loaded ahead and not
(which one a shell takes depends on its work items: 256 compute units): against
the VJP tile by tile, which has another forward pass (1e-12 per variable), and
the same bits for every chunk length."""
import numpy as np
import pytest
import torch

import coronal_inputs as ci
from helpers import rel_err_per_var

pytestmark = pytest.mark.gpu


# items: 49 x 20 192 (one round, ahead), 49 x 25 480, 65 x 12 450 (two rounds, not ahead), 49 x 120 768 (three, ahead)
@pytest.mark.parametrize("N,Nr,chunks", [(49, 20, (20, 3)), (49, 25, (1, 4, 25)), (65, 12, (2, 12)), (49, 120, (7,))])
def test_vjp_cell_by_cell(N, Nr, chunks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_04481_amd import Context, Grid, Params
    inst = ci.make_instance(N, Nr, "log", lmax=2, seed=60 + N)
    inst.U[8] = 1e-3 * np.random.default_rng(N).standard_normal(inst.ncells)
    ctx = Context(Grid(N, Nr, inst.r_nodes), Params())
    ctx.set_inner_br(torch.from_numpy(inst.br).cuda())
    U = torch.from_numpy(inst.U).cuda()
    w = torch.randn(U.shape, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(4))
    print(f"case: vjp {N} x {Nr}", flush=True)
    march, mbr = ctx.vjp(U, w)
    ref = None
    for kc in (0,) + chunks:
        print(f"case: vjp {N} x {Nr} over its weights, chunks of {kc}", flush=True)
        ctx.set_chunk_layers(kc)
        g = w.clone()
        _, b = ctx.vjp(U, g, out=g)
        if ref is None:
            ref = (g, b)
            assert float(rel_err_per_var(g.cpu(), march.cpu()).max()) <= 1e-12
            assert float(rel_err_per_var(b.cpu()[None], mbr.cpu()[None]).max()) <= 1e-12
        assert torch.equal(g, ref[0]) and torch.equal(b, ref[1]), kc
    assert ctx.status_flags() == 0
