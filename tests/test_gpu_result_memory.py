"""GPU checks of what calls leave in the caller's memory: a result written over
an input, and the solution of a solve that fails."""
import numpy as np
import pytest
import torch

import coronal_inputs as ci

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def shell(N, Nr, seed=77):
    from paper_2209_04481_amd import Context, Grid, Params
    inst = ci.make_instance(N, Nr, "log", lmax=2, seed=seed)
    inst.U[8] = 1e-3 * np.random.default_rng(seed).standard_normal(inst.ncells)
    ctx = Context(Grid(N, Nr, inst.r_nodes), Params())
    ctx.set_inner_br(torch.from_numpy(inst.br).cuda())
    return ctx, torch.from_numpy(inst.U).cuda()


# one tile and several (14 x 14 columns), one chunk of layers and many
@pytest.mark.parametrize("N,Nr", [(2, 1), (8, 9), (15, 40), (31, 30)])
def test_local_dt_over_the_state_it_reads(N, Nr):
    """The diagonal written over the state's own rows (or across two of them)
    has the bits of one written apart, and touches nothing else."""
    ctx, U = shell(N, Nr)
    nc = U.shape[1]
    ref = ctx.local_dt(U, 2.0)
    for at in (0, 4 * nc, 8 * nc, 3 * nc + nc // 2):
        print(f"case: local_dt {N} x {Nr} over entry {at}", flush=True)
        V = U.clone()
        got = ctx.local_dt(V, 2.0, out=V.view(-1)[at:at + nc]).clone()
        assert torch.equal(got, ref), at
        V.view(-1)[at:at + nc] = U.view(-1)[at:at + nc]
        assert torch.equal(V, U), at
