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


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("bad", ["rhs", "state", "diagonal"])
def test_a_solve_that_fails_leaves_the_zero_it_starts_from(bad, transpose):
    """A NaN in the right-hand side, the state or the diagonal ends the solve
    in its first cycle: x is then zero, whatever the memory held."""
    from paper_2209_04481_amd.binding import CfvNonPhysical
    ctx, U = shell(4, 6)
    b = torch.randn(U.shape, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    D = ctx.local_dt(U, 2.0)
    {"rhs": b, "state": U, "diagonal": D}[bad].view(-1)[11] = float("nan")
    x = torch.full_like(U, 7.0)
    print(f"case: solve 4 x 6, NaN in the {bad}, transpose {transpose}", flush=True)
    with pytest.raises(CfvNonPhysical):
        ctx.solve(U, D, b, transpose=transpose, m=5, max_restarts=1, out=x)
    assert not bool(x.any())
    # and the context solves again
    ctx2, U2 = shell(4, 6)
    b2 = torch.ones_like(U2)
    y, hist = ctx.solve(U2, ctx2.local_dt(U2, 2.0), b2, transpose=transpose, m=5)
    assert bool(torch.isfinite(y).all()) and len(hist) == 5
