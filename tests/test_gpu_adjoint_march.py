"""GPU checks of the VJP tile by tile where panels end in tiles one or two
columns wide (whose idle lanes repeat a column), and of chunks of several
layers and shells of one: each call is first shown to take that path, by the
kernels it records.  Against the oracle's reverse mode and against the same
call written over its weights (which goes cell by cell): 1e-12 per variable."""
import numpy as np
import pytest
import torch

import coronal_inputs as ci
from helpers import rel_err_per_var
from oracle import mhd, solve
from oracle.grid import Grid as OGrid

pytestmark = pytest.mark.gpu

# 4: one layer; 12, 16: partial and whole tiles, chunks of two layers; 17, 33: a last column of one; 18, 34: of two
CASES = [(4, 1, 0), (12, 60, 1), (16, 60, 0), (17, 8, 0), (17, 20, 1), (18, 8, 1), (18, 20, 0), (33, 8, 0), (34, 8, 1)]


def kernels(ctx, f):
    ctx.timing_enable(True)
    out = f()
    names = set(ctx.timing_read())
    ctx.timing_enable(False)
    return out, names


def problem(N, Nr, inner):
    from paper_2209_04481_amd import Context, Grid, Params
    inst = ci.make_instance(N, Nr, "log", lmax=2, seed=1400 + N + Nr)
    inst.U[8] = 1e-3 * np.random.default_rng(N + Nr).standard_normal(inst.ncells)   # psi != 0
    bth = torch.from_numpy(ci.btheta_map(N))
    ctx = Context(Grid(N, Nr, inst.r_nodes), Params(inner_mode=inner))
    ctx.set_inner_br(torch.from_numpy(inst.br).cuda())
    ctx.set_inner_btheta(bth.cuda())
    w = torch.from_numpy(np.random.default_rng(6).standard_normal(inst.U.shape))
    return inst, bth, ctx, w


def both_paths(ctx, U, w):
    Ud, wd = U.cuda(), w.cuda()
    (gU, gbr), names = kernels(ctx, lambda: ctx.vjp(Ud, wd))
    assert "adjoint_finish" in names and "adjoint_gather" not in names
    over = wd.clone()
    (_, b2), names = kernels(ctx, lambda: ctx.vjp(Ud, over, out=over))
    assert "adjoint_gather" in names and "adjoint_finish" not in names
    return [(gU.cpu(), gbr.cpu()), (over.cpu(), b2.cpu())]


@pytest.mark.parametrize("N,Nr,inner", CASES)
def test_vjp_by_the_march(N, Nr, inner):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case: vjp {N} x {Nr}, inner {inner}", flush=True)
    inst, bth, ctx, w = problem(N, Nr, inner)
    U, br = torch.from_numpy(inst.U), torch.from_numpy(inst.br)
    og, op = OGrid(N, Nr, inst.r_nodes), mhd.Params(inner_mode=inner, inner_btheta=bth)
    ro, bo = solve.vjp(og, U, br, op, w)
    for g, b in both_paths(ctx, U, w):
        assert float(rel_err_per_var(g, ro).max()) <= 1e-12
        assert float(rel_err_per_var(b[None], bo[None]).max()) <= 1e-12


# beyond the oracle's sizes: a second round of items that leaves compute units idle, narrow last tiles
@pytest.mark.parametrize("N,Nr", [(49, 20), (50, 20), (65, 12)])
def test_narrow_tiles_in_a_second_round(N, Nr):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case: vjp {N} x {Nr}", flush=True)
    inst, _, ctx, w = problem(N, Nr, 0)
    (gU, gbr), (over, b2) = both_paths(ctx, torch.from_numpy(inst.U), w)
    assert float(rel_err_per_var(gU, over).max()) <= 1e-12
    assert float(rel_err_per_var(gbr[None], b2[None]).max()) <= 1e-12
