"""GPU checks of the Arnoldi kernels at the sizes where their blocking can go
wrong: vectors shorter than one tile (1,024 entries) and of an odd number of
pairs per tile, several tiles and rounds per block, one and many groups of
basis vectors, and a Krylov space beyond what the lockstep least-squares
kernel keeps in LDS (64 columns).  Against the oracle's GMRES (modified
Gram-Schmidt in plain float64)."""
import numpy as np
import pytest
import torch

import coronal_inputs as ci
from helpers import rel_err_per_var
from oracle import mhd, solve
from oracle.grid import Grid as OGrid

pytestmark = pytest.mark.gpu

# (N, Nr, m): 216 entries (a fifth of a tile); 1,134 (a tile and a remainder); 24,192; 6,912 with m > 64
CASES = [(2, 1, 8), (3, 7, 30), (8, 7, 30), (4, 8, 70)]


def inputs():
    insts = [ci.make_instance(N, Nr, "log", lmax=2, seed=900 + q) for q, (N, Nr, _) in enumerate(CASES)]
    for i in insts:  # a nonzero cleaning variable: no limiter sits on its kink
        i.U[8] = 1e-3 * np.random.default_rng(i.seed).standard_normal(i.ncells)
    return insts


def context(inst):
    from paper_2209_04481_amd import Context, Grid, Params
    c = Context(Grid(inst.N, inst.Nr, inst.r_nodes), Params())
    c.set_inner_br(torch.from_numpy(inst.br).cuda())
    return c


def oracle_step(inst, m, jacobi):
    og = OGrid(inst.N, inst.Nr, inst.r_nodes)
    U = torch.from_numpy(inst.U)
    Un, hist, _ = solve.be_step(og, U, torch.from_numpy(inst.br), mhd.Params(), 1e3, m, jacobi=jacobi)
    return Un - U, np.asarray(hist)


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("jacobi", [False, True])
def test_arnoldi_sizes_single_and_lockstep_match_the_oracle(jacobi):
    """Histories within 1e-9 of the initial residual and updates within 1e-8,
    the bounds of the other solver checks; the small solves are rounded
    differently (sum orders), never by more than that."""
    from paper_2209_04481_amd import Ensemble
    insts = inputs()
    ref = [oracle_step(i, m, jacobi) for i, (_, _, m) in zip(insts, CASES)]
    ctxs = [context(i) for i in insts]
    Us = [torch.from_numpy(i.U).cuda() for i in insts]
    for q, (N, Nr, m) in enumerate(CASES):
        print(f"case: cfv_be_step {N} x {Nr}, GMRES({m}), jacobi {jacobi}", flush=True)
        ctxs[q].set_preconditioner(int(jacobi))
        Un, hist = ctxs[q].be_step(Us[q], cfl=1e3, m=m)
        dx, ho = ref[q]
        assert np.abs(np.asarray(hist) - ho).max() <= 1e-9, (N, Nr, m)
        assert float(rel_err_per_var((Un - Us[q]).cpu(), dx).max()) <= 1e-8, (N, Nr, m)
    ens = Ensemble(ctxs)
    ens.set_preconditioner(int(jacobi))
    for m in sorted({c[2] for c in CASES}):
        print(f"case: lockstep step of {CASES}, GMRES({m}), jacobi {jacobi}", flush=True)
        Un, hist = ens.be_step(Us, cfl=1e3, m=m)
        torch.cuda.synchronize()
        for q in [q for q, c in enumerate(CASES) if c[2] == m]:
            dx, ho = ref[q]
            assert np.abs(hist[q].cpu().numpy() - ho).max() <= 1e-9, CASES[q]
            assert float(rel_err_per_var((Un[q] - Us[q]).cpu(), dx).max()) <= 1e-8, CASES[q]


def test_solves_and_vjp_do_not_read_what_nothing_wrote():
    """Workspaces allocated where freed memory held NaN: a restarted transposed
    solve (its residual vector is first used by the second cycle), the forward
    one and the VJP give the bits of a first run."""
    def fill_free_memory():
        ts = [torch.full((1 << e,), float("nan"), dtype=torch.float64, device="cuda") for e in range(8, 26)
              for _ in range(4)]
        torch.cuda.synchronize()
        del ts
        torch.cuda.empty_cache()

    inst = ci.make_instance(6, 10, "log", lmax=2, seed=8)
    U = torch.from_numpy(inst.U).cuda()
    b = torch.randn(9, inst.ncells, dtype=torch.float64, device="cuda")
    got = []
    for _ in range(2):
        fill_free_memory()
        ctx = context(inst)
        D = ctx.local_dt(U, 0.5)
        x, _ = ctx.solve(U, D, b, transpose=True, m=7, max_restarts=3)
        y, _ = ctx.solve(U, D, b, m=7, max_restarts=3)
        gU, gbr = ctx.vjp(U, b)
        got.append((x.cpu(), y.cpu(), gU.cpu(), gbr.cpu()))
    for p, q in zip(*got):
        assert bool(torch.isfinite(p).all()) and torch.equal(p, q)


def plain_gmres(A, b, m, restarts, D=None):
    """Restarted GMRES(m) in float64 torch, one projection and one update per
    basis vector; D: the right preconditioner's diagonal.  (x, |r_j| / |b|)."""
    x, hist = torch.zeros_like(b), []
    for _ in range(restarts + 1):
        r = b - A(x)
        V, H = [r / r.norm()], torch.zeros(m + 1, m, dtype=torch.float64)
        for j in range(m):
            w = A(V[j] / D if D is not None else V[j])
            for i in range(j + 1):
                h = (w * V[i]).sum()
                H[i, j] = h
                w = w - h * V[i]
            H[j + 1, j] = w.norm()
            V.append(w / H[j + 1, j].to(w.device))
            e = torch.zeros(j + 2, 1, dtype=torch.float64)
            e[0] = r.norm()
            y = torch.linalg.lstsq(H[:j + 2, :j + 1], e).solution
            hist.append(float((H[:j + 2, :j + 1] @ y - e).norm() / b.norm()))
        d = sum(float(y[i]) * V[i] for i in range(m))
        x = x + (d / D if D is not None else d)
    return x, np.asarray(hist)


def large_shell(N, Nr, jacobi):
    inst = ci.make_instance(N, Nr, "log", lmax=2, seed=950 + N)
    inst.U[8] = 1e-3 * np.random.default_rng(inst.seed).standard_normal(inst.ncells)
    ctx = context(inst)
    ctx.set_preconditioner(int(jacobi))
    return ctx, torch.from_numpy(inst.U).cuda()


# 33 x 10: 574.3 tiles of 1,024 entries, so 288 blocks of two (the last ones of one, and of a part of one), in
# four groups of up to four basis vectors; 49 x 25: 3,165 tiles, 453 blocks of seven, three groups
@pytest.mark.parametrize("N,Nr,m,restarts,transpose,jacobi", [(33, 10, 14, 0, False, False), (33, 10, 7, 1, True, False),
                                                             (33, 10, 14, 1, False, True), (49, 25, 7, 0, True, True)])
def test_blocks_of_several_tiles_and_groups_of_several_vectors(N, Nr, m, restarts, transpose, jacobi):
    """A solve against plain GMRES with the library's own Jacobian products:
    histories within 1e-9 of the initial residual and solutions within 1e-8."""
    print(f"case: solve {N} x {Nr}, GMRES({m}), {restarts} restarts, transpose {transpose}, jacobi {jacobi}", flush=True)
    ctx, U = large_shell(N, Nr, jacobi)
    D = ctx.local_dt(U, 10.0)
    b = torch.randn(U.shape, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
    product = (lambda x: ctx.vjp(U, x, want_br=False)[0]) if transpose else (lambda x: ctx.jvp(U, x))
    xo, ho = plain_gmres(lambda x: D * x + product(x), b, m, restarts, D if jacobi else None)
    x, hist = ctx.solve(U, D, b, transpose=transpose, m=m, max_restarts=restarts)
    assert hist.shape == ho.shape and np.abs(hist - ho).max() <= 1e-9
    assert float(rel_err_per_var(x.cpu(), xo.cpu()).max()) <= 1e-8


@pytest.mark.parametrize("jacobi", [False, True])
def test_lockstep_blocks_of_several_tiles(jacobi):
    """Uneven instances whose shares of the blocks have several tiles each, the
    basis in two groups: against each instance's own step."""
    from paper_2209_04481_amd import Ensemble
    shapes = [(33, 10), (24, 20), (16, 7), (40, 9)]
    print(f"case: lockstep step of {shapes}, GMRES(12), jacobi {jacobi}", flush=True)
    ctxs, Us = zip(*[large_shell(N, Nr, jacobi) for N, Nr in shapes])
    ens = Ensemble(ctxs)
    ens.set_preconditioner(int(jacobi))
    Un, hist = ens.be_step(list(Us), cfl=10.0, m=12)
    torch.cuda.synchronize()
    for q, (ctx, U) in enumerate(zip(ctxs, Us)):
        ref, ho = ctx.be_step(U, cfl=10.0, m=12)
        assert np.abs(hist[q].cpu().numpy() - np.asarray(ho)).max() <= 1e-9, shapes[q]
        assert float(rel_err_per_var((Un[q] - U).cpu(), (ref - U).cpu()).max()) <= 1e-8, shapes[q]
