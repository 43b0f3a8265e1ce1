// Adjoint (vector-Jacobian product) of the residual: gU = J_U^T w and
// gbr = J_b^T w, as deterministic passes without atomics.
//
// The forward residual is R_c = sum_f (+-) F(q_L,f, q_R,f) - V_c S(U_c) with
// face states q = P + G.(x_f - x_cell), G = phi (.) g the limited least-squares
// gradient and P the primitives (ghost states from the boundary laws).
//
//   pass 1  forward gradient/limiter pass: primitives and limited gradients
//           (and the ghost states and tile-edge cells' face states) for the
//           march, primitives and the six face states for the cell-centric
//           pass.
//   pass 2  per cell c: for each face, the flux adjoint for c's own side
//           (and the ghost side on boundary faces) with face weight
//           w_L - w_R; then the adjoint of c's reconstruction, limiter and
//           least-squares gradient, with contributions to c itself, to its
//           six neighbours and to ghost states.
//   pass 3  per boundary column: the ghost states' adjoints back through the
//           boundary laws onto the boundary cells and the B_r map.
//   pass 4  gU = (dP/dU)^T Pb minus the gravity source adjoint, with Pb the
//           sum of a cell's own and its neighbours' contributions.
//
// Pass 2 runs as a radial march over tiles (cfv_adjmarch.hpp), which sums the
// contributions inside a tile as it goes and finishes every cell that needs
// nothing from beyond its tile, chunk or boundary; pass 4 then completes the
// rest.  It holds 476 registers per lane and 157 KB of LDS, one workgroup per
// CU, and reads 45 values and writes 9 per cell (27 more per ring slot),
// forming the face states from the gradients: as many bytes take 1.1 ms at
// 13.3M cells, the pass 4.5, bound by its own arithmetic (about 6,000 vector
// instructions a layer) and by LDS and dependent arithmetic with one wavefront
// per SIMD.  With 54 stored face states it read 72 values a cell and took 5.3
// ms.  The 13.3M-cell VJP takes 6.7 ms, the 1.66M-cell one 0.94; with every
// contribution through memory (the cell-centric passes of cfv_vjp.hpp, kept
// for the shells that fill tiles badly) 10.5 and 1.50.
#include "cfv_adjmarch.hpp"

namespace cfv {

int64_t vjp_workspace_doubles(const Shape& g) { return vjp_workspace_size(g); }

// the adjoint windows that hold a boundary-layer cell, in order (out: room
// for all of them, or null to count)
int64_t adjoint_boundary_windows(const Shape& g, int64_t* out) {
  int64_t n = 0;
  for (int64_t b = 0; b * kVBlock < g.ncells; ++b)
    if (adjoint_window_has_boundary(g, b * kVBlock)) {
      if (out) out[n] = b;
      ++n;
    }
  return n;
}

// kBoundary false: every window, those holding a boundary-layer cell left
// out; true: the windows listed in bw (their windows, each once or more: a
// window's rows are written, not accumulated, so a repeat writes the same)
template <bool kBoundary>
__global__ __launch_bounds__(kVBlock) void adjoint_kernel(DevGrid, const double* __restrict__ w,
                                                          const double* __restrict__ W, const double* __restrict__ Q,
                                                          double* __restrict__ A, double* __restrict__ Gg,
                                                          const int64_t* __restrict__ bw) {
  __shared__ double lW[63 * kVBlock];  // primitives (9 rows), then the face states (54)
  __shared__ double lw[9 * kVBlock];
  const DevGrid& d = first_kernel_arg<DevGrid>();
  const int64_t nc = d.g.ncells;
  const int64_t c0 = (kBoundary ? gld(bw, int64_t(blockIdx.x)) : int64_t(blockIdx.x)) * kVBlock;
  if (!kBoundary && adjoint_window_has_boundary(d.g, c0)) return;  // the same in every lane
  const int64_t c = c0 + threadIdx.x;
  if (c < nc) {
    // every load of the window issued before the first LDS store (one memory
    // latency for the 72 rows, not one per batch of rows)
    double t[72];
#pragma unroll
    for (int r = 0; r < 9; ++r) t[r] = gld(W, r * nc + c);
#pragma unroll
    for (int r = 0; r < 54; ++r) t[9 + r] = gld(Q, r * nc + c);
#pragma unroll
    for (int r = 0; r < 9; ++r) t[63 + r] = gld(w, r * nc + c);
#pragma unroll
    for (int r = 0; r < 63; ++r) lW[r * kVBlock + threadIdx.x] = t[r];
#pragma unroll
    for (int r = 0; r < 9; ++r) lw[r * kVBlock + threadIdx.x] = t[63 + r];
  }
  __syncthreads();
  if (c < nc) adjoint_cell<kBoundary>(d, w, W, Q, A, Gg, c, lW, lw, c0);
}

// Per boundary column: the ghost states' adjoints through the boundary laws
// (ghost_fold_column in cfv_vjp.hpp).
__global__ __launch_bounds__(kVBlock) void ghost_fold_kernel(DevGrid, const double* __restrict__ W,
                                                             const double* __restrict__ Gg, double* __restrict__ A,
                                                             double* __restrict__ gbr) {
  const DevGrid& d = first_kernel_arg<DevGrid>();
  const int64_t col = int64_t(blockIdx.x) * kVBlock + threadIdx.x;
  if (col >= d.g.nb) return;
  ghost_fold_column(d, W, Gg, A, gbr, col);
}

__global__ __launch_bounds__(kVBlock) void gather_kernel(DevGrid d, const double* __restrict__ U,
                                                         const double* __restrict__ w, const double* __restrict__ A,
                                                         double* __restrict__ gU) {
  const int64_t c = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c < d.g.ncells) gather_cell(d, U, w, A, gU, c);
}

// ------------------------------------------------------------- the march
// One tile and chunk per workgroup, items dealt to the XCDs in contiguous
// eighths (neighbouring tiles share an L2).
template <bool Narrow>
__global__ __launch_bounds__(kNT, 1) void adjoint_march_kernel(AdjArgs, int64_t total) {
  using WG = AdjMarch<Narrow>;
  __shared__ double lds[WG::kLds];
  const AdjArgs& a0 = constant_args(&first_kernel_arg<AdjArgs>());
  const int64_t per = (total + 7) / 8;
  const int64_t item = int64_t(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (int64_t(blockIdx.x / 8) >= per || item >= total) return;
  const int t = threadIdx.x;
  TileMap tm;
  tile_of_logical(a0.d.g, item, tm, a0.kc);
  AState st;
  WG::init(a0, tm, st, t, lds);
  WG::fetch_ring(a0, st, t, tm.k0);
  WG::publish(a0, tm, st, t, lds);
  WG::publish_states(a0, st, t, tm.k0, lds);
  for (int k = tm.k0;;) {
    const AdjArgs& a = per_layer(a0);
    const bool more = k + 1 < tm.k1;
    __syncthreads();
    WG::faces(a, tm, st, lane_here(t), k, lds);
    __syncthreads();
    WG::gradient(a, tm, st, lane_here(t), k, lds);
    __syncthreads();
    if (more) WG::publish(a, tm, st, lane_here(t), lds);
    WG::gather(a, tm, st, lane_here(t), k, lds);
    if (!more) break;
    __syncthreads();
    ++k;
    WG::publish_states(a, st, lane_here(t), k, lds);
  }
}

__global__ __launch_bounds__(kVBlock) void adj_ghost_kernel(AdjArgs) {
  const AdjArgs& a = first_kernel_arg<AdjArgs>();
  const int64_t col = int64_t(blockIdx.x) * kVBlock + threadIdx.x;
  if (col >= a.d.g.nb) return;
  const int y = int(blockIdx.y), side = y >= 10 ? 1 : 0, in = side ? y - 10 : y;
  if (in == 9 && !a.gbr) return;
  adj_ghost_input(a, col, side, in);
}

__global__ __launch_bounds__(kVBlock) void adjoint_finish_kernel(AdjArgs) {
  const AdjArgs& a = first_kernel_arg<AdjArgs>();
  const int64_t c = int64_t(blockIdx.x) * kVBlock + threadIdx.x;
  if (c < a.d.g.ncells) adjoint_finish_cell(a, c);
}

// Layers per chunk of the adjoint's march for a shell, or 0 where the
// cell-centric passes are the better path.  A tile's layer takes a workgroup
// 20-22 us however many of its 256 lanes hold cells, and
// a chunk about one layer more; 256 consecutive cells take the cell-centric
// passes about 45 us and those passes 55 us more of launches and tails.  So
// tiles that divide a panel badly (N = 17 in four tiles of 16: 24 tiles for
// 6.8 tiles of cells) or hardly fill one (N <= 6 with many layers) go cell by
// cell.  In us, by the march and cell by cell: 17 x 100 323 and 259, 33 x 60 475
// and 449, 6 x 200 175 and 161, 4 x 300 261 and 165; 17 x 40 160 and 185, 49 x 60
// 792 and 908, 32 x 60 235 and 386, 20 x 60 214 and 231, 24 x 80 273 and 346, 16 x
// 40 82 and 138, 8 x 16 65 and 118.  (The estimate is a few us out where both are
// near, 8 x 120 127 and 144, 17 x 60 218 and 204.)
// (N < 4 too: the march's edge contributions, 576 values per tile and layer,
// take the place of the cells' 54 face-state values.)
int adjoint_march_chunk(const Shape& g, int cus) {
  if (g.N < 4) return 0;
  const int64_t tiles = 6LL * march_tiles_1d(g.N) * march_tiles_1d(g.N);
  const int kc = balanced_chunk(tiles, g.Nr, cus, 1);
  const int64_t items = tiles * ((g.Nr + kc - 1) / kc);
  const int64_t march = (items + cus - 1) / cus * (kc + 1) * 22 + 15;
  const int64_t windows = (g.ncells + kVBlock - 1) / kVBlock;
  const int64_t cells = (windows + cus - 1) / cus * 45 + 55;
  return march <= cells ? kc : 0;
}

// Whether narrow tiles' idle lanes repeat their columns (AdjMarch): where
// wavefronts of four or eight lanes can run with no fuller tile in their
// shader engine.  That is a panel of one full tile among four (N = 17, 18: 17 x
// 40 234 us with idle lanes, 160 without), and a last round of items that
// leaves compute units idle (49 x 60, 480 items on 256: 982 and 792; 65 x 60,
// 750: 1,377 and 1,192).  Rounds that fill the device hide it (49 x 120, 768
// items: 1,428 and 1,445; 34 x 60, one round: 457 and 460).
static bool repeat_narrow_tiles(const Shape& g, int64_t items, int cus) {
  if (g.N % kTI != 1 && g.N % kTI != 2) return false;
  return g.N <= kTI + 2 || (items > cus && items % cus != 0);
}

// the adjoint and the passes after it, tile by tile
static void launch_adjoint_march(const AdjArgs& a, int cus, hipStream_t s, KernelTimer* t) {
  const Shape& g = a.d.g;
  {
    TimedScope ts(t, "adjoint", s);
    const int64_t total = march_logical_blocks(g, a.kc);
    const dim3 grid(unsigned((total + 7) / 8 * 8));
    if (repeat_narrow_tiles(g, total, cus))
      hipLaunchKernelGGL(adjoint_march_kernel<true>, grid, dim3(kNT), 0, s, a, total);
    else
      hipLaunchKernelGGL(adjoint_march_kernel<false>, grid, dim3(kNT), 0, s, a, total);
  }
  {
    TimedScope ts(t, "adjoint_ghosts", s);
    hipLaunchKernelGGL(adj_ghost_kernel, dim3(unsigned((g.nb + kVBlock - 1) / kVBlock), 19), dim3(kVBlock), 0, s, a);
  }
  TimedScope ts(t, "adjoint_finish", s);
  hipLaunchKernelGGL(adjoint_finish_kernel, dim3(unsigned((g.ncells + kVBlock - 1) / kVBlock)), dim3(kVBlock), 0, s, a);
}

// and cell by cell
static void launch_adjoint_cells(const DevGrid& d, const double* U, const double* w, double* gU, double* gbr, double* W,
                                 double* A, const int64_t* bw, int64_t nbw, hipStream_t s, KernelTimer* t) {
  const int64_t nc = d.g.ncells;
  const dim3 grid(unsigned((nc + kVBlock - 1) / kVBlock));
  double* Q = A + int64_t(63) * nc;
  double* Gg = A + int64_t(63 + 54) * nc;
  {
    // interior windows, then those with boundary-layer cells (bw[nbw])
    TimedScope ts(t, "adjoint", s);
    hipLaunchKernelGGL(adjoint_kernel<false>, grid, dim3(kVBlock), 0, s, d, w, W, Q, A, Gg, bw);
    if (nbw > 0) hipLaunchKernelGGL(adjoint_kernel<true>, dim3(unsigned(nbw)), dim3(kVBlock), 0, s, d, w, W, Q, A, Gg, bw);
  }
  {
    TimedScope ts(t, "adjoint_ghosts", s);
    hipLaunchKernelGGL(ghost_fold_kernel, dim3(unsigned((d.g.nb + kVBlock - 1) / kVBlock)), dim3(kVBlock), 0, s, d, W,
                       Gg, A, gbr);
  }
  TimedScope ts(t, "adjoint_gather", s);
  hipLaunchKernelGGL(gather_kernel, grid, dim3(kVBlock), 0, s, d, U, w, A, gU);
}

// kc: layers per chunk of the forward pass; ahead: face_states_ahead; akc: layers
// per chunk of the adjoint's march (adjoint_march_chunk); cus: the device's
// compute units
hipError_t launch_vjp(const DevGrid& d, const double* U, const double* w, double* gU, double* gbr, double* W,
                      double* A, double* E, int kc, bool ahead, int akc, int cus, const int64_t* bw,
                      int64_t nbw, hipStream_t s, KernelTimer* t) {
  const int64_t nc = d.g.ncells;
  // pass 1: the forward gradient march writes the primitives (rows 0..8 of
  // W), and the limited gradients (its other 27) with the ghost states and the
  // tile-edge rows, or for the cell-centric passes the face states (the
  // workspace's last 54 rows)
  MarchArgs fa{d, U, nullptr, nullptr, W + int64_t(9) * nc, nullptr, nullptr, nullptr, W, nullptr};
  // the march writes gU while other tiles still read w, and reads U after: a
  // result over either goes cell by cell, whose last pass reads a cell's own
  // values and then writes them
  const int64_t n = 9 * nc;
  if ((gU < w + n && w < gU + n) || (gU < U + n && U < gU + n)) akc = 0;
  // the march's buffers take the cell-centric passes' rows: the seams (at most
  // 18 (Nr - 1) 6 N^2) and ghosts the 63 of contributions, the edges' the face
  // states'
  AdjArgs a{d, U, w, W, W + int64_t(9) * nc, E, A + int64_t(36) * nc, gU, A + int64_t(63) * nc, A,
            A + int64_t(63 + 54) * nc, A + int64_t(18) * nc, gbr, akc};
  if (akc > 0) {
    fa.Gs = A + int64_t(36) * nc;
    fa.E = E;
  } else {
    fa.Q = A + int64_t(63) * nc;
  }
  if (hipError_t e = launch_march_grad(fa, kc, ahead, s, t)) return e;
  if (akc > 0)
    launch_adjoint_march(a, cus, s, t);
  else
    launch_adjoint_cells(d, U, w, gU, gbr, W, A, bw, nbw, s, t);
  return hipGetLastError();
}

}  // namespace cfv
