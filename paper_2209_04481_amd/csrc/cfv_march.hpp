// Phase functions of the tiled radial-march kernels (see march.hip).
// Everything here is __host__ __device__ so that the same code runs on the
// GPU and under a host emulation of a workgroup.
#pragma once
#include "cfv_kernels.hpp"

namespace cfv {

constexpr int kTI = 16, kTJ = 16, kNT = kTI * kTJ;  // tile of columns
constexpr int kKC = 16;                             // radial layers per chunk (default)

struct MarchArgs {
  DevGrid d;
  const double* U;
  const double* Ud;   // tangent of U (Dual only; null means zero)
  const double* dbr;  // tangent of the B_r map (Dual only; nullable)
  double* G;          // limited gradients [27][ncells]
  double* Gd;         // their tangents (Dual only)
  double* R;          // residual (nullable for Dual)
  double* Rd;         // tangent of the residual (Dual only)
  double* P = nullptr;  // primitives [9][ncells] written by the gradient pass (nullable)
  double* Q = nullptr;  // face states [6 x 9][ncells] (row 9 lf + v) written by the face-state gradient pass
  double* E = nullptr;  // dual march: tile-edge face states (edge_buffer_doubles), written by the gradient
                        // pass, read by the flux pass's ring
  double* D = nullptr;  // the fused march with face speeds: sum_f s_f |S_f| / cfl per cell
  double cfl = 1.0;
  double* Gs = nullptr;  // the face-state gradient pass: inner and outer ghost states [2][9][6 N^2] (nullable)
};

// what the fused march computes: the residual, the face speeds' sum
// (backward-Euler diagonal), or both in one pass
enum MarchOut : int { kOutResidual = 0, kOutSpeeds = 1, kOutBoth = 2 };

struct TileMap {
  int p, j0, i0, k0, k1;
};

// Tile-edge face states of the dual march: for every tile, layer and edge
// slot (64 slots: 16 east faces of the last column by row, 16 north faces of
// the last row by column, 16 west faces of the first column by row, 16 south
// faces of the first row by column), the edge cell's state on that face (9
// values, then their 9 tangents), at [tile][layer][18][64].  The gradient
// pass writes them (its edge cells have their limited gradients at hand);
// the flux pass's ring reads a neighbour tile's 18 contiguous rows instead of
// that cell's primitives and gradients (72 values, strided by N along the
// tile's east and west edges).
constexpr int kEdgeSlots = 64, kEdgeLayer = 18 * kEdgeSlots;
__host__ __device__ __forceinline__ int march_tiles_1d(int N) { return (N + 15) / 16; }
__host__ __device__ __forceinline__ int64_t edge_buffer_doubles(const Shape& g) {
  const int64_t nt = march_tiles_1d(g.N);
  return 6 * nt * nt * int64_t(g.Nr) * kEdgeLayer;
}
__host__ __device__ __forceinline__ int64_t march_tile_index(const Shape& g, int p, int j0, int i0) {
  const int64_t nt = march_tiles_1d(g.N);
  return (int64_t(p) * nt + j0 / 16) * nt + i0 / 16;
}

// work items (tile, chunk of kc layers) of one instance
__host__ __device__ __forceinline__ int64_t march_logical_blocks(const Shape& g, int kc) {
  const int64_t nti = (g.N + kTI - 1) / kTI, ntj = (g.N + kTJ - 1) / kTJ, nch = (g.Nr + kc - 1) / kc;
  return 6 * ntj * nti * nch;
}

// Chunk length for a march over `tiles` column tiles of Nr layers with
// `slots` workgroups resident at once: of the chunk counts n, the one that
// minimises the rounds of work items times the layers an item marches (its
// own, plus `extra`: one warm-up and one cool-down layer); kc = ceil(Nr / n).
inline int balanced_chunk(int64_t tiles, int Nr, int64_t slots, int extra = 2) {
  int best = Nr;
  int64_t best_cost = -1;
  for (int n = 1; n <= Nr; ++n) {
    const int kc = (Nr + n - 1) / n;
    if ((Nr + kc - 1) / kc != n) continue;  // the same chunks as a smaller n
    const int64_t rounds = (tiles * n + slots - 1) / slots;
    const int64_t cost = rounds * (kc + extra);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = kc;
    }
  }
  return best;
}

// Whether the VJP's face-state pass loads its layers ahead (GradWG), at one
// workgroup per CU, or not, at two.  It is for shells that fill tiles badly; by
// the shell's own chunk length kc, whatever the caller's, since the two are not
// the same bits.  Not ahead where the items take two rounds of one workgroup
// per CU and one of two.  In us, the pass ahead and not: 33 x 160 (486 items on
// 256 CUs) 371 and 280, 33 x 300 767 and 650; the whole VJP 49 x 60 (480) 904 and
// 880.  Otherwise, the VJP in one round 33 x 40 324 and 331, 17 x 200 463 and 550
// (its narrow tiles' idle lanes run along), in three 65 x 60 1,534 and 1,559.
inline bool face_states_ahead(const Shape& g, int kc, int cus) {
  const int64_t items = march_logical_blocks(g, kc);
  return items <= cus || items > 2 * int64_t(cus);
}

// launch size: a multiple of 8 so that the XCD split is a bijection
__host__ __device__ __forceinline__ int64_t march_blocks(const Shape& g, int kc) {
  return (march_logical_blocks(g, kc) + 7) / 8 * 8;
}

// logical block l (chunk fastest, then tile i, tile j, panel) -> tile and chunk
__host__ __device__ __forceinline__ void tile_of_logical(const Shape& g, int64_t l, TileMap& tm, int kc) {
  const int64_t nti = (g.N + kTI - 1) / kTI, ntj = (g.N + kTJ - 1) / kTJ, nch = (g.Nr + kc - 1) / kc;
  int64_t r = l;
  const int ch = int(r % nch);
  r /= nch;
  const int ti = int(r % nti);
  r /= nti;
  const int tj = int(r % ntj);
  tm.p = int(r / ntj);
  tm.j0 = tj * kTJ;
  tm.i0 = ti * kTI;
  tm.k0 = ch * kc;
  tm.k1 = tm.k0 + kc < g.Nr ? tm.k0 + kc : g.Nr;
}

// ------------------------------------------------------------- small helpers
template <class T>
__host__ __device__ __forceinline__ T* lds_as(double* lds) {
  return reinterpret_cast<T*>(lds);
}

// A launch's descriptor (no kernel writes it while one runs) read through
// the constant address space: at a uniform address its fields become scalar
// loads, which the vector memory counter does not track, so reading one does
// not wait for the loads and stores in flight (a vector load of the field
// would: the compiler cannot prove that the kernel's own stores leave the
// descriptor alone).
template <class A>
__host__ __device__ __forceinline__ const A& constant_args(const A* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return *(const A*)reinterpret_cast<const __attribute__((address_space(4))) A*>(uniform_address(p));
#else
  return *p;
#endif
}

#if defined(__HIPCC__)
// the same descriptor, but a value the compiler cannot follow: reads through
// it are not hoisted out of the layer loop (the descriptor's fields would
// otherwise stay in scalar registers across the whole item and spill)
template <class A>
__device__ __forceinline__ const A& per_layer(const A& a) {
  const A* p = &a;
  asm volatile("" : "+s"(p));
  return constant_args(p);
}
#endif

// as ldT, both arrays there: without a branch, behind which every later wait
// for an older load would have to be for this one too
__host__ __device__ __forceinline__ void ld_both(const double* a, const double*, int64_t i, double& x) { x = gld(a, i); }
__host__ __device__ __forceinline__ void ld_both(const double* a, const double* b, int64_t i, Dual& x) {
  x = Dual(gld(a, i), gld(b, i));
}
// row v of the state, on its way: without a tangent array its tangent is not
// one until arrived() has zeroed it
template <class T>
__host__ __device__ __forceinline__ void fetch_state(const MarchArgs& a, int64_t c, int v, T u[9]) {
  ld_both(a.U, a.Ud ? a.Ud : a.U, v * a.d.g.ncells + c, u[v]);
}
__host__ __device__ __forceinline__ void arrived(const MarchArgs&, double*) {}
__host__ __device__ __forceinline__ void arrived(const MarchArgs& a, Dual u[9]) {
  if (!a.Ud)
    for (int v = 0; v < 9; ++v) u[v].d = 0.0;
}

template <class T>
__host__ __device__ __forceinline__ void load_prims(const MarchArgs& a, int64_t c, T P[9]) {
  const int64_t nc = a.d.g.ncells;
  T u[9];
  for (int v = 0; v < 9; ++v) ldT(a.U, a.Ud, v * nc + c, u[v]);
  cons_to_prim(u, P, a.d.pr.gamma);
}

// Nothing moves across this point: the compiler otherwise gathers loads that
// are spread through the arithmetic on purpose, or starts the next face's
// reads early, and at one wavefront per SIMD the registers they wait in are
// worth more than the latency they hide.
__host__ __device__ __forceinline__ void keep_order() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// x is wanted here: the compiler may otherwise sink a face's arithmetic to
// where its sums are used, below the other faces', with every operand waiting
// in registers
__host__ __device__ __forceinline__ void settle(double& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#else
  (void)x;
#endif
}
__host__ __device__ __forceinline__ void settle(Dual& x) {
  settle(x.v);
  settle(x.d);
}

// the lane number, but a value the compiler cannot follow: LDS addresses
// built from it are formed where they are used.  (An LDS instruction's offset
// field holds 64 KB; the rows beyond need an address of their own, and all of
// them, loop invariant, would be kept in registers across the layers.)
__host__ __device__ __forceinline__ int lane_here(int t) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(t));
#endif
  return t;
}

// column -> (panel, j, i); columns are below 2^31 (32-bit division)
__host__ __device__ __forceinline__ void column_pji(const Shape& g, int64_t col, int& p, int& j, int& i) {
  const uint32_t n = uint32_t(g.N);
  uint32_t t = uint32_t(col);
  i = int(t % n);
  t /= n;
  j = int(t % n);
  p = int(t / n);
}

template <class T>
__host__ __device__ __forceinline__ T map_br(const MarchArgs& a, int64_t col) {
  T b;
  ldT(a.d.br, a.dbr, col, b);
  return b;
}

// canonical flux across a face: owner on the left
template <class T, class Between = Nothing>
__host__ __device__ __forceinline__ void face_flux(bool own, const T qs[9], const T qo[9], V3 S, T F[9], const Params& pr,
                                                   Between between = Between()) {
  const T* L = own ? qs : qo;
  const T* R = own ? qo : qs;
  rusanov(L, R, S, F, pr, between);
}

// ======================================================== gradient pass
// The dual pass (7.6 GB at 13.3M cells, 1.5 ms as a copy) takes 2.55 ms there
// and 358 us at 1.66M, bound by its own arithmetic and stores with one
// wavefront per SIMD; with a layer's loads issued where they are wanted,
// instead of through the layer below's gradients, 2.99 ms and 407 us.  The
// VJP's forward pass (4.8 GB) takes 1.52 ms and 236 us (loads where they are
// wanted and two wavefronts per SIMD, which spilled: 1.69 and 300).
// LDS plane of (kTI + 2) x (kTJ + 2) positions: the tile at offset (1, 1)
// and a ring.  Every in-plane neighbour of an active cell has a position:
// an active in-tile cell publishes itself; for a neighbour that is not (tile
// edge, panel edge, or beyond a partial tile) the one active cell next to it
// stores its centroid sums once per item, and the second wavefront loads its
// primitives for every layer (ring()).
constexpr int kPW = kTI + 2, kPH = kTJ + 2, kPlane = kPW * kPH;
__host__ __device__ __forceinline__ int plane_pos(int ti, int tj) { return (tj + 1) * kPW + (ti + 1); }
__host__ __device__ __forceinline__ void dir_offset(int q, int& dx, int& dy) {
  dx = q == 0 ? -1 : q == 1 ? 1 : 0;
  dy = q == 2 ? -1 : q == 3 ? 1 : 0;
}

template <class T>
struct GState {
  int p, j, i;
  int64_t col;
  bool act;
  T Pm[9], P0[9], Pp[9];
  T u[9], ur[9];  // the state of the layer above Pp's, and a ring lane's of the layer above P0's, on their way
  int64_t rc0;  // ring threads: the ring slot's cell at layer 0 (-1: no slot)
  unsigned emask;  // the tile edges the cell lies on (bit = edge slot kind 0..3)
  int es0, es1;    // the edge slots of the first two of them (-1: none)
  unsigned erest;  // and the others (one-cell-wide tiles only)
  V3 fe0, fe1;     // their face-centroid offsets per unit rs_k
  // the column's geometry per item (centroid sum, radial face centroid per
  // unit radius, angular face-centroid offsets per unit rs_k)
  V3 cc, xr, fe[4];
};

// Ring slot r (0..63) of a tile: the out-of-tile neighbour across one edge
// face of the tile (kind 0: east of row idx's last cell, 1: north of column
// idx's last cell, 2: west of row idx's first cell, 3: south of column idx's
// first cell).  Returns false for a slot beyond a partial tile; otherwise the
// tile cell (ti, tj), the face direction q (0..3: W, E, S, N) and the
// neighbour's column.
__host__ __device__ __forceinline__ bool ring_slot(const MarchArgs& a, const TileMap& tm, int r, int& ti, int& tj,
                                                   int& q, int64_t& ncol) {
  const Shape& g = a.d.g;
  const int kind = r >> 4, idx = r & 15;
  const int tiL = (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
  const int tjL = (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
  ti = kind == 0 ? tiL : kind == 2 ? 0 : idx;
  tj = kind == 1 ? tjL : kind == 3 ? 0 : idx;
  q = kind == 0 ? 1 : kind == 1 ? 3 : kind == 2 ? 0 : 2;
  if (ti > tiL || tj > tjL) return false;
  ncol = gld(a.d.G.cn, q * a.d.G.ncol + column_of(g, tm.p, tm.j0 + tj, tm.i0 + ti));
  return true;
}

// Ahead: layers are loaded through the layer below's gradients, for one
// wavefront per SIMD, whose loads nothing else hides.  Without it they are
// loaded where they are wanted, and lanes without a cell load and compute
// nothing.
template <class T, bool Ahead = true>
struct GradWG {
  static constexpr int kTw = int(sizeof(T) / sizeof(double));
  // primitives plane (9 T per position), then the column centroid sums (3)
  static constexpr int kCs = 9 * kPlane * kTw;
  // dual pass and mode 2: a layer's tile-edge face states, staged for one
  // coalesced write ([18][64] doubles, the edge buffer's layout)
  static constexpr int kEs = kCs + 3 * kPlane;
  static constexpr int kLds = kEs + kEdgeLayer;

  __host__ __device__ static bool in_tile_active(const Shape& g, const TileMap& tm, int ti, int tj) {
    return ti >= 0 && ti < kTI && tj >= 0 && tj < kTJ && tm.i0 + ti < g.N && tm.j0 + tj < g.N;
  }

  __host__ __device__ static void init(const MarchArgs& a, const TileMap& tm, GState<T>& st, int t, double* lds) {
    const Shape& g = a.d.g;
    const GeomRef& G = a.d.G;
    const int ti = t % kTI, tj = t / kTI;
    st.p = tm.p;
    st.j = tm.j0 + tj;
    st.i = tm.i0 + ti;
    st.act = st.j < g.N && st.i < g.N;
    st.rc0 = -1;
    {
      // east (kind 0), north (1), west (2), south (3) tile edges of the cell
      const int tiL = (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
      const int tjL = (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
      st.emask = unsigned(ti == tiL) | unsigned(tj == tjL) << 1 | unsigned(ti == 0) << 2 | unsigned(tj == 0) << 3;
      st.es0 = st.es1 = -1;
      st.erest = 0;
    }
    const int slot = ring_slot_of(t);
    if (slot >= 0) {  // the ring slot's neighbour cell, decoded once per item
      int ti2, tj2, q;
      int64_t ncol;
      if (ring_slot(a, tm, slot, ti2, tj2, q, ncol)) {
        int np, nj, ni;
        column_pji(g, ncol, np, nj, ni);
        st.rc0 = cell_index(g, np, 0, nj, ni);
      }
    }
    if (!st.act) {
      // every lane runs through the gradients (a branch around its prefetches
      // would make later waits wait for them): one without a cell takes the
      // panel's last, and leaves nothing
      st.j = st.j < g.N ? st.j : g.N - 1;
      st.i = st.i < g.N ? st.i : g.N - 1;
      st.col = column_of(g, st.p, st.j, st.i);
      for (int v = 0; v < 9; ++v) st.Pm[v] = st.P0[v] = st.Pp[v] = T(0.0);
      st.cc = cg3(G, CG_CSUM, st.col);
      st.xr = cg3(G, CG_XR, st.col);
      for (int q = 0; q < 4; ++q) st.fe[q] = 2.0 * cg3(G, CG_ANG + 6 * q + 3, st.col) - st.cc;
      st.fe0 = st.fe1 = mk(0.0, 0.0, 0.0);
    }
    if (!st.act) return;
    st.col = column_of(g, st.p, st.j, st.i);
    double* cs = lds + kCs;
    const V3 c0 = cg3(G, CG_CSUM, st.col);
    const int me = plane_pos(ti, tj);
    cs[me] = c0.x; cs[kPlane + me] = c0.y; cs[2 * kPlane + me] = c0.z;
    for (int q = 0; q < 4; ++q) {
      int dx, dy;
      dir_offset(q, dx, dy);
      if (in_tile_active(g, tm, ti + dx, tj + dy)) continue;
      const V3 cn = cg3(G, CG_CSUM, gld(G.cn, q * G.ncol + st.col));
      const int pos = plane_pos(ti + dx, tj + dy);
      cs[pos] = cn.x; cs[kPlane + pos] = cn.y; cs[2 * kPlane + pos] = cn.z;
    }
    for (int v = 0; v < 9; ++v) st.Pm[v] = st.P0[v] = st.Pp[v] = T(0.0);
    st.cc = c0;
    st.xr = cg3(G, CG_XR, st.col);
    for (int q = 0; q < 4; ++q) st.fe[q] = 2.0 * cg3(G, CG_ANG + 6 * q + 3, st.col) - c0;
    // the first two tile edges of the cell as slots and face offsets (kind
    // 0..3: east, north, west, south faces, q = 1, 3, 0, 2)
    st.fe0 = st.fe1 = mk(0.0, 0.0, 0.0);
    for (int kind = 0; kind < 4; ++kind) {
      if (!((st.emask >> kind) & 1u)) continue;
      const int q = kind == 0 ? 1 : kind == 1 ? 3 : kind == 2 ? 0 : 2;
      const int slot = kind * 16 + ((kind & 1) ? ti : tj);
      const V3 f = q == 0 ? st.fe[0] : q == 1 ? st.fe[1] : q == 2 ? st.fe[2] : st.fe[3];
      if (st.es0 < 0) { st.es0 = slot; st.fe0 = f; }
      else if (st.es1 < 0) { st.es1 = slot; st.fe1 = f; }
      else st.erest |= 1u << kind;
    }
  }

  // First layer of the march of a chunk [k0, k1): the layers k0 - 1 and k0
  // enter the registers through the warm-up iterations k < k0, which run this
  // phase alone, so every layer's primitives come from the same code whatever
  // the chunk length (and the outputs with them, bit for bit).
  __host__ __device__ static int first_layer(const TileMap& tm) { return tm.k0 >= 1 ? tm.k0 - 2 : -1; }

  // layer k: the primitives of layer k + 1; publish layer k's in LDS (a
  // warm-up iteration only shifts the registers instead), a ring lane also its
  // ring position's.  The states were fetched through the layer below's
  // gradients: with one wavefront per SIMD nothing else hides a load.
  // The second wavefront has all 64 ring slots (with 16 in each, all four
  // wavefronts took as long for their ring loads as it does: the dual pass
  // 2.58 against 2.55 ms at 13.3M cells, 376 against 358 us at 1.66M).
  __host__ __device__ static int ring_slot_of(int t) { return t >= kNT / 4 && t < kNT / 2 ? t - kNT / 4 : -1; }
  // row v of layer k's state (of one that is there, where k is not: unused)
  __host__ __device__ static void fetch(const MarchArgs& a, GState<T>& st, int k, int v) {
    const int kk = k < 0 ? 0 : k < a.d.g.Nr ? k : a.d.g.Nr - 1;
    fetch_state(a, cell_index(a.d.g, st.p, kk, st.j, st.i), v, st.u);
  }
  __host__ __device__ static void fetch_ring(const MarchArgs& a, GState<T>& st, int k, int v) {
    const int kk = k < a.d.g.Nr ? k : a.d.g.Nr - 1;
    fetch_state(a, st.rc0 + int64_t(kk) * a.d.g.N * a.d.g.N, v, st.ur);
  }
  __host__ __device__ static void publish(const MarchArgs& a, const TileMap& tm, GState<T>& st, int t, int k,
                                          double* lds) {
    const Shape& g = a.d.g;
    if (Ahead && st.rc0 >= 0) {  // rc0 >= 0: a ring lane with a neighbour
      if (k >= tm.k0) {
        arrived(a, st.ur);
        ring(a, tm, ring_slot_of(t), st.ur, lds);
      } else if (k + 1 == tm.k0) {
#pragma unroll
        for (int v = 0; v < 9; ++v) fetch_ring(a, st, tm.k0, v);
      }
    }
    if (Ahead && k == first_layer(tm))
#pragma unroll
      for (int v = 0; v < 9; ++v) fetch(a, st, k + 1, v);
    if (k + 1 >= 0 && k + 1 < g.Nr) {
      if constexpr (Ahead) {
        arrived(a, st.u);
        cons_to_prim(st.u, st.Pp, a.d.pr.gamma);
      } else if (st.act) {
        load_prims(a, cell_index(g, st.p, k + 1, st.j, st.i), st.Pp);
      }
    }
    if (Ahead && k < tm.k0)
#pragma unroll
      for (int v = 0; v < 9; ++v) fetch(a, st, k + 2, v);
    if (k < tm.k0) {
      for (int v = 0; v < 9; ++v) {
        st.Pm[v] = st.P0[v];
        st.P0[v] = st.Pp[v];
      }
    } else if (st.act) {
      T* L = lds_as<T>(lds);
      const int me = plane_pos(t % kTI, t / kTI);
      for (int v = 0; v < 9; ++v) L[v * kPlane + me] = st.P0[v];
      if (a.P) {
        const int64_t c = cell_index(g, st.p, k, st.j, st.i);
        for (int v = 0; v < 9; ++v) gst(a.P, v * g.ncells + c, val(st.P0[v]));
      }
    }
    if (!Ahead && st.rc0 >= 0 && k >= tm.k0) {
      T ur[9];
#pragma unroll
      for (int v = 0; v < 9; ++v) ldT(a.U, a.Ud, v * g.ncells + st.rc0 + int64_t(k) * g.N * g.N, ur[v]);
      ring(a, tm, ring_slot_of(t), ur, lds);
    }
  }

  // (the host emulations' step between publishing and the barrier: publish
  // fills the ring itself, no kernel calls this)
  __host__ __device__ static void ring_late(const MarchArgs&, const TileMap&, const GState<T>&, int, int, double*) {}

  // Ring position r of layer k from the neighbour's state u (the plane's
  // out-of-tile neighbours, filled by one wavefront in one pass instead of a
  // divergent pass per direction in every wavefront): kind 0 east of row idx's last cell, 1 north of
  // column idx's last cell, 2 west of row idx's first cell, 3 south of
  // column idx's first cell.
  __host__ __device__ static void ring(const MarchArgs& a, const TileMap& tm, int r, const T u[9], double* lds) {
    const Shape& g = a.d.g;
    const int kind = r >> 4, idx = r & 15;
    const int tiL = (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
    const int tjL = (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
    const int ti = kind == 0 ? tiL : kind == 2 ? 0 : idx;
    const int tj = kind == 1 ? tjL : kind == 3 ? 0 : idx;
    const int q = kind == 0 ? 1 : kind == 1 ? 3 : kind == 2 ? 0 : 2;
    int dx, dy;
    dir_offset(q, dx, dy);
    T qn[9];
    cons_to_prim(u, qn, a.d.pr.gamma);
    T* L = lds_as<T>(lds);
    const int pos = plane_pos(ti + dx, tj + dy);
    for (int v = 0; v < 9; ++v) L[v * kPlane + pos] = qn[v];
  }

  // row v of an edge slot: the state on the face, and its tangent (dual pass)
  // or the cell's primitive (mode 2)
  __host__ __device__ static void stage(double* Es, int v, int slot, Dual qf, Dual) {
    Es[v * kEdgeSlots + slot] = qf.v;
    Es[(9 + v) * kEdgeSlots + slot] = qf.d;
  }
  __host__ __device__ static void stage(double* Es, int v, int slot, double qf, double p) {
    Es[v * kEdgeSlots + slot] = qf;
    Es[(9 + v) * kEdgeSlots + slot] = p;
  }

  // Mode 0: the limited gradients to a.G.  Mode 1: the reconstructed face
  // states to a.Q instead.  Mode 2: the gradients, and what the adjoint's
  // march wants besides: the ghost states to a.Gs, the tile-edge cells' states
  // on their edge faces and primitives staged for the edge buffer.  Modes 1
  // and 2 (the VJP's forward passes) record non-physical face states.
  template <int Mode = 0>
  __host__ __device__ static void compute(const MarchArgs& a, const TileMap& tm, GState<T>& st, int t, int k,
                                          double* lds) {
    if (!Ahead && !st.act) return;
    const Shape& g = a.d.g;
    const GeomRef& G = a.d.G;
    const T* L = lds_as<T>(lds);
    const double* cs = lds + kCs;
    const int ti = t % kTI, tj = t / kTI;
    const double r0 = radius_uniform(G, k), r1 = radius_uniform(G, k + 1);
    const double rs = 0.125 * (r0 + r1);
    const V3 xc = rs * st.cc;
    // geometry: neighbour offsets and face-centroid offsets
    V3 dx[6], dxf[6];
    int pos[4];
    {
      // a layer's centroid is rs_k cc, an angular face's centroid 2 rs_k b_q,
      // a radial face's r xr: offsets from the item's constants
      const V3 xf0 = r0 * st.xr, xf1 = r1 * st.xr;
      dxf[0] = xf0 - xc;
      dxf[1] = xf1 - xc;
      if (k > 0) {
        dx[0] = (0.125 * (radius_uniform(G, k - 1) + r0) - rs) * st.cc;
      } else {
        const V3 S = (r0 * r0) * cg3(G, CG_SR, st.col);
        dx[0] = ghost_centre(xc, S, xf0) - xc;
      }
      if (k + 1 < g.Nr) {
        dx[1] = (0.125 * (r1 + radius_uniform(G, k + 2)) - rs) * st.cc;
      } else {
        const V3 S = (r1 * r1) * cg3(G, CG_SR, st.col);
        dx[1] = ghost_centre(xc, S, xf1) - xc;
      }
#pragma unroll
      for (int lf = 2; lf < 6; ++lf) {
        int ddx, ddy;
        dir_offset(lf - 2, ddx, ddy);
        pos[lf - 2] = plane_pos(ti + ddx, tj + ddy);
        const int q = pos[lf - 2];
        dxf[lf] = rs * st.fe[lf - 2];
        dx[lf] = rs * (mk(cs[q], cs[kPlane + q], cs[2 * kPlane + q]) - st.cc);
      }
    }
    const LsqWeights W(dx);
    // ghost states on the boundary layers
    T gin[9], gout[9];
    if (k == 0) {
      V3 xG;
      ghost_prims(a.d, st.p, k, st.j, st.i, 0, st.P0, xc, map_br<T>(a, st.col), gin, xG);
    }
    if (k + 1 == g.Nr) {
      V3 xG;
      ghost_prims(a.d, st.p, k, st.j, st.i, 1, st.P0, xc, T(0.0), gout, xG);
    }
    const int64_t c = cell_index(g, st.p, k, st.j, st.i);
    constexpr bool Faces = Mode == 1;
    bool bad = false;
    if constexpr (Mode != 0) {
      if (k == 0) bad = bad || !physical(gin);
      if (k + 1 == g.Nr) bad = bad || !physical(gout);
      if (a.Gs && st.act && k == 0)
        for (int v = 0; v < 9; ++v) gst(a.Gs, v * g.nb + st.col, val(gin[v]));
      if (a.Gs && st.act && k + 1 == g.Nr)
        for (int v = 0; v < 9; ++v) gst(a.Gs, (9 + v) * g.nb + st.col, val(gout[v]));
    }
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      // the next layers' loads, between the variables (the ring's in three
      // groups: all before the first variable 2.76 ms at 13.3M cells and 349 us
      // at 1.66M, one a variable 2.50 and 365, so 2.55 and 358)
      if (Ahead) fetch(a, st, k + 2, v);
      if (Ahead && v % 3 == 0 && st.rc0 >= 0)
#pragma unroll
        for (int r = v; r < v + 3; ++r) fetch_ring(a, st, k + 1, r);
      T qn[6];
      qn[0] = k > 0 ? st.Pm[v] : gin[v];
      qn[1] = k + 1 < g.Nr ? st.Pp[v] : gout[v];
#pragma unroll
      for (int q = 0; q < 4; ++q) qn[2 + q] = L[v * kPlane + pos[q]];
      T gx, gy, gz;
      limited_grad(W, dxf, a.d.pr.limiter, st.P0[v], qn, gx, gy, gz);
      if constexpr (!Faces) {
        if (st.act) {
          stT(a.G, a.Gd, (3 * v) * g.ncells + c, gx);
          stT(a.G, a.Gd, (3 * v + 1) * g.ncells + c, gy);
          stT(a.G, a.Gd, (3 * v + 2) * g.ncells + c, gz);
        }
        if constexpr (Mode == 2) {
          if (v == 0 || v == 7)
#pragma unroll
            for (int lf = 0; lf < 6; ++lf)
              bad = bad || !(val(st.P0[v] + (gx * dxf[lf].x + gy * dxf[lf].y + gz * dxf[lf].z)) > 0.0);
        }
        if constexpr (sizeof(T) > sizeof(double) || Mode == 2) {
          // the states on the cell's tile-edge faces (the same expression as
          // the flux pass's reconstruction) for the neighbour tiles' rings,
          // staged in LDS (flush_edges writes the layer's block)
          double* Es = lds + kEs;
          if (st.es0 >= 0) {  // rs_k fe is dxf of that face: the same products
            const V3 d0 = rs * st.fe0;
            const T qf = st.P0[v] + (gx * d0.x + gy * d0.y + gz * d0.z);
            stage(Es, v, st.es0, qf, st.P0[v]);
          }
          if (st.es1 >= 0) {
            const V3 d1 = rs * st.fe1;
            const T qf = st.P0[v] + (gx * d1.x + gy * d1.y + gz * d1.z);
            stage(Es, v, st.es1, qf, st.P0[v]);
          }
          if (st.erest) {
#pragma unroll
            for (int kind = 0; kind < 4; ++kind) {
              if (!((st.erest >> kind) & 1u)) continue;
              const int lf = kind == 0 ? 3 : kind == 1 ? 5 : kind == 2 ? 2 : 4;  // E, N, W, S
              const T qf = st.P0[v] + (gx * dxf[lf].x + gy * dxf[lf].y + gz * dxf[lf].z);
              const int slot = kind * 16 + ((kind & 1) ? ti : tj);
              stage(Es, v, slot, qf, st.P0[v]);
            }
          }
        }
      } else {  // instead of the gradient, the reconstructed state at each face centroid
#pragma unroll
        for (int lf = 0; lf < 6; ++lf) {
          const double qf = val(st.P0[v] + (gx * dxf[lf].x + gy * dxf[lf].y + gz * dxf[lf].z));
          if (st.act) gst(a.Q, (9 * lf + v) * g.ncells + c, qf);
          if (v == 0 || v == 7) bad = bad || !(qf > 0.0);
        }
      }
    }
    if constexpr (Mode != 0) record_nonphysical(a.d, st.act && bad);
    for (int v = 0; v < 9; ++v) {
      st.Pm[v] = st.P0[v];
      st.P0[v] = st.Pp[v];
    }
    (void)tm;
  }

  // dual pass and mode 2, after the barrier that ends layer k's compute step: lanes
  // 128..191 write the layer's staged tile-edge states (slots of edge cells
  // beyond a partial tile hold stale values that no ring reads)
  __host__ __device__ static void flush_edges(const MarchArgs& a, const TileMap& tm, int t, int k,
                                              const double* lds) {
    if (!a.E || t < 2 * kEdgeSlots || t >= 3 * kEdgeSlots) return;
    const Shape& g = a.d.g;
    const int r = t - 2 * kEdgeSlots;
    const int64_t eb = (march_tile_index(g, tm.p, tm.j0, tm.i0) * g.Nr + k) * kEdgeLayer + r;
    const double* Es = lds + kEs;
#pragma unroll
    for (int row = 0; row < 18; ++row) gst(a.E, eb + row * kEdgeSlots, Es[row * kEdgeSlots + r]);
  }
};

// ============================================================ flux pass
// Per layer a cell's 72 values (state and limited gradients with tangents) make
// six face states, then three fluxes: below, east, north (and the first
// wavefront the tile's west and south edges').  The pass is held by one
// wavefront per SIMD (512 registers, 160 KB of LDS), so nothing but its own
// instructions hides a load: the next layer's are issued a few at a time
// between the pieces of this layer's fluxes, which takes 72 doubles of
// registers; to have room for them the face states are formed a variable at a
// time and all angular ones go to LDS, and a flux takes the place there of the
// state it was made of.  On the 13.3M-cell shell the pass takes 2.88 ms (8.6 GB;
// 3.64 with a layer's loads issued together at its start), on 1.66M cells 413
// us (549).  Per layer of 33,000 cycles: arithmetic of four fluxes 16,000, face
// states 5,000, summing 2,300, the memory's share 19,600 beneath them.
template <class T>
struct FState {
  int64_t col, c0;  // its column, its cell at layer 0 (lanes without one: the panel's last)
  bool act;
  T u[9], G[27];   // layer k + 1's state and limited gradients, on their way
  double ring[5];  // the lane's share of its ring slot's values, likewise
  T qtop[9];  // top-face state of layer k
  T acc[9];   // residual of layer k so far
  bool bad;   // a face state of this column met a non-positive density or pressure
  int64_t ebase;  // ring slot t & 63: its state in the edge buffer at layer 0 (-1: no slot)
  unsigned own;   // bit q: the cell owns its angular face q (W, E, S, N); bit 4: the edge face the lane computes
  // the column's geometry per item: radial face centroid per unit radius, solid-angle
  // factor, centroid sum, angular face-centroid offsets per unit rs_k
  V3 xr, cc, fe[4];
  double om;
};

template <class T>
__host__ __device__ __forceinline__ void store_res(const MarchArgs& a, int64_t c, const T r[9]);
template <>
__host__ __device__ __forceinline__ void store_res<double>(const MarchArgs& a, int64_t c, const double r[9]) {
  for (int v = 0; v < 9; ++v) gst(a.R, v * a.d.g.ncells + c, r[v]);
}
template <>
__host__ __device__ __forceinline__ void store_res<Dual>(const MarchArgs& a, int64_t c, const Dual r[9]) {
  for (int v = 0; v < 9; ++v) {
    if (a.R) gst(a.R, v * a.d.g.ncells + c, r[v].v);
    gst(a.Rd, v * a.d.g.ncells + c, r[v].d);
  }
}

template <class T>
struct FluxWG {
  // LDS, in units of T: the west and south face states of the tile's cells
  // (18 rows of kNT), each replaced by the flux through that face, signed for
  // the cell, by the one lane that reads it; their east and north face states
  // (18 rows); the states of the out-of-tile neighbours across the tile's four
  // edges on the shared faces (9 rows of kRing: east edge by row, north by
  // column, west by row, south by column).  kEdge: the tile's west and south
  // edge faces.
  static constexpr int kRing = 4 * 16, kEdge = 2 * 16;
  static_assert(kTI == 16 && kTJ == 16, "ring and edge slots are laid out for 16 x 16 tiles");
  static constexpr int kRingOff = 36 * kNT;
  // then, in doubles, area vectors (what room there is): of the columns'
  // radial faces per unit radius squared, of the edge faces per unit
  // (r_k+1^2 - r_k^2) / 2
  static constexpr int kSr = (kRingOff + 9 * kRing) * int(sizeof(T) / sizeof(double)), kSx = kSr + 3 * kNT;
  static constexpr int kLds = kSx + 3 * kEdge;

  // last active column and row of the tile (partial tiles at the panel edge)
  __host__ __device__ static int last_ti(const Shape& g, const TileMap& tm) {
    return (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
  }
  __host__ __device__ static int last_tj(const Shape& g, const TileMap& tm) {
    return (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
  }

  // Layer k's state and gradients, a part (0: the state, 1..3: nine gradient
  // rows) at a time through the layer below's fluxes: a CU takes about 66
  // cycles per wavefront load however many are waiting, and a wavefront
  // stands still while its loads queue, so a layer's 72 issued together are
  // 19,000 cycles without arithmetic.  (Lanes without a cell load the
  // panel's last: with a branch around them, every later wait for an older
  // load would have to be for these too.)
  __host__ __device__ static void fetch(const MarchArgs& a, FState<T>& st, int k, int part, int v0 = 0, int v1 = 9) {
    const Shape& g = a.d.g;
    const int64_t c = st.c0 + int64_t(k) * g.N * g.N;
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      if (v < v0 || v >= v1) continue;
      if (part == 0)
        fetch_state(a, c, v, st.u);
      else
        ld_both(a.G, a.Gd, (9 * (part - 1) + v) * g.ncells + c, st.G[9 * (part - 1) + v]);
    }
  }
  // a part in four pieces between those of a flux
  struct Spread {
    const MarchArgs& a;
    FState<T>& st;
    int k, part;
    __host__ __device__ __forceinline__ void operator()(int i, T* F) const {
      if (i >= 3)
#pragma unroll
        for (int v = 0; v < 9; ++v) settle(F[v]);
      if (i == 4) return;
      keep_order();
      fetch(a, st, k, part, (9 * i + 3) / 4, (9 * i + 12) / 4);
      keep_order();
    }
  };
  // The ring slots of layer k: the states of the out-of-tile neighbours across
  // the tile's edge faces, on those faces, as the neighbour tiles' gradient
  // passes left them in the edge buffer.  A slot's rows are loaded by four
  // lanes, one per wavefront: lane t takes the rows t / 64, t / 64 + 4, ...
  // (a slot without a neighbour, or a row beyond the last, loads something
  // that is not used)
  static constexpr int kRows = 9 * int(sizeof(T) / sizeof(double)), kShare = (kRows + 3) / 4;
  __host__ __device__ static void fetch_ring(const MarchArgs& a, FState<T>& st, int t, int k) {
    const int64_t e = (st.ebase >= 0 ? st.ebase : 0) + int64_t(k) * kEdgeLayer;
#pragma unroll
    for (int n = 0; n < kShare; ++n) {
      const int row = (t >> 6) + 4 * n;  // the same in every lane of a wavefront
      st.ring[n] = gld(a.E, e + (row < kRows ? row : 0) * kEdgeSlots);
    }
  }
  __host__ __device__ static void ring_store(const FState<T>& st, int t, double* lds) {
    if (st.ebase < 0) return;
    constexpr int w = int(sizeof(T) / sizeof(double));
    double* Rg = lds + kRingOff * w;
#pragma unroll
    for (int n = 0; n < kShare; ++n) {
      const int row = (t >> 6) + 4 * n, v = row % 9, d = row / 9;  // values, then tangents
      if (row < kRows) Rg[(v * kRing + (t & 63)) * w + d] = st.ring[n];
    }
  }

  __host__ __device__ static void init(const MarchArgs& a, const TileMap& tm, FState<T>& st, int t) {
    const Shape& g = a.d.g;
    const int j = tm.j0 + t / kTI, i = tm.i0 + t % kTI;
    st.act = j < g.N && i < g.N;
    st.c0 = cell_index(g, tm.p, 0, j < g.N ? j : g.N - 1, i < g.N ? i : g.N - 1);
    st.col = column_of(g, tm.p, j < g.N ? j : g.N - 1, i < g.N ? i : g.N - 1);
    st.bad = false;
    for (int v = 0; v < 9; ++v) st.qtop[v] = T(0.0);
    st.ebase = -1;
    st.own = 0;
    const GeomRef& G = a.d.G;
    if (st.act) {
      st.xr = cg3(G, CG_XR, st.col);
      st.cc = cg3(G, CG_CSUM, st.col);
      st.om = gld(G.cg, CG_OMEGA * G.ncol + st.col);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        st.fe[q] = face_offset(G, st, q);
        st.own |= unsigned((gld(G.cn, (4 + q) * G.ncol + st.col) >> 8) != 0) << q;
      }
    }
    int eti, etj;
    if (edge_face(g, tm, t, eti, etj)) {
      const int q = t < 16 ? 2 : 0;
      const int64_t col = column_of(g, tm.p, tm.j0 + etj, tm.i0 + eti);
      st.own |= unsigned((gld(G.cn, (4 + q) * G.ncol + col) >> 8) != 0) << 4;
    }
    int ti, tj, q;
    int64_t ncol;
    if (ring_slot(a, tm, t & 63, ti, tj, q, ncol)) {  // the ring slot's source in the edge buffer
      // the neighbour cell, its tile and the edge slot of its face back
      // toward this tile (local faces 2..5: W, E, S, N)
      int np, nj, ni;
      column_pji(g, ncol, np, nj, ni);
      const int back = (gld(G.cn, (4 + q) * G.ncol + column_of(g, tm.p, tm.j0 + tj, tm.i0 + ti)) & 0xff) - 2;
      const int kind = back == 1 ? 0 : back == 3 ? 1 : back == 0 ? 2 : 3;
      const int slot = kind * 16 + ((kind & 1) ? ni % 16 : nj % 16);
      const int64_t tile = march_tile_index(g, np, nj - nj % 16, ni - ni % 16);
      st.ebase = tile * g.Nr * kEdgeLayer + slot;
    }
    const int k = first_layer(tm);
#pragma unroll
    for (int part = 0; part < 4; ++part) fetch(a, st, k, part);
    fetch_ring(a, st, t, k);
  }
  __host__ __device__ static V3 face_offset(const GeomRef& G, const FState<T>& st, int q) {
    return 2.0 * cg3(G, CG_ANG + 6 * q + 3, st.col) - st.cc;
  }
  __host__ __device__ static void put3(double* at, int stride, V3 x) {
    at[0] = x.x;
    at[stride] = x.y;
    at[2 * stride] = x.z;
  }
  __host__ __device__ static V3 get3(const double* at, int stride) { return mk(at[0], at[stride], at[2 * stride]); }
  // the tile-edge face that lane t < kEdge computes besides its cell's: the
  // south face of column t or the west face of row t - 16
  __host__ __device__ static bool edge_face(const Shape& g, const TileMap& tm, int t, int& eti, int& etj) {
    eti = t < 16 ? t : 0;
    etj = t < 16 ? 0 : t - 16;
    return t < kEdge && eti <= last_ti(g, tm) && etj <= last_tj(g, tm);
  }

  // Layers of the march of a chunk [k0, k1): a warm-up iteration k0 - 1
  // gives the top-face state of the layer below the chunk, a cool-down
  // iteration k1 the flux through the chunk's top face, both from the same
  // code as every other layer's (so the outputs do not depend on the chunk
  // length, bit for bit).
  __host__ __device__ static int first_layer(const TileMap& tm) { return tm.k0 > 0 ? tm.k0 - 1 : 0; }
  __host__ __device__ static int last_layer(const Shape& g, const TileMap& tm) {
    return tm.k1 < g.Nr ? tm.k1 : tm.k1 - 1;
  }

  // layer k's face states and its bottom face's flux, which completes the
  // residual of layer k - 1.  A warm-up layer (k < k0) runs this phase alone
  // for its top-face state, a cool-down layer (k = k1) for the flux through
  // the chunk's top face.
  __host__ __device__ static void states(const MarchArgs& a, const TileMap& tm, FState<T>& st, int t, int k,
                                         double* lds) {
    const bool marched = k >= tm.k0 && k < tm.k1;
    if (k == first_layer(tm)) {  // once per item
      int eti, etj;
      if (st.act) put3(lds + kSr + t, kNT, cg3(a.d.G, CG_SR, st.col));
      if (edge_face(a.d.g, tm, t, eti, etj))
        put3(lds + kSx + t, kEdge, cg3(a.d.G, CG_ANG + (t < 16 ? 12 : 0), column_of(a.d.g, tm.p, tm.j0 + etj, tm.i0 + eti)));
    }
    if (marched) ring_store(st, t, lds);
    const int kn = next_layer(a.d.g, tm, k);
    if (k < tm.k0) fetch_ring(a, st, t, kn);
    if (!st.act) return;
    const Shape& g = a.d.g;
    const GeomRef& G = a.d.G;
    const int64_t c = st.c0 + int64_t(k) * g.N * g.N;
    const double r0 = radius_uniform(G, k), r1 = radius_uniform(G, k + 1), rs = 0.125 * (r0 + r1);
    const V3 xc = rs * st.cc;
    T P[9], qT[9], qL[9], qR[9], grav[9];
    arrived(a, st.u);
    cons_to_prim(st.u, P, a.d.pr.gamma);
    gravity_source(st.u, xc, (r1 * r1 * r1 - r0 * r0 * r0) * st.om * (1.0 / 3.0), a.d.pr.G, grav);
    // the six face states, a variable at a time: its four values become two
    // that stay in registers (the top face's, and on the radial face below),
    // the angular faces' go to LDS
    {
      T* Sb = lds_as<T>(lds);
      const V3 dw = rs * st.fe[0], de = rs * st.fe[1], ds = rs * st.fe[2], dn = rs * st.fe[3];
      const V3 dt = r1 * st.xr - xc, db = r0 * st.xr - xc;
#pragma unroll
      for (int v = 0; v < 9; ++v) {
        keep_order();
        const T gx = st.G[3 * v], gy = st.G[3 * v + 1], gz = st.G[3 * v + 2];
        qT[v] = P[v] + (gx * dt.x + gy * dt.y + gz * dt.z);
        qR[v] = P[v] + (gx * db.x + gy * db.y + gz * db.z);
        if (v == 0 || v == 7) st.bad = st.bad || !(val(qT[v]) > 0.0 && val(qR[v]) > 0.0);
        if (!marched) continue;
        const T w = P[v] + (gx * dw.x + gy * dw.y + gz * dw.z), s = P[v] + (gx * ds.x + gy * ds.y + gz * ds.z);
        const T e = P[v] + (gx * de.x + gy * de.y + gz * de.z), n = P[v] + (gx * dn.x + gy * dn.y + gz * dn.z);
        if (v == 0 || v == 7)
          st.bad = st.bad || !(val(w) > 0.0 && val(s) > 0.0 && val(e) > 0.0 && val(n) > 0.0);
        Sb[v * kNT + t] = w;
        Sb[(9 + v) * kNT + t] = s;
        Sb[(18 + v) * kNT + t] = e;
        Sb[(27 + v) * kNT + t] = n;
      }
    }
    if (k < tm.k0) {
#pragma unroll
      for (int v = 0; v < 9; ++v) st.qtop[v] = qT[v];
      keep_order();
#pragma unroll
      for (int part = 0; part < 4; ++part) fetch(a, st, kn, part);
      return;
    }
#pragma unroll
    for (int v = 0; v < 9; ++v) qL[v] = st.qtop[v];
    if (k == 0) {  // the inner boundary face: the cell's, its area vector outward (one layer: its state is read again)
#pragma unroll
      for (int v = 0; v < 9; ++v) qL[v] = qR[v];
      V3 xG;
      load_prims(a, c, P);
      ghost_prims(a.d, tm.p, k, tm.j0 + t / kTI, tm.i0 + t % kTI, 0, P, xc, map_br<T>(a, st.col), qR, xG);
      st.bad = st.bad || !physical(qR);
    }
    keep_order();
    {
      T F[9];
      const V3 S = (r0 * r0) * get3(lds + kSr + t, kNT);
      rusanov(qL, qR, k == 0 ? mk(-S.x, -S.y, -S.z) : S, F, a.d.pr, Spread{a, st, kn, 0});
      if (k > tm.k0) {
#pragma unroll
        for (int v = 0; v < 9; ++v) st.acc[v] += F[v];
        store_res(a, c - int64_t(g.N) * g.N, st.acc);
      }
      const double sg = k == 0 ? 1.0 : -1.0;
#pragma unroll
      for (int v = 0; v < 9; ++v) {
        st.acc[v] = F[v] * sg - grav[v];
        st.qtop[v] = qT[v];
      }
    }
    // outer boundary face (likewise)
    if (k == g.Nr - 1) {
      T qG[9], F[9];
      V3 xG;
      load_prims(a, c, P);
      ghost_prims(a.d, tm.p, k, tm.j0 + t / kTI, tm.i0 + t % kTI, 1, P, xc, T(0.0), qG, xG);
      st.bad = st.bad || !physical(qG);
      rusanov(st.qtop, qG, (r1 * r1) * get3(lds + kSr + t, kNT), F, a.d.pr);
      for (int v = 0; v < 9; ++v) st.acc[v] += F[v];
    }
  }
  // the item's last layer loads its own again (unused)
  __host__ __device__ static int next_layer(const Shape& g, const TileMap& tm, int k) {
    return k < last_layer(g, tm) ? k + 1 : k;
  }

  // east and north faces of every cell (neighbour states from LDS: in-tile
  // or ring), the flux left for the neighbour in place of its state; the west
  // and south faces on the tile's edges by the first kEdge threads, for the
  // edge cells
  __host__ __device__ static void faces(const MarchArgs& a, const TileMap& tm, FState<T>& st, int t, int k,
                                        double* lds) {
    const Shape& g = a.d.g;
    T* Sb = lds_as<T>(lds);
    const T* Rg = lds_as<T>(lds) + kRingOff;
    const int ti = t % kTI, tj = t / kTI;
    const int tiL = last_ti(g, tm), tjL = last_tj(g, tm);
    const int kn = next_layer(g, tm, k);
    const double r0 = radius_uniform(a.d.G, k), r1 = radius_uniform(a.d.G, k + 1);
    const double ra = 0.5 * (r1 * r1 - r0 * r0);
    // the east and north faces' area vectors (LDS has no room for them)
    const V3 se = cg3(a.d.G, CG_ANG + 6, st.col), sn = cg3(a.d.G, CG_ANG + 18, st.col);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      keep_order();
      {
        const bool own = (st.own >> (h == 0 ? 1 : 3)) & 1u;
        // the neighbour's state from the tile or the ring, one code path
        // for both (lanes of one wavefront take either)
        const bool in = h == 0 ? ti < tiL : tj < tjL;
        const T* src = h == 0 ? (in ? Sb + t + 1 : Rg + tj) : (in ? Sb + 9 * kNT + t + kTI : Rg + 16 + ti);
        const int stride = in ? kNT : kRing;
        T qs[9], qo[9], F[9];
#pragma unroll
        for (int v = 0; v < 9; ++v) {
          qs[v] = Sb[(18 + 9 * h + v) * kNT + t];
          qo[v] = src[v * stride];
        }
        face_flux(own, qs, qo, ra * (h == 0 ? se : sn), F, a.d.pr, Spread{a, st, kn, 1 + h});
        if (!st.act) continue;
        const double sg = own ? 1.0 : -1.0;  // a product by +-1: the same bits as the select
#pragma unroll
        for (int v = 0; v < 9; ++v) {
          st.acc[v] += F[v] * sg;
          if (in) Sb[(9 * h + v) * kNT + t + (h == 0 ? 1 : kTI)] = F[v] * -sg;
        }
      }
      keep_order();
    }
    // (the first wavefront: every lane, so that its loads go between the
    // pieces; the lanes without an edge face leave nothing)
    keep_order();
    if (first_wavefront(t)) {
      int eti, etj;
      const bool south = t < 16, own = (st.own >> 4) & 1u;
      const int tc = south ? t : ((t - 16) & 15) * kTI;
      T qs[9], qo[9], F[9];
#pragma unroll
      for (int v = 0; v < 9; ++v) {
        qs[v] = Sb[((south ? 9 : 0) + v) * kNT + tc];
        qo[v] = Rg[v * kRing + (south ? 48 + t : 32 + ((t - 16) & 15))];
      }
      face_flux(own, qs, qo, ra * get3(lds + kSx + (t & 31), kEdge), F, a.d.pr, Spread{a, st, kn, 3});
      if (edge_face(g, tm, t, eti, etj))
#pragma unroll
        for (int v = 0; v < 9; ++v) Sb[((south ? 9 : 0) + v) * kNT + tc] = own ? F[v] : -F[v];
    } else {
      fetch(a, st, kn, 3);
    }
  }
  // (the same in every lane: a branch that no wavefront takes both ways)
  __host__ __device__ static bool first_wavefront(int t) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readfirstlane(t) < 64;
#else
    return t < 64;
#endif
  }

  __host__ __device__ static void accumulate(const MarchArgs& a, const TileMap& tm, FState<T>& st, int t, int k,
                                             double* lds) {
    fetch_ring(a, st, t, next_layer(a.d.g, tm, k));
    if (!st.act) return;
    const Shape& g = a.d.g;
    const T* Sb = lds_as<T>(lds);
    // (read again each layer: through the fluxes there is no register for them)
    const V3 b0 = cg3(a.d.G, CG_ANG + 3, st.col), b1 = cg3(a.d.G, CG_ANG + 9, st.col),
             b2 = cg3(a.d.G, CG_ANG + 15, st.col);
#pragma unroll
    for (int v = 0; v < 9; ++v) st.acc[v] += Sb[v * kNT + t];
#pragma unroll
    for (int v = 0; v < 9; ++v) st.acc[v] += Sb[(9 + v) * kNT + t];
    st.fe[0] = 2.0 * b0 - st.cc;
    st.fe[1] = 2.0 * b1 - st.cc;
    st.fe[2] = 2.0 * b2 - st.cc;
    if (k == g.Nr - 1) store_res(a, st.c0 + int64_t(k) * g.N * g.N, st.acc);
    (void)tm;
  }

  __host__ __device__ static void finish(const MarchArgs& a, const TileMap&, FState<T>& st, int) {
    record_nonphysical(a.d, st.act && st.bad);
  }
};

// One instance.
// kc: layers per work item (chunk)
hipError_t launch_march(const MarchArgs& a, bool dual, int kc, hipStream_t s, KernelTimer* t);
// The fused march of one instance (out: MarchOut).
hipError_t launch_fused(const MarchArgs& a, int kc, int out, hipStream_t s, KernelTimer* t);
// The VJP's forward pass (double): primitives into a.P, and the face states
// into a.Q, or (a.Q null) the limited gradients into a.G, the ghost states
// into a.Gs and the tile-edge cells' rows into a.E.  ahead: face_states_ahead.
hipError_t launch_march_grad(const MarchArgs& a, int kc, bool ahead, hipStream_t s, KernelTimer* t);

// Ensemble launch: n instances described by args[n] (device; null: one
// instance, described by the kernel's second argument), with
// item_off[n + 1] (device) the prefix sums of march_logical_blocks per
// instance (unused when n = 1).  Items (instance, tile, chunk) are taken in
// the order perm[total] (device; null = identity) either statically (each of
// the 8 XCDs takes a contiguous eighth of the list, strided over its
// workgroups) or from a device counter (queue != 0; counters[2] are reset by
// the launch itself).
struct EnsembleLaunch {
  const MarchArgs* args;
  const int64_t* item_off;
  const int64_t* perm;
  unsigned* counters;
  int n;
  int64_t total;
  int queue;
  unsigned blocks;
  int kc = kKC;  // layers per chunk (the items' depth), for both marches
};
hipError_t launch_march_ensemble(const EnsembleLaunch& e, bool dual, hipStream_t s, KernelTimer* t);
hipError_t launch_fused_ensemble(const EnsembleLaunch& e, int out, hipStream_t s, KernelTimer* t);

}  // namespace cfv
