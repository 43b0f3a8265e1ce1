// Phase functions of the adjoint's radial march (vjp.hip): per layer of a
// 16 x 16 tile of columns, the adjoint of every cell's face fluxes, limiter
// and gradient, with the contributions to neighbouring cells exchanged in
// LDS and registers, so that they do not go through memory (a cell's 54
// values to its six neighbours, written and read back, were a third of the
// VJP's traffic).
//
// Inputs are what the forward pass left (primitives P and limited gradients G,
// the tile-edge cells' states on their edge faces) and the weights w.  A
// cell's six face states follow from its P and G.  Its neighbours on the same
// layer are read from LDS (primitives and weights in planes with a ring, the
// face states by direction); the layers k - 1 and k + 1 of its own column are
// in registers, each value loaded from memory once.  Contributions:
//   to the layer below   complete that layer's cell, which is then written,
//   to the layer above   are carried one layer in registers,
//   across in-tile faces go through LDS (in the face states' place),
//   across the tile's edges and across the chunk's ends go to an edge and a
//                        seam buffer, and to the boundary ghosts to their
//                        rows; the cells they are for are left as adjoints of
//                        their primitives, which adjoint_finish_cell completes.
// No cell is computed twice, whatever the tiles and chunks.
//
// Everything here is __host__ __device__ (as the other marches').
#pragma once
#include "cfv_vjp.hpp"

namespace cfv {

struct AdjArgs {
  DevGrid d;
  const double* U;  // state (the finishing pass)
  const double* w;  // weights [9][ncells]
  const double* P;  // primitives [9][ncells]
  const double* G;  // limited gradients [27][ncells]
  const double* B;  // tile-edge cells' states on the edge faces and primitives: [tile][layer][18][64]
  const double* Gs; // inner and outer ghost states [2][9][6 N^2]
  double* gU;       // result [9][ncells]
  double* E;        // contributions across tile edges: [tile][layer][9][64], by the edge slot they leave through
  double* S;        // contributions across chunk ends: [chunk end][down, up][9][6 N^2]
  double* Gg;       // adjoints of the inner and outer ghost states: [2][9][6 N^2]
  double* Gp;       // these through the boundary laws onto the boundary cell: [2][9][6 N^2]
  double* gbr;      // nullable
  int kc;           // layers per chunk
};

constexpr int kAdjEdgeLayer = 9 * kEdgeSlots;
inline int64_t adj_seam_doubles(const Shape& g, int kc) {
  return int64_t((g.Nr + kc - 1) / kc - 1) * 18 * g.nb;
}

// whether the march leaves a cell to the finishing pass
__host__ __device__ __forceinline__ bool adj_unfinished(const Shape& g, int kc, int k, int j, int i) {
  const int ti = i % kTI, tj = j % kTJ;
  return ti == 0 || tj == 0 || ti == kTI - 1 || tj == kTJ - 1 || i == g.N - 1 || j == g.N - 1 || k == 0 ||
         k == g.Nr - 1 || k % kc == 0 || k % kc == kc - 1;
}

// gravity's adjoint: R -= V (0, rho g, 0, g . m, 0) at the centroid xc; wg: the weights of momentum and energy
__host__ __device__ __forceinline__ void gravity_adjoint(V3 xc, double vol, double G, const double wg[4], double Ub[9]) {
  const double r = norm3(xc);
  const double f = -G / (r * r * r) * vol;
  const V3 gv = mk(f * xc.x, f * xc.y, f * xc.z);
  Ub[0] -= gv.x * wg[0] + gv.y * wg[1] + gv.z * wg[2];
  Ub[1] -= gv.x * wg[3];
  Ub[2] -= gv.y * wg[3];
  Ub[3] -= gv.z * wg[3];
}

struct AState {
  int p, j, i;
  int64_t col;
  bool act, edge;  // edge: on the tile's rim
  V3 sr, xr;       // radial faces per unit radius
  double om;       // the column's solid-angle factor
  V3 fa[4];        // angular faces' area vectors per unit (r_k+1^2 - r_k^2) / 2
  unsigned own;    // bit q: the cell owns its angular face q
  int64_t rc0;     // ring slot t & 63: its cell at layer 0 (-1: none)
  int64_t rb0;     // and that cell's entry in the edge buffer at layer 0
  double Pm[9], P0[9], Pp[9];  // primitives of layers k - 1, k (until they are in LDS) and k + 1 (ghosts beyond the boundaries)
  double w0[9], wp[9];         // weights of layers k (until in LDS) and k + 1 (zero beyond the boundary)
  double wg[4];    // layer k - 1's weights that gravity's adjoint takes (momentum and energy)
  double G[27];    // limited gradients of layer k until its face states are formed, then of layer k + 1
  double qT[9];    // state of layer k on its top face
  double qb[9];    // adjoint of layer k's state on its bottom face, from the flux adjoint of the layer below
  double acc[9];   // adjoint of the primitives of layer k - 1 so far, then of layer k
  double Pb[9], Gb[27];  // adjoints of layer k's primitives (with the contribution from below) and limited gradients
  double ring[7];  // the lane's share of its slot's 27 values
};

// Narrow: for shells whose panels end in tiles one or two columns wide.  The
// lanes of such a tile that would have no cell repeat its columns, lane by
// lane the same values to the same places, so that all 64 lanes of its
// wavefronts work.  With 4 or 8 of them working, a layer took 35 us instead of
// 20 wherever no fuller tile ran in the same shader engine: the wavefronts
// wait for issue (SQ_WAIT_INST_ANY twice as high, no instruction cache
// misses), those of a tile with one wavefront do not.  An instance of its own:
// the column from the cell instead of the lane number costs full tiles 1%
// (48 x 120 954 and 967 us).
template <bool Narrow>
struct AdjMarch {
  // LDS: planes of primitives and weights of layer k (18 x 18 positions, the
  // tile and a ring), the column centroid sums (a plane of 3), the cells'
  // angular face-centroid offsets per unit rs_k (12 rows of 256), and per
  // direction q (W, E, S, N) nine rows of the cells' states on that face, with
  // 16 more entries for the ring cells that face the tile there; later, in
  // their place, the contributions leaving through that face
  static constexpr int kRow = kNT + 16;
  static constexpr int kP = 0, kW = kP + 9 * kPlane, kCs = kW + 9 * kPlane, kFe = kCs + 3 * kPlane,
                       kX = kFe + 12 * kNT, kLds = kX + 36 * kRow;
  __host__ __device__ static int x_at(int q, int v) { return kX + (9 * q + v) * kRow; }
  __host__ __device__ static int tile_i(const AState& st, int t) { return Narrow ? st.i % kTI : t % kTI; }

  __host__ __device__ static void load9(const double* a, int64_t nc, int64_t c, double q[9]) {
#pragma unroll
    for (int v = 0; v < 9; ++v) q[v] = gld(a, v * nc + c);
  }
  // the state at an offset d from the centroid
  __host__ __device__ static void recon9(const double P[9], const double G[27], V3 d, double q[9]) {
#pragma unroll
    for (int v = 0; v < 9; ++v) q[v] = P[v] + (G[3 * v] * d.x + G[3 * v + 1] * d.y + G[3 * v + 2] * d.z);
  }

  __host__ __device__ static void init(const AdjArgs& a, const TileMap& tm, AState& st, int t, double* lds) {
    const Shape& g = a.d.g;
    const GeomRef& G = a.d.G;
    const int tiL = (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
    const int tjL = (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
    const int ti = Narrow && tiL < 2 ? t % kTI & tiL : t % kTI, tj = t / kTI;
    st.p = tm.p;
    st.j = tm.j0 + tj;
    st.i = tm.i0 + ti;
    st.act = ti <= tiL && tj <= tjL;
    st.edge = ti == 0 || tj == 0 || ti == tiL || tj == tjL;
    st.rc0 = -1;
    {  // the ring slots, as the other marches', each shared by four lanes
      MarchArgs m;
      m.d = a.d;
      int ti2, tj2, q;
      int64_t ncol;
      if (ring_slot(m, tm, t & 63, ti2, tj2, q, ncol)) {
        int np, nj, ni;
        column_pji(g, ncol, np, nj, ni);
        st.rc0 = cell_index(g, np, 0, nj, ni);
        const int back = (gld(G.cn, (4 + q) * G.ncol + column_of(g, tm.p, tm.j0 + tj2, tm.i0 + ti2)) & 0xff) - 2;
        const int kind = back == 1 ? 0 : back == 3 ? 1 : back == 0 ? 2 : 3;
        st.rb0 = march_tile_index(g, np, nj - nj % kTJ, ni - ni % kTI) * g.Nr * kEdgeLayer + kind * 16 +
                 ((kind & 1) ? ni % kTI : nj % kTJ);
      }
    }
    if (!st.act) return;
    st.col = column_of(g, st.p, st.j, st.i);
    st.sr = cg3(G, CG_SR, st.col);
    st.xr = cg3(G, CG_XR, st.col);
    st.om = gld(G.cg, CG_OMEGA * G.ncol + st.col);
    const V3 cc = cg3(G, CG_CSUM, st.col);
    const int me = plane_pos(ti, tj);
    lds[kCs + me] = cc.x;
    lds[kCs + kPlane + me] = cc.y;
    lds[kCs + 2 * kPlane + me] = cc.z;
    st.own = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const V3 f = 2.0 * cg3(G, CG_ANG + 6 * q + 3, st.col) - cc;
      lds[kFe + (3 * q) * kNT + t] = f.x;
      lds[kFe + (3 * q + 1) * kNT + t] = f.y;
      lds[kFe + (3 * q + 2) * kNT + t] = f.z;
      st.own |= unsigned((gld(G.cn, (4 + q) * G.ncol + st.col) >> 8) != 0) << q;
      st.fa[q] = cg3(G, CG_ANG + 6 * q, st.col);
      int dx, dy;
      dir_offset(q, dx, dy);
      if (ti + dx >= 0 && ti + dx <= tiL && tj + dy >= 0 && tj + dy <= tjL) continue;
      const V3 cn = cg3(G, CG_CSUM, gld(G.cn, q * G.ncol + st.col));
      const int pos = plane_pos(ti + dx, tj + dy);
      lds[kCs + pos] = cn.x;
      lds[kCs + kPlane + pos] = cn.y;
      lds[kCs + 2 * kPlane + pos] = cn.z;
    }
    // the chunk's first layer, and the flux adjoint of its bottom face: with
    // the layer below's top state, or the inner ghost
    const int64_t NN = int64_t(g.N) * g.N, c = cell_index(g, st.p, tm.k0, st.j, st.i);
    const double r0 = radius_uniform(G, tm.k0);
    const bool bnd = tm.k0 == 0;  // the inner boundary face belongs to the cell and points inward
    double qB[9], qo[9], qL[9], qR[9], wb[9], qLb[9], qRb[9];
    load9(a.P, g.ncells, c, st.P0);
    load9(a.w, g.ncells, c, st.w0);
#pragma unroll
    for (int v = 0; v < 27; ++v) st.G[v] = gld(a.G, v * g.ncells + c);
    recon9(st.P0, st.G, r0 * st.xr - (0.125 * (r0 + radius_uniform(G, tm.k0 + 1))) * cc, qB);
    if (bnd) {
      load9(a.Gs, g.nb, st.col, st.Pm);
      load9(a.Gs, g.nb, st.col, qo);
    } else {
      load9(a.P, g.ncells, c - NN, st.Pm);
      double Gm[27];
#pragma unroll
      for (int v = 0; v < 27; ++v) Gm[v] = gld(a.G, v * g.ncells + c - NN);
      recon9(st.Pm, Gm, r0 * st.xr - (0.125 * (radius_uniform(G, tm.k0 - 1) + r0)) * cc, qo);
      load9(a.w, g.ncells, c - NN, wb);
    }
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      qL[v] = bnd ? qB[v] : qo[v];
      qR[v] = bnd ? qo[v] : qB[v];
      wb[v] = bnd ? st.w0[v] : wb[v] - st.w0[v];
      qLb[v] = qRb[v] = 0.0;
    }
    rusanov_adjoint(qL, qR, (bnd ? -(r0 * r0) : r0 * r0) * st.sr, wb, qLb, qRb, a.d.pr, true, true);
#pragma unroll
    for (int v = 0; v < 9; ++v) st.qb[v] = bnd ? qLb[v] : qRb[v];
    if (bnd)
#pragma unroll
      for (int v = 0; v < 9; ++v) gst(a.Gg, v * g.nb + st.col, qRb[v]);
#pragma unroll
    for (int v = 0; v < 9; ++v) st.Pb[v] = st.acc[v] = 0.0;
  }

  // Loads are issued a few at a time through the arithmetic.  A CU takes about
  // 66 cycles per wavefront load however many are waiting (its share of the
  // memory rate), and a wavefront stands still while its loads queue: issued
  // together, a layer's 79 (face states instead of gradients) held it up for
  // 16,000 of 62,000 cycles.
  // The 27 values of a ring slot (the neighbour's primitives and state on the
  // shared face, from the edge buffer, and its weights) are loaded by four
  // lanes, one per wavefront, so that no wavefront has them all: lane t takes
  // the values t / 64, t / 64 + 4, ...  (a slot without a neighbour, or the
  // 28th value, loads something that is not used)
  static constexpr int kRingShare = 7;
  __host__ __device__ static void fetch_ring(const AdjArgs& a, AState& st, int t, int k) {
    const Shape& g = a.d.g;
    const int64_t rc = (st.rc0 >= 0 ? st.rc0 : 0) + int64_t(k) * g.N * g.N;
    const int64_t rb = (st.rc0 >= 0 ? st.rb0 : 0) + int64_t(k) * kEdgeLayer;
#pragma unroll
    for (int e = 0; e < kRingShare; ++e) {
      const int v = (t >> 6) + 4 * e;  // the same in every lane of a wavefront: 0..17 edge rows, 18.. weights
      const int wr = v < 27 ? v - 18 : 8;
      st.ring[e] = v < 18 ? gld(a.B, rb + v * kEdgeSlots) : gld(a.w, wr * g.ncells + rc);
    }
  }
  // part 0..3 of layer k + 1's rows: gradients, then primitives and weights
  // (above the outermost layer the outer ghost's primitives; the gradients
  // there are loaded from layer k and not used, the ghost's weight, zero, is
  // put in where it is used)
  __host__ __device__ static void fetch_above(const AdjArgs& a, AState& st, int k, int part) {
    const Shape& g = a.d.g;
    const int64_t nc = g.ncells, c = cell_index(g, st.p, k, st.j, st.i);
    const bool top = k + 1 >= g.Nr;  // the same in every lane
    const int64_t up = top ? c : c + int64_t(g.N) * g.N;
    if (part < 3) {
#pragma unroll
      for (int v = 0; v < 9; ++v) st.G[9 * part + v] = gld(a.G, (9 * part + v) * nc + up);
      return;
    }
    const double* Pb = top ? a.Gs + 9 * g.nb : a.P;
    const int64_t Ps = top ? g.nb : nc, Po = top ? st.col : up;
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      st.Pp[v] = gld(Pb, v * Ps + Po);
      st.wp[v] = gld(a.w, v * nc + up);
    }
  }

  // Layer k's primitives and weights and the ring's values to LDS (nothing
  // the layer below's exchange reads).
  __host__ __device__ static void publish(const AdjArgs& a, const TileMap& tm, AState& st, int t, double* lds) {
    const Shape& g = a.d.g;
    if (st.act) {
      const int me = plane_pos(tile_i(st, t), t / kTI);
#pragma unroll
      for (int v = 0; v < 9; ++v) {
        lds[kP + v * kPlane + me] = st.P0[v];
        lds[kW + v * kPlane + me] = st.w0[v];
      }
    }
    if (st.rc0 >= 0) {
      const int r = t & 63, kind = r >> 4, idx = r & 15;
      const int tiL = (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
      const int tjL = (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
      const int ti = kind == 0 ? tiL + 1 : kind == 2 ? -1 : idx;
      const int tj = kind == 1 ? tjL + 1 : kind == 3 ? -1 : idx;
      const int pos = plane_pos(ti, tj);
      // the array the tile's cells read it from: an east neighbour is read as a west-face state, and so on
      const int q = kind == 0 ? 0 : kind == 1 ? 2 : kind == 2 ? 1 : 3;
#pragma unroll
      for (int e = 0; e < kRingShare; ++e) {
        const int v = (t >> 6) + 4 * e;
        const int at = v < 9 ? x_at(q, v) + kNT + idx : v < 18 ? kP + (v - 9) * kPlane + pos : kW + (v - 18) * kPlane + pos;
        if (v < 27) lds[at] = st.ring[e];
      }
    }
  }

  // Layer k's angular face states to LDS, once the layer below's
  // contributions are gone, and its state on the top face.
  __host__ __device__ static void publish_states(const AdjArgs& a, AState& st, int t, int k, double* lds) {
    if (!st.act) return;
    const GeomRef& G = a.d.G;
    const int me = plane_pos(tile_i(st, t), t / kTI);
    const double r0 = radius_uniform(G, k), r1 = radius_uniform(G, k + 1), rs = 0.125 * (r0 + r1);
    double P[9], q9[9];
#pragma unroll
    for (int v = 0; v < 9; ++v) P[v] = lds[kP + v * kPlane + me];
    recon9(P, st.G, r1 * st.xr - rs * centroid_sum(lds, me), st.qT);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      recon9(P, st.G, rs * face_offset(lds, q, t), q9);
#pragma unroll
      for (int v = 0; v < 9; ++v) lds[x_at(q, v) + t] = q9[v];
    }
  }

  // a face state's adjoint into Pb and Gb (ds: the face's offset from the centroid)
  __host__ __device__ static void face_state(AState& st, const double qb[9], V3 ds) {
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      st.Pb[v] += qb[v];
      st.Gb[3 * v] += qb[v] * ds.x;
      st.Gb[3 * v + 1] += qb[v] * ds.y;
      st.Gb[3 * v + 2] += qb[v] * ds.z;
    }
#pragma unroll
    for (int v = 0; v < 9; ++v) settle(st.Pb[v]);
#pragma unroll
    for (int v = 0; v < 27; ++v) settle(st.Gb[v]);
  }

  __host__ __device__ static V3 centroid_sum(const double* lds, int pos) {
    return mk(lds[kCs + pos], lds[kCs + kPlane + pos], lds[kCs + 2 * kPlane + pos]);
  }
  __host__ __device__ static V3 face_offset(const double* lds, int q, int t) {
    return mk(lds[kFe + (3 * q) * kNT + t], lds[kFe + (3 * q + 1) * kNT + t], lds[kFe + (3 * q + 2) * kNT + t]);
  }

  // the chunk's last layer loads its own again (unused)
  __host__ __device__ static int next_layer(const TileMap& tm, int k) { return k + 1 < tm.k1 ? k + 1 : k; }

  // All six faces of layer k's cell.
  __host__ __device__ static void faces(const AdjArgs& a, const TileMap& tm, AState& st, int t, int k,
                                        const double* lds) {
    if (!st.act) return;
    const Shape& g = a.d.g;
    const GeomRef& G = a.d.G;
    const int ti = tile_i(st, t), tj = t / kTI, me = plane_pos(ti, tj);
    const int tiL = (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
    const int tjL = (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
    const double r0 = radius_uniform(G, k), r1 = radius_uniform(G, k + 1);
    const double rs = 0.125 * (r0 + r1), ra = 0.5 * (r1 * r1 - r0 * r0);
    const V3 xc = rs * centroid_sum(lds, me);
#pragma unroll
    for (int v = 0; v < 27; ++v) st.Gb[v] = 0.0;
    fetch_above(a, st, k, 0);
    // bottom face: its flux adjoint came with the layer below
    face_state(st, st.qb, r0 * st.xr - xc);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int dx, dy;
      dir_offset(q, dx, dy);
      keep_order();
      const bool in = q == 0 ? ti > 0 : q == 1 ? ti < tiL : q == 2 ? tj > 0 : tj < tjL;
      // the neighbour's state on the face: its opposite direction's rows, at its lane or in the ring's entries
      const int qo_dir = q ^ 1, lane = in ? t + dx + dy * kTI : kNT + (q < 2 ? tj : ti);
      const int pos = plane_pos(ti + dx, tj + dy);
      const bool own = (st.own >> q) & 1u;
      const double sg = own ? 1.0 : -1.0;
      double qs[9], qo[9], wb[9], qb[9];
#pragma unroll
      for (int v = 0; v < 9; ++v) {
        qs[v] = lds[x_at(q, v) + t];
        qo[v] = lds[x_at(qo_dir, v) + lane];
        wb[v] = (lds[kW + v * kPlane + me] - lds[kW + v * kPlane + pos]) * sg;
        qb[v] = 0.0;
      }
      rusanov_adjoint_side(qs, qo, ra * st.fa[q], wb, qb, a.d.pr, own);
      face_state(st, qb, rs * face_offset(lds, q, t));
      if (q < 3) fetch_above(a, st, k, q + 1);
    }
    keep_order();
    // top face, both sides in one evaluation: the upper one is the next
    // layer's, or the outer ghost's
    {
      double wb[9], qLb[9], qRb[9], qn[9];
      // the state above: the next layer's, or the outer ghost's
      if (k + 1 < g.Nr) {
        recon9(st.Pp, st.G, r1 * st.xr - (0.125 * (r1 + radius_uniform(G, k + 2))) * centroid_sum(lds, me), qn);
      } else {
#pragma unroll
        for (int v = 0; v < 9; ++v) qn[v] = st.Pp[v];
      }
#pragma unroll
      for (int v = 0; v < 9; ++v) {
        wb[v] = lds[kW + v * kPlane + me] - (k == g.Nr - 1 ? 0.0 : st.wp[v]);
        qLb[v] = qRb[v] = 0.0;
      }
      rusanov_adjoint(st.qT, qn, (r1 * r1) * st.sr, wb, qLb, qRb, a.d.pr, true, true);
      face_state(st, qLb, r1 * st.xr - xc);
      if (k == g.Nr - 1)
        for (int v = 0; v < 9; ++v) gst(a.Gg, (9 + v) * g.nb + st.col, qRb[v]);
#pragma unroll
      for (int v = 0; v < 9; ++v) st.qb[v] = qRb[v];
    }
  }

  // The gradient and limiter adjoint of layer k's cell: contributions to its
  // neighbours to where they go (see above); the layer below, complete, is
  // written; the cell's own sum moves to acc.
  __host__ __device__ static void gradient(const AdjArgs& a, const TileMap& tm, AState& st, int t, int k, double* lds) {
    fetch_ring(a, st, t, next_layer(tm, k));
    if (!st.act) return;
    const Shape& g = a.d.g;
    const GeomRef& G = a.d.G;
    const int ti = tile_i(st, t), tj = t / kTI, me = plane_pos(ti, tj);
    const double r0 = radius_uniform(G, k), r1 = radius_uniform(G, k + 1);
    const double rs = 0.125 * (r0 + r1);
    const V3 cc = centroid_sum(lds, me), xc = rs * cc;
    V3 dx[6], dxf[6];
    int pos[4];
    const V3 xf0 = r0 * st.xr, xf1 = r1 * st.xr;
    dxf[0] = xf0 - xc;
    dxf[1] = xf1 - xc;
    dx[0] = k > 0 ? (0.125 * (radius_uniform(G, k - 1) + r0) - rs) * cc : ghost_centre(xc, (r0 * r0) * st.sr, xf0) - xc;
    dx[1] = k + 1 < g.Nr ? (0.125 * (r1 + radius_uniform(G, k + 2)) - rs) * cc
                         : ghost_centre(xc, (r1 * r1) * st.sr, xf1) - xc;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int ddx, ddy;
      dir_offset(q, ddx, ddy);
      pos[q] = plane_pos(ti + ddx, tj + ddy);
      dxf[2 + q] = rs * face_offset(lds, q, t);
      dx[2 + q] = rs * (centroid_sum(lds, pos[q]) - cc);
    }
    const LsqWeights Lw(dx);
    double up[9];
    const bool first = !Narrow || t % kTI == ti;  // the others add the same to the same entries
    const int64_t seam0 = k == tm.k0 && k > 0 ? int64_t(k / a.kc - 1) * 18 * g.nb : 0;
    const int64_t seam1 = k == tm.k1 - 1 && k + 1 < g.Nr ? int64_t(k / a.kc) * 18 * g.nb : 0;
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      keep_order();
      double qn[6];
      qn[0] = st.Pm[v];
      qn[1] = st.Pp[v];
#pragma unroll
      for (int q = 0; q < 4; ++q) qn[2 + q] = lds[kP + v * kPlane + pos[q]];
      const double pc = lds[kP + v * kPlane + me];
      double o[6];
      const double pb = variable_adjoint(Lw, dxf, a.d.pr.limiter, pc, qn, st.Gb[3 * v], st.Gb[3 * v + 1],
                                         st.Gb[3 * v + 2], o);
      const double own = st.Pb[v] + pb;
#pragma unroll
      for (int q = 0; q < 4; ++q) lds[x_at(q, v) + t] = o[2 + q];
      if (k == 0) {
        if (first) gst(a.Gg, v * g.nb + st.col, gld(a.Gg, v * g.nb + st.col) + o[0]);
      } else if (k == tm.k0)
        gst(a.S, seam0 + v * g.nb + st.col, o[0]);
      else
        st.acc[v] += o[0];  // of layer k - 1, now complete
      if (k == g.Nr - 1) {
        if (first) gst(a.Gg, (9 + v) * g.nb + st.col, gld(a.Gg, (9 + v) * g.nb + st.col) + o[1]);
      } else if (k == tm.k1 - 1)
        gst(a.S, seam1 + (9 + v) * g.nb + st.col, o[1]);
      up[v] = o[1];
      st.Pb[v] = own;
      settle(up[v]);
      settle(st.Pb[v]);
      settle(st.acc[v]);
      // the layer moves up
      st.P0[v] = st.Pp[v];
      st.w0[v] = st.wp[v];
    }
    if (k > tm.k0) emit(a, tm, st, t, k - 1, st.Pm, st.wg, lds);
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      st.acc[v] = st.Pb[v];
      st.Pb[v] = up[v];
      st.Pm[v] = lds[kP + v * kPlane + me];
    }
    layer_weights(lds, me, st.wg);
  }
  // the weights gravity's adjoint takes, from the plane
  __host__ __device__ static void layer_weights(const double* lds, int me, double wg[4]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) wg[d] = lds[kW + (1 + d) * kPlane + me];
    wg[3] = lds[kW + 7 * kPlane + me];
  }

  // One variable's gradient and limiter adjoint (gb: the limited gradient's
  // adjoint): returns the cell's own share and o, the six neighbours'.  The
  // limiter's choice is limited_grad's (its comment has the rule).
  __host__ __device__ static double variable_adjoint(const LsqWeights& Lw, const V3 dxf[6], int limiter, double qc,
                                                     const double qn[6], double gbx, double gby, double gbz,
                                                     double o[6]) {
    // (selects throughout: a branch per choice, most of them divergent, was
    // 45 blocks per variable)
    double gx = 0.0, gy = 0.0, gz = 0.0, qmax = qc, qmin = qc, pb = 0.0;
    int amax = -1, amin = -1;
#pragma unroll
    for (int lf = 0; lf < 6; ++lf) {
      const double dq = qn[lf] - qc;
      gx += Lw.W[lf].x * dq; gy += Lw.W[lf].y * dq; gz += Lw.W[lf].z * dq;
      const bool hi = !(qmax >= qn[lf]), lo = !(qmin <= qn[lf]);
      qmax = hi ? qn[lf] : qmax;
      amax = hi ? lf : amax;
      qmin = lo ? qn[lf] : qmin;
      amin = lo ? lf : amin;
      o[lf] = 0.0;
    }
    if (limiter) {
      double dhi = 0.0, dlo = 0.0;
      int fhi = 6, flo = 6;
#pragma unroll
      for (int f = 0; f < 6; ++f) {
        const double d2 = gx * dxf[f].x + gy * dxf[f].y + gz * dxf[f].z;
        const bool hi = d2 > dhi, lo = d2 < dlo;
        dhi = hi ? d2 : dhi;
        fhi = hi ? f : fhi;
        dlo = lo ? d2 : dlo;
        flo = lo ? f : flo;
      }
      const double up = qmax - qc, down = qc - qmin;
      const bool hi = up < dhi;  // the largest projection's ratio is below 1
      const double bn = hi ? up : 1.0, bd = hi ? dhi : 1.0;
      const double lhs = down * bd, rhs = bn * -dlo;
      const bool lo = (lhs < rhs) | ((lhs == rhs) & hi & (flo < fhi));
      const bool any = hi | lo;
      const int act = lo ? flo : hi ? fhi : -1;
      const double num = lo ? qmin - qc : qmax - qc;
      const double den = lo ? dlo : hi ? dhi : 1.0;
      const double rd = recip(den);
      const double phi = any ? ratio_refined(num, den) : 1.0;
      const double phib = any ? gbx * gx + gby * gy + gbz * gz : 0.0;
      gbx *= phi; gby *= phi; gbz *= phi;
      const double numb = any ? phib * rd : 0.0, denb = any ? -phib * phi * rd : 0.0;
      // den = g . dxf[act] (masked: a run-time index would put dxf in scratch)
#pragma unroll
      for (int f = 0; f < 6; ++f) {
        const double wf = f == act ? denb : 0.0;
        gbx += wf * dxf[f].x; gby += wf * dxf[f].y; gbz += wf * dxf[f].z;
      }
      const int ext = lo ? amin : amax;
      pb -= ext >= 0 ? numb : 0.0;
#pragma unroll
      for (int lf = 0; lf < 6; ++lf) o[lf] = ext == lf ? numb : 0.0;
    }
#pragma unroll
    for (int lf = 0; lf < 6; ++lf) {
      const double s = Lw.W[lf].x * gbx + Lw.W[lf].y * gby + Lw.W[lf].z * gbz;
      pb -= s;
      o[lf] += s;
    }
    return pb;
  }

  // write layer kk's cell: its gradient, or (left to the finishing pass) the
  // adjoint of its primitives
  __host__ __device__ static void emit(const AdjArgs& a, const TileMap& tm, const AState& st, int t, int kk,
                                       const double q[9], const double wg[4], const double* lds) {
    const Shape& g = a.d.g;
    const GeomRef& G = a.d.G;
    const double r0 = radius_uniform(G, kk), r1 = radius_uniform(G, kk + 1);
    double Ub[9];
    prim_adjoint_prims(q, st.acc, Ub, a.d.pr.gamma);
    const double vol = (r1 * r1 * r1 - r0 * r0 * r0) * st.om * (1.0 / 3.0);
    gravity_adjoint((0.125 * (r0 + r1)) * centroid_sum(lds, plane_pos(tile_i(st, t), t / kTI)), vol, a.d.pr.G, wg, Ub);
    const bool raw = st.edge || kk == 0 || kk == g.Nr - 1 || kk == tm.k0 || kk == tm.k1 - 1;
    const int64_t c = cell_index(g, st.p, kk, st.j, st.i);
#pragma unroll
    for (int v = 0; v < 9; ++v) gst(a.gU, v * g.ncells + c, raw ? st.acc[v] : Ub[v]);
  }

  // The in-tile neighbours' contributions; the tile edges' to the edge buffer
  // (one wavefront, coalesced).
  __host__ __device__ static void gather(const AdjArgs& a, const TileMap& tm, AState& st, int t, int k,
                                         const double* lds) {
    const Shape& g = a.d.g;
    const int ti = tile_i(st, t), tj = t / kTI;
    const int tiL = (g.N - tm.i0 < kTI ? g.N - tm.i0 : kTI) - 1;
    const int tjL = (g.N - tm.j0 < kTJ ? g.N - tm.j0 : kTJ) - 1;
    if (t >= 2 * kEdgeSlots && t < 3 * kEdgeSlots) {
      const int r = t - 2 * kEdgeSlots, kind = r >> 4, idx = r & 15;
      const int eti = kind == 0 ? tiL : kind == 2 ? 0 : idx, etj = kind == 1 ? tjL : kind == 3 ? 0 : idx;
      if (eti <= tiL && etj <= tjL) {
        const int q = kind == 0 ? 1 : kind == 1 ? 3 : kind == 2 ? 0 : 2;
        const int64_t e = (march_tile_index(g, tm.p, tm.j0, tm.i0) * g.Nr + k) * kAdjEdgeLayer + r;
#pragma unroll
        for (int v = 0; v < 9; ++v) gst(a.E, e + v * kEdgeSlots, lds[x_at(q, v) + etj * kTI + eti]);
      }
    }
    if (!st.act) return;
    if (ti > 0)
#pragma unroll
      for (int v = 0; v < 9; ++v) st.acc[v] += lds[x_at(1, v) + t - 1];
    if (ti < tiL)
#pragma unroll
      for (int v = 0; v < 9; ++v) st.acc[v] += lds[x_at(0, v) + t + 1];
    if (tj > 0)
#pragma unroll
      for (int v = 0; v < 9; ++v) st.acc[v] += lds[x_at(3, v) + t - kTI];
    if (tj < tjL)
#pragma unroll
      for (int v = 0; v < 9; ++v) st.acc[v] += lds[x_at(2, v) + t + kTI];
    // the chunk's last layer (its sum is never complete here)
    if (k == tm.k1 - 1) {
      double q[9], wg[4];
      const int me = plane_pos(ti, tj);
#pragma unroll
      for (int v = 0; v < 9; ++v) q[v] = lds[kP + v * kPlane + me];
      layer_weights(lds, me, wg);
      emit(a, tm, st, t, k, q, wg, lds);
    }
  }
};

using AdjWG = AdjMarch<true>;  // whichever the shell (the host emulation)

// Per boundary column, side and input a of the boundary law (0..8 the cell's
// primitives, 9 the B_r map): the ghost state's adjoint through the law, one
// forward derivative each (ghost_adjoint of cfv_vjp.hpp runs the ten one
// after the other).
__host__ __device__ inline void adj_ghost_input(const AdjArgs& a, int64_t col, int side, int in) {
  const Shape& g = a.d.g;
  int p, j, i;
  column_pji(g, col, p, j, i);
  const int k = side == 0 ? 0 : g.Nr - 1;
  const int64_t c = cell_index(g, p, k, j, i);
  Dual q[9], qG[9];
#pragma unroll
  for (int v = 0; v < 9; ++v) q[v] = Dual(gld(a.P, v * g.ncells + c), v == in ? 1.0 : 0.0);
  V3 xG;
  ghost_prims(a.d, p, k, j, i, side, q, cell_centre(a.d.G, g, p, k, j, i),
              Dual(side == 0 ? gld(a.d.br, col) : 0.0, in == 9 ? 1.0 : 0.0), qG, xG);
  double s = 0.0;
#pragma unroll
  for (int v = 0; v < 9; ++v) s += qG[v].d * gld(a.Gg, (9 * side + v) * g.nb + col);
  if (in < 9) gst(a.Gp, (9 * side + in) * g.nb + col, s);
  else gst(a.gbr, col, s);
}

// A cell the march left unfinished: the contributions from beyond its tile,
// its chunk and the boundaries, then its gradient.
__host__ __device__ inline void adjoint_finish_cell(const AdjArgs& a, int64_t c) {
  const Shape& g = a.d.g;
  int p, k, j, i;
  decode(g, c, p, k, j, i);
  if (!adj_unfinished(g, a.kc, k, j, i)) return;
  const int64_t nc = g.ncells, col = column_of(g, p, j, i);
  double Pb[9], u[9], wg[4], Ub[9];
#pragma unroll
  for (int v = 0; v < 9; ++v) {
    Pb[v] = gld(a.gU, v * nc + c);
    u[v] = gld(a.U, v * nc + c);
  }
#pragma unroll
  for (int d = 0; d < 4; ++d) wg[d] = gld(a.w, (d < 3 ? 1 + d : 7) * nc + c);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int ti = i % kTI, tj = j % kTJ;
    const bool out = q == 0 ? ti == 0 : q == 1 ? (ti == kTI - 1 || i == g.N - 1) : q == 2 ? tj == 0
                                                                                  : (tj == kTJ - 1 || j == g.N - 1);
    if (!out) continue;
    int np, nj, ni;
    column_pji(g, gld(a.d.G.cn, q * a.d.G.ncol + col), np, nj, ni);
    const int back = (gld(a.d.G.cn, (4 + q) * a.d.G.ncol + col) & 0xff) - 2;
    const int kind = back == 1 ? 0 : back == 3 ? 1 : back == 0 ? 2 : 3;
    const int64_t e = (march_tile_index(g, np, nj - nj % kTJ, ni - ni % kTI) * g.Nr + k) * kAdjEdgeLayer + kind * 16 +
                      ((kind & 1) ? ni % kTI : nj % kTJ);
#pragma unroll
    for (int v = 0; v < 9; ++v) Pb[v] += gld(a.E, e + v * kEdgeSlots);
  }
  if (k % a.kc == 0 && k > 0) {  // up from the chunk below
    const int64_t s = int64_t(k / a.kc - 1) * 18 * g.nb + 9 * g.nb + col;
#pragma unroll
    for (int v = 0; v < 9; ++v) Pb[v] += gld(a.S, s + v * g.nb);
  }
  if (k % a.kc == a.kc - 1 && k + 1 < g.Nr) {  // down from the chunk above
    const int64_t s = int64_t(k / a.kc) * 18 * g.nb + col;
#pragma unroll
    for (int v = 0; v < 9; ++v) Pb[v] += gld(a.S, s + v * g.nb);
  }
  if (k == 0)
#pragma unroll
    for (int v = 0; v < 9; ++v) Pb[v] += gld(a.Gp, v * g.nb + col);
  if (k == g.Nr - 1)
#pragma unroll
    for (int v = 0; v < 9; ++v) Pb[v] += gld(a.Gp, (9 + v) * g.nb + col);
  prim_adjoint(u, Pb, Ub, a.d.pr.gamma);
  gravity_adjoint(cell_centre(a.d.G, g, p, k, j, i), cell_volume(a.d.G, g, p, k, j, i), a.d.pr.G, wg, Ub);
#pragma unroll
  for (int v = 0; v < 9; ++v) gst(a.gU, v * nc + c, Ub[v]);
}

}  // namespace cfv
