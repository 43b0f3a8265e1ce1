// The Arnoldi step's vector kernels (see cfv_krylov.hpp).  All sums have a
// fixed order (lanes of a wavefront as a tree, a block's tiles in order,
// wavefronts in order, blocks in order), so results are reproducible; no
// atomics.
//
// What bounds it: memory.  On the 1.66M-cell shell (119 MB a vector) the two
// passes over the basis run at 4.5 (dots) and 5.4 TB/s (update) against 5.1
// for a copy; a GMRES(30) sweep of them takes 27 ms where one pass per basis
// vector and projection took 44.  On small shells it was launches: a step
// with basis size j took 2 (j + 1) + 3 of them and takes 4 now, 46 instead of
// 130 us per step at 61,440 cells and j = 15.
//
// Every vector is read 16 bytes per lane: the library owns all of them (a
// vector has 9 x 6 N^2 Nr entries, an even number, so each starts on a
// 16-byte boundary).
#include "cfv_krylov.hpp"

#include "cfv_math.hpp"

namespace cfv {

namespace {
constexpr int kT = kKrylovThreads, kPairs = kKrylovEntries / 2, kWaves = kT / 64;

typedef double Pair __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Pair pair(double a, double b) { return Pair{a, b}; }

__device__ __forceinline__ Pair ld2(const double* p, int64_t i) {
  return *(const __attribute__((address_space(1))) Pair*)(p + i);
}
__device__ __forceinline__ void st2(double* p, int64_t i, Pair v) {
  *(__attribute__((address_space(1))) Pair*)(p + i) = v;
}

// sum over the wavefront of a (returned in lanes 0..31's lane 0) and of b
// (lane 32): the first exchange swaps halves, so both take one reduction
__device__ __forceinline__ double wave_sum_pair(double a, double b) {
  const bool low = (threadIdx.x & 63) < 32;
  double x = low ? a : b;
  x += __shfl_xor(low ? b : a, 32, 64);
  for (int o = 16; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ double wave_sum(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

__device__ __forceinline__ const KrylovSys& system_of(const KrylovSys* sys, const int32_t* owner) {
  return sys[owner ? owner[blockIdx.x] : 0];
}
}  // namespace

// V_{j+1} = w + diag x, and the block's partial sums of <V_i, V_{j+1}> (i <= j)
// and <V_i, V_j> (i < j).  With the preconditioner x = D^-1 V_j, so diag x is
// V_j itself.  A tile's entries of V_{j+1} and V_j stay in registers while the
// basis streams past, so the pass reads each basis vector once.  blockIdx.y
// takes a group of `group` basis vectors, so that short vectors fill the chip
// too: each group reads w, V_j and the diagonal and forms V_{j+1}'s entries
// again, the first one stores them.
__global__ __launch_bounds__(kT) void krylov_dots_kernel(const KrylovSys* __restrict__ sys,
                                                         const int32_t* __restrict__ owner, int j, int group) {
  __shared__ double acc[kWaves][2 * (kKrylovMaxM + 1)];
  const KrylovSys& S = system_of(sys, owner);
  const int64_t n = S.n, nc = S.nc;
  const int b = int(blockIdx.x) - S.b0, nb = S.nb;
  const int i0 = int(blockIdx.y) * group, i1 = i0 + group < j + 1 ? i0 + group : j + 1;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double* __restrict__ V = S.V;
  const double* __restrict__ vj = V + int64_t(j) * n;
  double* __restrict__ vn = S.V + int64_t(j + 1) * n;
  if ((lane & 31) == 0)  // lane 0 owns the even entries, lane 32 the odd ones
    for (int i = i0; i < i1; ++i) acc[wv][2 * (i - i0) + (lane >> 5)] = 0.0;
  for (int64_t tile = b; tile * kKrylovTile < n; tile += nb) {
    const int64_t e0 = tile * kKrylovTile + 2 * threadIdx.x;
    Pair x[kPairs], u[kPairs];
    bool in[kPairs];
#pragma unroll
    for (int q = 0; q < kPairs; ++q) {
      const int64_t e = e0 + 2 * kT * q;
      in[q] = e < n;
      x[q] = u[q] = pair(0.0, 0.0);
      if (!in[q]) continue;
      x[q] = ld2(S.w, e);
      u[q] = ld2(vj, e);
      if (S.z) {
        x[q].x += u[q].x;
        x[q].y += u[q].y;
      } else {
        const Pair d = ld2(S.diag, e % nc);  // nc is even: a pair never spans two variables
        x[q].x += d.x * u[q].x;
        x[q].y += d.y * u[q].y;
      }
      if (blockIdx.y == 0) st2(vn, e, x[q]);
    }
#pragma unroll 4
    for (int i = i0; i < i1; ++i) {
      const double* __restrict__ vi = V + int64_t(i) * n;
      double sx = 0.0, su = 0.0;
#pragma unroll
      for (int q = 0; q < kPairs; ++q) {
        const Pair y = ld2(vi, in[q] ? e0 + 2 * kT * q : 0);  // beyond the end: times zero
        sx += y.x * x[q].x;
        sx += y.y * x[q].y;
        su += y.x * u[q].x;
        su += y.y * u[q].y;
      }
      const double t = wave_sum_pair(sx, su);
      if ((lane & 31) == 0) acc[wv][2 * (i - i0) + (lane >> 5)] += t;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 2 * (i1 - i0); q += kT) {
    double t = 0.0;
    for (int w2 = 0; w2 < kWaves; ++w2) t += acc[w2][q];
    S.part[int64_t(2 * i0 + q) * nb + b] = t;
  }
}

// The column's coefficients: fold the partial sums into a = V^T w and the row
// t = V^T v_j, append row j of M = (I + L)^-1 (row j of I + L is t, so the
// row is e_j - t^T M), and h = M a.  One workgroup per system: a dot product
// per wavefront, no serial chain over the basis.
constexpr int kCoeffThreads = 1024;
__global__ __launch_bounds__(kCoeffThreads) void krylov_coeff_kernel(const KrylovSys* __restrict__ sys, int m, int j) {
  constexpr int kW = kCoeffThreads / 64;
  __shared__ double a[kKrylovMaxM + 1], t[kKrylovMaxM + 1], row[kW][kKrylovMaxM + 1];
  const KrylovSys& S = sys[blockIdx.x];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int q = wv; q < 2 * (j + 1); q += kW) {
    const double* p = S.part + int64_t(q) * S.nb;
    double s = 0.0;
#pragma unroll 8
    for (int b = lane; b < S.nb; b += 64) s += p[b];
    s = wave_sum(s);
    if (lane == 0) ((q & 1) ? t : a)[q >> 1] = s;
  }
  __syncthreads();
  // partial rows of t^T M: wavefront wv takes k = wv, wv + kW, ...
  for (int c = lane; c < j; c += 64) {
    double s = 0.0;
    for (int k = wv; k < j; k += kW)
      if (k >= c) s += t[k] * S.M[int64_t(k) * m + c];
    row[wv][c] = s;
  }
  __syncthreads();
  for (int c = threadIdx.x; c <= j; c += kCoeffThreads) {
    double s = 0.0;
    if (c < j)
      for (int q = 0; q < kW; ++q) s -= row[q][c];
    const double r = c == j ? 1.0 : s;
    S.M[int64_t(j) * m + c] = r;
    t[c] = r;  // row j of M (t itself is no longer needed)
  }
  __syncthreads();
  for (int i = wv; i <= j; i += kW) {
    double s = 0.0;
    for (int k = lane; k <= i; k += 64) s += (i == j ? t[k] : S.M[int64_t(i) * m + k]) * a[k];
    s = wave_sum(s);
    if (lane == 0) S.H[int64_t(j) * (m + 2) + i] = s;
  }
}

// V_{j+1} -= sum_i h_i V_i and the block's partial sum of its squares
__global__ __launch_bounds__(kT) void krylov_update_kernel(const KrylovSys* __restrict__ sys,
                                                           const int32_t* __restrict__ owner, int m, int j) {
  __shared__ double h[kKrylovMaxM + 1], sh[kWaves];
  const KrylovSys& S = system_of(sys, owner);
  const int64_t n = S.n;
  const int b = int(blockIdx.x) - S.b0, nb = S.nb;
  const double* __restrict__ V = S.V;
  double* __restrict__ vn = S.V + int64_t(j + 1) * n;
  for (int i = threadIdx.x; i <= j; i += kT) h[i] = S.H[int64_t(j) * (m + 2) + i];
  __syncthreads();
  double s = 0.0;
  for (int64_t tile = b; tile * kKrylovTile < n; tile += nb) {
    const int64_t e0 = tile * kKrylovTile + 2 * threadIdx.x;
    Pair x[kPairs];
#pragma unroll
    for (int q = 0; q < kPairs; ++q)
      x[q] = e0 + 2 * kT * q < n ? ld2(vn, e0 + 2 * kT * q) : pair(0.0, 0.0);
#pragma unroll 8
    for (int i = 0; i <= j; ++i) {
      const double* __restrict__ vi = V + int64_t(i) * n;
      const double hi = h[i];
#pragma unroll
      for (int q = 0; q < kPairs; ++q) {
        const int64_t e = e0 + 2 * kT * q;
        const Pair y = ld2(vi, e < n ? e : 0);  // beyond the end: not stored, not summed
        x[q].x -= hi * y.x;
        x[q].y -= hi * y.y;
      }
    }
#pragma unroll
    for (int q = 0; q < kPairs; ++q) {
      if (e0 + 2 * kT * q >= n) continue;
      st2(vn, e0 + 2 * kT * q, x[q]);
      s += x[q].x * x[q].x;
      s += x[q].y * x[q].y;
    }
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int q = 0; q < kWaves; ++q) r += sh[q];
    S.part[int64_t(2 * (m + 1)) * nb + b] = r;
  }
}

// h_{j+1,j} = |V_{j+1}| (every block folds the partial sums itself, in one
// order), V_{j+1} /= h, z = V_{j+1} / diag; the first block stores h and the
// host's copy of the column.
__global__ __launch_bounds__(kT) void krylov_scale_kernel(const KrylovSys* __restrict__ sys,
                                                          const int32_t* __restrict__ owner, int m, int j) {
  __shared__ double sh[kWaves];
  const KrylovSys& S = system_of(sys, owner);
  const int64_t n = S.n, nc = S.nc;
  const int b = int(blockIdx.x) - S.b0, nb = S.nb;
  double* __restrict__ vn = S.V + int64_t(j + 1) * n;
  const double* __restrict__ p = S.part + int64_t(2 * (m + 1)) * nb;
  double s = 0.0;
#pragma unroll 2
  for (int q = threadIdx.x; q < nb; q += kT) s += p[q];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  double t = 0.0;
  for (int q = 0; q < kWaves; ++q) t += sh[q];
  const double h = ::sqrt(t);
  if (b == 0) {
    double* col = S.H + int64_t(j) * (m + 2);
    if (threadIdx.x == 0) col[j + 1] = h;
    if (S.host_H)
      for (int i = threadIdx.x; i <= j + 1; i += kT) S.host_H[int64_t(j) * (m + 2) + i] = i <= j ? col[i] : h;
  }
  const bool live = h > 0.0;
  for (int64_t tile = b; tile * kKrylovTile < n; tile += nb) {
#pragma unroll
    for (int q = 0; q < kPairs; ++q) {
      const int64_t e = tile * kKrylovTile + 2 * threadIdx.x + 2 * kT * q;
      if (e >= n) continue;
      const Pair x = ld2(vn, e);
      const Pair y = live ? pair(x.x / h, x.y / h) : pair(0.0, 0.0);
      st2(vn, e, y);
      if (S.z) {
        const Pair d = ld2(S.diag, e % nc);
        st2(S.z, e, pair(y.x / d.x, y.y / d.y));
      }
    }
  }
}

// out = base + D^-1 V y (base null: zero; D only with the preconditioner).
// base and out are the caller's: 8-byte accesses.
__global__ __launch_bounds__(kT) void krylov_combine_kernel(const KrylovSys* __restrict__ sys,
                                                            const KrylovOut* __restrict__ out,
                                                            const int32_t* __restrict__ owner) {
  __shared__ double y[kKrylovMaxM + 1];
  const int q0 = owner ? owner[blockIdx.x] : 0;
  const KrylovSys& S = sys[q0];
  const KrylovOut& O = out[q0];
  const int64_t n = S.n, nc = S.nc;
  const int b = int(blockIdx.x) - S.b0, nb = S.nb;
  const int k = O.kdone ? int(*O.kdone) : O.k;
  for (int i = threadIdx.x; i < k; i += kT) y[i] = O.y[i];
  __syncthreads();
  for (int64_t tile = b; tile * kKrylovTile < n; tile += nb) {
    const int64_t e0 = tile * kKrylovTile + 2 * threadIdx.x;
    Pair x[kPairs];
#pragma unroll
    for (int q = 0; q < kPairs; ++q) x[q] = pair(0.0, 0.0);
#pragma unroll 8
    for (int i = 0; i < k; ++i) {
      const double* __restrict__ vi = S.V + int64_t(i) * n;
      const double yi = y[i];
#pragma unroll
      for (int q = 0; q < kPairs; ++q) {
        const int64_t e = e0 + 2 * kT * q;
        const Pair v = ld2(vi, e < n ? e : 0);  // beyond the end: not stored
        x[q].x += yi * v.x;
        x[q].y += yi * v.y;
      }
    }
#pragma unroll
    for (int q = 0; q < kPairs; ++q) {
      const int64_t e = e0 + 2 * kT * q;
      if (e >= n) continue;
      if (S.z) {
        const Pair d = ld2(S.diag, e % nc);
        x[q].x /= d.x;
        x[q].y /= d.y;
      }
      const double b0 = O.base ? gld(O.base, e) : 0.0, b1 = O.base ? gld(O.base, e + 1) : 0.0;
      gst(O.out, e, b0 + x[q].x);
      gst(O.out, e + 1, b1 + x[q].y);
    }
  }
}

__global__ void krylov_put_kernel(KrylovSys a, KrylovOut b, KrylovSys* __restrict__ sys, KrylovOut* __restrict__ out) {
  *sys = a;
  *out = b;
}

hipError_t launch_krylov_put(const KrylovSys& a, const KrylovOut& b, KrylovSys* sys, KrylovOut* out, hipStream_t s) {
  hipLaunchKernelGGL(krylov_put_kernel, dim3(1), dim3(1), 0, s, a, b, sys, out);
  return hipGetLastError();
}

hipError_t launch_krylov_combine(const KrylovSys* sys, const KrylovOut* out, const int32_t* owner, int blocks,
                                 hipStream_t s) {
  hipLaunchKernelGGL(krylov_combine_kernel, dim3(unsigned(blocks)), dim3(kT), 0, s, sys, out, owner);
  return hipGetLastError();
}

hipError_t launch_krylov_step(const KrylovSys* sys, const int32_t* owner, int systems, int blocks, int m, int j,
                              hipStream_t s) {
  // groups of basis vectors: enough of them that with the blocks every CU has
  // four workgroups (1,024).  One system has at most kKrylovMaxBlocks blocks, so
  // two groups or more; the ensemble's blocks, about 1,024, fall a little short
  // of it and make two.
  int groups = (1024 + blocks - 1) / blocks;
  if (groups > j + 1) groups = j + 1;
  const int group = (j + 1 + groups - 1) / groups;
  groups = (j + 1 + group - 1) / group;
  hipLaunchKernelGGL(krylov_dots_kernel, dim3(unsigned(blocks), unsigned(groups)), dim3(kT), 0, s, sys, owner, j, group);
  hipLaunchKernelGGL(krylov_coeff_kernel, dim3(unsigned(systems)), dim3(kCoeffThreads), 0, s, sys, m, j);
  hipLaunchKernelGGL(krylov_update_kernel, dim3(unsigned(blocks)), dim3(kT), 0, s, sys, owner, m, j);
  hipLaunchKernelGGL(krylov_scale_kernel, dim3(unsigned(blocks)), dim3(kT), 0, s, sys, owner, m, j);
  return hipGetLastError();
}

}  // namespace cfv
