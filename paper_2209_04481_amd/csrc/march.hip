// Tiled two-pass radial-march kernels: the forward derivative (JVP, T =
// Dual) and the VJP's forward pass (T = double, face states written); the
// residual itself runs as one fused pass (fused.hip).
//
// A workgroup owns a 16 x 16 tile of columns (i, j) of one panel and a chunk
// of radial layers, and marches upward in k:
//
//  grad pass  per layer: each thread converts its cell to primitives once and
//             publishes them in LDS; the least-squares gradient and the
//             Barth-Jespersen factor then read in-tile neighbours from LDS,
//             radial neighbours from registers (the march keeps layers k-1,
//             k, k+1), and only tile-edge neighbours from global memory.
//             Output: the limited gradient (27 values per cell).
//  flux pass  per layer: each thread reconstructs its six face states; the
//             west and south states go to LDS, so every angular face inside
//             the tile is evaluated once, by its east/north cell; the radial
//             face between k-1 and k is evaluated once from the state carried
//             in registers.  Face fluxes are exchanged through LDS and summed
//             with the sign of the side (canonical owner orientation).
//
// Both passes are written as barrier-separated phase functions over a
// per-thread state, so the same code also runs under a host emulation.  A
// chunk enters and leaves through warm-up and cool-down iterations of the
// same phases, so the outputs do not depend on the chunk length.
#include "cfv_kernels.hpp"
#include "cfv_march.hpp"

namespace cfv {

// --------------------------------------------------------------- device glue
// One (tile, chunk) of each pass; the single-instance kernels run one per
// workgroup, the ensemble kernels (ensemble.hip) loop over a queue of them.
template <class T, int Mode = 0, bool Ahead = true>
__device__ __forceinline__ void grad_march_tile(const MarchArgs& a0, const TileMap& tm, double* lds) {
  using WG = GradWG<T, Ahead>;
  const int t = threadIdx.x;
  GState<T> st;
  WG::init(a0, tm, st, t, lds);
  for (int k = WG::first_layer(tm); k < tm.k1; ++k) {
    const MarchArgs& a = per_layer(a0);
    // (the second wavefront also fills the plane's ring of out-of-tile
    // neighbours)
    WG::publish(a, tm, st, t, k, lds);
    if (k < tm.k0) continue;  // warm-up: registers only
    __syncthreads();
    WG::template compute<Mode>(a, tm, st, t, k, lds);
    // the plane is written again by the next layer (a second plane to drop
    // this barrier made both gradient passes slower: more LDS per workgroup)
    __syncthreads();
    // the staged tile-edge states, written again only after the next layer's
    // first barrier
    if (sizeof(T) > sizeof(double) || Mode == 2) WG::flush_edges(a, tm, t, k, lds);
  }
}

template <class T>
__device__ __forceinline__ void flux_march_tile(const MarchArgs& a0, const TileMap& tm, double* lds) {
  const int t = threadIdx.x;
  FState<T> st;
  FluxWG<T>::init(a0, tm, st, t);
  const int kl = FluxWG<T>::last_layer(a0.d.g, tm);
  for (int k = FluxWG<T>::first_layer(tm); k <= kl; ++k) {
    const MarchArgs& a = per_layer(a0);
    FluxWG<T>::states(a, tm, st, lane_here(t), k, lds);
    if (k < tm.k0 || k >= tm.k1) continue;  // warm-up or cool-down: registers only
    __syncthreads();
    FluxWG<T>::faces(a, tm, st, lane_here(t), k, lds);
    __syncthreads();
    // no barrier after it: the next layer's states and ring slots overwrite
    // buffers that only the face phase (before the barrier above) reads
    FluxWG<T>::accumulate(a, tm, st, lane_here(t), k, lds);
  }
  FluxWG<T>::finish(a0, tm, st, t);
}

// ----------------------------------------------------------------- ensemble
__global__ void reset_counters_kernel(unsigned* c) {
  if (threadIdx.x < 2) c[threadIdx.x] = 0u;
}

// next item of this workgroup: static (XCD-aware strided) or from the queue
__device__ __forceinline__ int64_t next_item(const EnsembleLaunch& e, int64_t step, unsigned* counter, int* slot) {
  if (e.queue) {
    __syncthreads();  // every thread has read the previous slot
    if (threadIdx.x == 0) *slot = int(atomicAdd(counter, 1u));
    __syncthreads();
    return *slot;
  }
  // workgroup b sits on XCD b % 8 as the (b / 8)-th of Q = blocks / 8; the
  // XCD's workgroups share a contiguous eighth of the queue
  const int64_t Q = e.blocks / 8, per = (e.total + 7) / 8;
  const int64_t x = blockIdx.x % 8, r = blockIdx.x / 8;
  const int64_t w = r + step * Q, idx = x * per + w;
  return w < per && idx < e.total ? idx : e.total;
}

// the item index is the same in every lane: say so, so that descriptor and
// table reads become scalar loads
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint64_t u = uint64_t(v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(u));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(u >> 32));
  return int64_t((uint64_t(hi) << 32) | lo);
}

__device__ __forceinline__ int find_instance(const int64_t* __restrict__ off, int n, int64_t w) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= w) lo = mid; else hi = mid;
  }
  return lo;
}

// One wavefront per SIMD where the next layer's loads wait in registers: the
// JVP passes (474 and 512 of them; the flux pass also has 160 KB of LDS) and
// the VJP's forward passes (377; at two per SIMD they spill, 2.26 against 1.52
// ms at 13.3M cells).  The forward pass without loads ahead: two, 160 B of
// scratch a lane.
// Aligned, so that what else is compiled here does not move them: the JVP
// passes are 65 and 71 KB against a 64 KB instruction cache, and 1 KB further on
// the same instructions took up to 1% longer (21 x 37 124.0 against 122.8 us, 8 x
// 60 76.0 against 75.0; alignments of 1, 2, 4 and 8 KB within 0.5%).
template <class T, bool Flux, int Mode = 0, bool Ahead = true>
__attribute__((aligned(2048))) __global__
__launch_bounds__(kNT, Ahead ? 1 : 2) void march_ensemble_kernel(EnsembleLaunch e, MarchArgs) {
  constexpr int kL = Flux ? FluxWG<T>::kLds : GradWG<T>::kLds;
  __shared__ double lds[kL];
  __shared__ int slot;
  unsigned* counter = e.counters + (Flux ? 1 : 0);
  for (int64_t step = 0;; ++step) {
    const int64_t q = uniform(next_item(e, step, counter, &slot));
    if (q >= e.total) break;
    const int64_t w = e.perm ? uniform(e.perm[q]) : q;
    const int inst = e.n > 1 ? int(uniform(find_instance(e.item_off, e.n, w))) : 0;
    const MarchArgs& a = constant_args(e.args ? e.args + inst : second_kernel_arg<EnsembleLaunch, MarchArgs>());
    TileMap tm;
    tile_of_logical(a.d.g, e.n > 1 ? w - e.item_off[inst] : w, tm, e.kc);
    __syncthreads();  // the previous item's LDS reads are done
    if (Flux)
      flux_march_tile<T>(a, tm, lds);
    else
      grad_march_tile<T, Mode, Ahead>(a, tm, lds);
  }
}

// dual: the JVP's two passes; otherwise the fused residual march, and e must
// then describe its items (fused_items per instance, chunks of e.kc layers)
hipError_t launch_march_ensemble(const EnsembleLaunch& e, bool dual, hipStream_t s, KernelTimer* t) {
  if (e.total <= 0) return hipSuccess;
  if (!dual) return launch_fused_ensemble(e, kOutResidual, s, t);
  if (e.queue) hipLaunchKernelGGL(reset_counters_kernel, dim3(1), dim3(64), 0, s, e.counters);
  {
    TimedScope ts(t, "grad_march_ens_jvp", s);
    hipLaunchKernelGGL((march_ensemble_kernel<Dual, false>), dim3(e.blocks), dim3(kNT), 0, s, e, MarchArgs{});
  }
  TimedScope ts(t, "flux_march_ens_jvp", s);
  hipLaunchKernelGGL((march_ensemble_kernel<Dual, true>), dim3(e.blocks), dim3(kNT), 0, s, e, MarchArgs{});
  return hipGetLastError();
}

// One instance: its descriptor travels with the launch (a copy of its own into
// device memory was one more launch, 4 us of a 30 us residual on a small
// shell); the same persistent kernels run with one workgroup per item (no
// queue, no table).
static EnsembleLaunch one_instance(const MarchArgs& a, int kc) {
  return EnsembleLaunch{nullptr, nullptr, nullptr, nullptr, 1, march_logical_blocks(a.d.g, kc), 0,
                        unsigned(march_blocks(a.d.g, kc)), kc};
}

hipError_t launch_march(const MarchArgs& a, bool dual, int kc, hipStream_t s, KernelTimer* t) {
  if (!dual) return launch_fused(a, kc, kOutResidual, s, t);  // the residual: one fused pass (fused.hip)
  if (!a.E) return hipErrorInvalidValue;  // the flux pass's ring reads the tile-edge states
  const EnsembleLaunch e = one_instance(a, kc);
  {
    TimedScope ts(t, "grad_march_jvp", s);
    hipLaunchKernelGGL((march_ensemble_kernel<Dual, false>), dim3(e.blocks), dim3(kNT), 0, s, e, a);
  }
  TimedScope ts(t, "flux_march_jvp", s);
  hipLaunchKernelGGL((march_ensemble_kernel<Dual, true>), dim3(e.blocks), dim3(kNT), 0, s, e, a);
  return hipGetLastError();
}

hipError_t launch_march_grad(const MarchArgs& a, int kc, bool ahead, hipStream_t s, KernelTimer* t) {
  const EnsembleLaunch e = one_instance(a, kc);
  TimedScope ts(t, "grad_march_fwd", s);
  if (a.Q && !ahead)
    hipLaunchKernelGGL((march_ensemble_kernel<double, false, 1, false>), dim3(e.blocks), dim3(kNT), 0, s, e, a);
  else if (a.Q)
    hipLaunchKernelGGL((march_ensemble_kernel<double, false, 1>), dim3(e.blocks), dim3(kNT), 0, s, e, a);
  else
    hipLaunchKernelGGL((march_ensemble_kernel<double, false, 2>), dim3(e.blocks), dim3(kNT), 0, s, e, a);
  return hipGetLastError();
}

}  // namespace cfv
