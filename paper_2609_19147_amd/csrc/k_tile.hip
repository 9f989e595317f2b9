// Tile passes: multi-qubit butterflies staged through LDS.
//
// One workgroup owns one coset of the tile bits [0, L) U [a, a+h): it loads
// the coset's 2^m amplitudes (m = L + h) with 16-byte accesses -- runs of 2^L
// consecutive amplitudes, so every access is coalesced -- into LDS, runs the
// pass's rounds and stores the tile back in place.  A round moves, per
// thread, the 2^4 amplitudes that differ in the round's four tile bits into
// registers, multiplies them by a diagonal layer's phase if the round carries
// one, applies the round's single-bit operations and writes them back.
//
// Operations (paper, Section "Kernel Taxonomy"): per-wire 2x2 products of a
// single-qubit window (tensor-product layers), Hadamard butterflies (Walsh
// layers), and QFT stages -- the Hadamard butterfly of bit p followed by the
// stage's whole controlled-phase ladder as one twiddle exp(i pi low / 2^p),
// low = index mod 2^p.  The twiddle splits into a per-register-group factor
// (bits outside the round, one sincospi per group) times a host-built
// intra-round factor.
#include "kernels.h"
#include "rho.h"
#include "tile_rounds.h"

namespace qs {

namespace {

constexpr int kMaxThreads = 512;
constexpr int kChunk = 8;  // 16-byte accesses in flight per thread

// ---- load: pairs (pos, pos+1) are adjacent in memory (tile bit 0 = state bit 0).
// Tiles of >= 1024 amplitudes give every thread a multiple of kChunk pairs,
// so the batch of loads is issued without per-element guards.
// complex128: one 16-byte amplitude per lane and access, consecutive lanes on
// consecutive amplitudes (a pair per lane would be two 16-byte accesses at a
// 32-byte lane stride, each half-filling its requests)
template <bool kKeep>
__device__ __forceinline__ void tile_load_c128(const TileKArgs<double>& A, const Ctx& C, cplx<double>* T) {
  const uint32_t M = 1u << A.m, nthr = blockDim.x;
  const cplx<double>* __restrict__ psi = A.psi;
  constexpr int K = 2 * kChunk;
  for (uint32_t p0 = threadIdx.x; p0 < M; p0 += nthr * K) {
    cplx<double> v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t pos = p0 + nthr * k;
      if (pos < M) v[k] = ld_state<kKeep>(psi + (C.base | C.dep(pos)));
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t pos = p0 + nthr * k;
      if (pos < M) T[lds_off(pos)] = v[k];
    }
  }
}

template <class R, bool kKeep = false>
__device__ __forceinline__ void tile_load(const TileKArgs<R>& A, const Ctx& C, cplx<R>* T) {
  const uint32_t M = 1u << A.m, stride = 2 * blockDim.x;
  if (A.init_amp != 0.0) {
    // the uniform initial state, made here instead of read from HBM
    const cplx2<R> v{cplx<R>{(R)A.init_amp, R(0)}, cplx<R>{(R)A.init_amp, R(0)}};
    for (uint32_t pos = 2 * threadIdx.x; pos < M; pos += stride) *reinterpret_cast<cplx2<R>*>(T + lds_off(pos)) = v;
    return;
  }
  if constexpr (sizeof(R) == 8) {
    tile_load_c128<kKeep>(A, C, T);
    return;
  }
  const cplx<R>* __restrict__ psi = A.psi;
  if (M >= stride * kChunk) {
    for (uint32_t p0 = 2 * threadIdx.x; p0 < M; p0 += stride * kChunk) {
      cplx2<R> v[kChunk];
#pragma unroll
      for (int k = 0; k < kChunk; ++k)
        v[k] = ld_state<kKeep>(reinterpret_cast<const cplx2<R>*>(psi + (C.base | C.dep(p0 + stride * k))));
#pragma unroll
      for (int k = 0; k < kChunk; ++k) *reinterpret_cast<cplx2<R>*>(T + lds_off(p0 + stride * k)) = v[k];
    }
  } else {
    for (uint32_t pos = 2 * threadIdx.x; pos < M; pos += stride)
      *reinterpret_cast<cplx2<R>*>(T + lds_off(pos)) =
          ld_state<kKeep>(reinterpret_cast<const cplx2<R>*>(psi + (C.base | C.dep(pos))));
  }
}
// Stores the tile; returns this thread's FP64 sum of |psi|^2 over what it
// stored when the pass reports its norm (0 otherwise).
template <class R, bool kKeep = false>
__device__ __forceinline__ double tile_store(const TileKArgs<R>& A, const Ctx& C, const cplx<R>* T, uint32_t nthr) {
  // threads [0, nthr) store the tile
  const uint32_t M = 1u << A.m, stride = 2 * nthr;
  double nacc = 0.0;
  cplx<R>* __restrict__ psi = A.psi;
  // with the pass's butterfly normalisation
  const R sc = (R)A.scale;
  const bool do_scale = A.scale != 1.0;
  if constexpr (sizeof(R) == 8) {
    // complex128: one amplitude per lane and access (as in the load)
    constexpr int K = 2 * kChunk;
    for (uint32_t p0 = threadIdx.x; p0 < M; p0 += nthr * K) {
      cplx<R> v[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t pos = p0 + nthr * k;
        if (pos < M) v[k] = T[lds_off(pos)];
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t pos = p0 + nthr * k;
        if (pos < M) {
          if (do_scale) v[k] = cscale(v[k], sc);
          st_state<kKeep>(psi + (C.base | C.dep(pos)), v[k]);
          if (A.norm_part != nullptr) nacc += abs2_d(v[k]);
        }
      }
    }
    return nacc;
  }
  if (M >= stride * kChunk) {
    for (uint32_t p0 = 2 * threadIdx.x; p0 < M; p0 += stride * kChunk) {
      cplx2<R> v[kChunk];
#pragma unroll
      for (int k = 0; k < kChunk; ++k) v[k] = *reinterpret_cast<const cplx2<R>*>(T + lds_off(p0 + stride * k));
      if (do_scale) {
#pragma unroll
        for (int k = 0; k < kChunk; ++k) {
          v[k].a = cscale(v[k].a, sc);
          v[k].b = cscale(v[k].b, sc);
        }
      }
#pragma unroll
      for (int k = 0; k < kChunk; ++k)
        st_state<kKeep>(reinterpret_cast<cplx2<R>*>(psi + (C.base | C.dep(p0 + stride * k))), v[k]);
      if (A.norm_part != nullptr) {
#pragma unroll
        for (int k = 0; k < kChunk; ++k) nacc += abs2_d(v[k].a) + abs2_d(v[k].b);
      }
    }
  } else {
    for (uint32_t pos = 2 * threadIdx.x; pos < M; pos += stride) {
      cplx2<R> v = *reinterpret_cast<const cplx2<R>*>(T + lds_off(pos));
      if (do_scale) {
        v.a = cscale(v.a, sc);
        v.b = cscale(v.b, sc);
      }
      st_state<kKeep>(reinterpret_cast<cplx2<R>*>(psi + (C.base | C.dep(pos))), v);
      if (A.norm_part != nullptr) nacc += abs2_d(v.a) + abs2_d(v.b);
    }
  }
  return nacc;
}
// kKeep: cached accesses to the state.  A template parameter: a branch in one
// kernel cost the streaming passes 1 to 3% (a larger kernel, more scalar spills).
template <class R, bool kDiag, bool kKeep = false, int kQft = 2>
__device__ __forceinline__ void tile_body(const TileKArgs<R>& A, const uint32_t coset) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<R>* T = reinterpret_cast<cplx<R>*>(smem_raw);
  const Ctx C = coset_ctx(A, coset);
  tile_load<R, kKeep>(A, C, T);
  __syncthreads();
  tile_rounds<R, kDiag, false, kQft>(A, C, T, blockDim.x, threadIdx.x);
  const double nacc = tile_store<R, kKeep>(A, C, T, blockDim.x);
  if (A.norm_part != nullptr) {
    const double t = block_sum_fixed(nacc);
    if (threadIdx.x == 0) A.norm_part[coset] = t;
  }
}

template <class R, bool kDiag, int kQft>
__global__ void __launch_bounds__(kMaxThreads) tile_kernel(TileKArgs<R> A) {
  tile_body<R, kDiag, false, kQft>(A, A.order ? blockIdx.x : xcd_block(blockIdx.x, gridDim.x));
}

// complex64 passes: registers capped at 128 so that four waves fit per SIMD
// (two 512-thread workgroups of 2^13-amplitude tiles, or four of 2^12, share
// a CU's LDS).
template <bool kDiag, bool kKeep, int kQft>
__global__ void __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(4)))
tile_kernel_c64(TileKArgs<float> A) {
  tile_body<float, kDiag, kKeep, kQft>(A, A.order ? blockIdx.x : xcd_block(blockIdx.x, gridDim.x));
}

// ---- software-pipelined tile passes ------------------------------------------
// A tile that fills a CU's LDS (2^13 complex128 or 2^14 complex64 amplitudes)
// leaves one workgroup per CU, so a workgroup per coset would load, run its
// rounds and store strictly one after the other.  Instead one workgroup per
// CU walks the cosets w, w + G, w + 2G, ... (G workgroups) and issues the
// loads of its next coset into registers before it runs the current coset's
// rounds: HBM reads overlap the rounds and the stores.  A thread moves
// kPipeK 16-byte accesses per coset (an amplitude pair each for complex64,
// one amplitude for complex128); the first PipeAccess::pre of them are
// prefetched, the rest (complex128 only, whose rounds need the registers)
// are issued at the top of the coset's turn, ahead of the prefetched ones'
// LDS writes.
constexpr int kPipeK = 16;
template <class R>
struct PipeAccess;
template <>
struct PipeAccess<float> {
  using T = cplx2<float>;
  static constexpr uint32_t amps = 2;
  static constexpr int pre = 16;
};
template <>
struct PipeAccess<double> {
  using T = cplx<double>;
  static constexpr uint32_t amps = 1;
  static constexpr int pre = 8;
};

template <class R, int K0, int K1>
__device__ __forceinline__ void pipe_issue(const TileKArgs<R>& A, const Ctx& C, typename PipeAccess<R>::T* v) {
  using E = typename PipeAccess<R>::T;
  constexpr uint32_t apa = PipeAccess<R>::amps;
  const uint32_t step = apa * blockDim.x;
#pragma unroll
  for (int k = K0; k < K1; ++k) {
    const uint32_t pos = apa * threadIdx.x + step * k;
    v[k - K0] = ld_nt(reinterpret_cast<const E*>(A.psi + (C.base | C.dep(pos))));
  }
}
template <class R, int K0, int K1>
__device__ __forceinline__ void pipe_to_lds(const typename PipeAccess<R>::T* v, cplx<R>* T) {
  using E = typename PipeAccess<R>::T;
  constexpr uint32_t apa = PipeAccess<R>::amps;
  const uint32_t step = apa * blockDim.x;
#pragma unroll
  for (int k = K0; k < K1; ++k) {
    const uint32_t pos = apa * threadIdx.x + step * k;
    *reinterpret_cast<E*>(T + lds_off(pos)) = v[k - K0];
  }
}

// tile_store for a tile of exactly kN accesses per thread: with the number of
// stores known, the wait for the next coset's loads, issued before them, does not
// wait for them too (a loop of stores does: it counts as any number).
template <class R, int kN>
__device__ __forceinline__ double pipe_store(const TileKArgs<R>& A, const Ctx& C, const cplx<R>* T) {
  using E = typename PipeAccess<R>::T;
  constexpr uint32_t apa = PipeAccess<R>::amps;
  constexpr int kB = kN < kChunk * 2 / (int)apa ? kN : kChunk * 2 / (int)apa;
  const uint32_t step = apa * blockDim.x, p0 = apa * threadIdx.x;
  const R sc = (R)A.scale;
  const bool do_scale = A.scale != 1.0;
  double nacc = 0.0;
#pragma unroll
  for (int b = 0; b < kN; b += kB) {
    union {
      E e;
      cplx<R> c[apa];
    } v[kB];
#pragma unroll
    for (int k = 0; k < kB; ++k) v[k].e = *reinterpret_cast<const E*>(T + lds_off(p0 + step * (b + k)));
    if (do_scale) {
#pragma unroll
      for (int k = 0; k < kB; ++k)
#pragma unroll
        for (int i = 0; i < (int)apa; ++i) v[k].c[i] = cscale(v[k].c[i], sc);
    }
#pragma unroll
    for (int k = 0; k < kB; ++k) st_nt(reinterpret_cast<E*>(A.psi + (C.base | C.dep(p0 + step * (b + k)))), v[k].e);
    if (A.norm_part != nullptr) {
#pragma unroll
      for (int k = 0; k < kB; ++k)
#pragma unroll
        for (int i = 0; i < (int)apa; ++i) nacc += abs2_d(v[k].c[i]);
    }
  }
  return nacc;
}

// Requires 2^m = blockDim.x * kPipeK * PipeAccess<R>::amps (checked on the host).
template <class R, int kQft>
__global__ void __launch_bounds__(kMaxThreads) tile_kernel_pipe(TileKArgs<R> A, uint32_t n_cosets) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<R>* T = reinterpret_cast<cplx<R>*>(smem_raw);
  constexpr int P = PipeAccess<R>::pre;
  typename PipeAccess<R>::T v[P];
  const uint32_t G = gridDim.x;
  uint32_t c = A.order ? blockIdx.x : xcd_block(blockIdx.x, G);
  if (c < n_cosets) pipe_issue<R, 0, P>(A, coset_ctx(A, c), v);
  for (; c < n_cosets; c += G) {
    const Ctx C = coset_ctx(A, c);
    __syncthreads();  // the previous coset's store has finished reading the tile
    if constexpr (P < kPipeK) {
      typename PipeAccess<R>::T w[kPipeK - P];
      pipe_issue<R, P, kPipeK>(A, C, w);
      pipe_to_lds<R, 0, P>(v, T);
      pipe_to_lds<R, P, kPipeK>(w, T);
    } else {
      pipe_to_lds<R, 0, P>(v, T);
    }
    __syncthreads();
    if (c + G < n_cosets) pipe_issue<R, 0, P>(A, coset_ctx(A, c + G), v);
    tile_rounds<R, false, false, kQft>(A, C, T, blockDim.x, threadIdx.x);
    const double nacc = pipe_store<R, kPipeK>(A, C, T);
    if (A.norm_part != nullptr) {
      const double t = block_sum_fixed(nacc);
      if (threadIdx.x == 0) A.norm_part[c] = t;
    }
  }
}

// ---- warp-specialised persistent passes ---------------------------------------
// For complex128 tiles that fill a CU's LDS (2^13 amplitudes) and whose pass
// reports no norm: one persistent workgroup per CU of kWsConsumers threads
// that run the rounds and store each tile, and kWsProducers threads that
// hold the next coset's tile in registers (kWsK 16-byte loads each, issued
// as soon as the current tile is in LDS) and write it into LDS once the
// consumers have stored theirs.  HBM reads overlap the rounds and the
// stores; the LDS hand-over is the only serial step.  Producer and consumer
// code are separate loops (disjoint register live ranges) with the same
// sequence of workgroup barriers: per coset, one per round, one after the
// store and, when a next coset exists, one after its tile is written.
constexpr uint32_t kWsConsumers = 256, kWsProducers = 256;
constexpr int kWsK = 32;  // 16-byte accesses per producer thread and tile

template <class R>
__device__ __forceinline__ void ws_issue(const TileKArgs<R>& A, const Ctx& C, uint32_t pt,
                                         typename PipeAccess<R>::T* v) {
  using E = typename PipeAccess<R>::T;
  constexpr uint32_t apa = PipeAccess<R>::amps;
#pragma unroll
  for (int k = 0; k < kWsK; ++k) {
    const uint32_t pos = apa * (pt + kWsProducers * k);
    v[k] = ld_nt(reinterpret_cast<const E*>(A.psi + (C.base | C.dep(pos))));
  }
}
template <class R>
__device__ __forceinline__ void ws_to_lds(const typename PipeAccess<R>::T* v, uint32_t pt, cplx<R>* T) {
  using E = typename PipeAccess<R>::T;
  constexpr uint32_t apa = PipeAccess<R>::amps;
#pragma unroll
  for (int k = 0; k < kWsK; ++k) *reinterpret_cast<E*>(T + lds_off(apa * (pt + kWsProducers * k))) = v[k];
}

// Requires 2^m = kWsProducers * kWsK * PipeAccess<R>::amps and norm_part == null
// (checked on the host).
template <class R, int kQft>
__global__ void __launch_bounds__(kWsConsumers + kWsProducers) tile_kernel_ws(TileKArgs<R> A, uint32_t n_cosets) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<R>* T = reinterpret_cast<cplx<R>*>(smem_raw);
  const uint32_t G = gridDim.x;
  const uint32_t c0 = A.order ? blockIdx.x : xcd_block(blockIdx.x, G);
  if (c0 >= n_cosets) return;  // the whole workgroup leaves together
  const uint32_t R_ = A.n_rounds;
  if (threadIdx.x >= kWsConsumers) {
    const uint32_t pt = threadIdx.x - kWsConsumers;
    typename PipeAccess<R>::T v[kWsK];
    ws_issue<R>(A, coset_ctx(A, c0), pt, v);
    ws_to_lds<R>(v, pt, T);
    __syncthreads();  // first tile in LDS
    for (uint32_t c = c0; c < n_cosets; c += G) {
      const bool next = c + G < n_cosets;
      if (next) ws_issue<R>(A, coset_ctx(A, c + G), pt, v);
      for (uint32_t r = 0; r < R_; ++r) __syncthreads();  // the consumers' rounds
      __syncthreads();  // the consumers have stored the tile
      if (next) {
        ws_to_lds<R>(v, pt, T);
        __syncthreads();  // next tile in LDS
      }
    }
  } else {
    __syncthreads();  // first tile in LDS
    for (uint32_t c = c0; c < n_cosets; c += G) {
      const bool next = c + G < n_cosets;
      const Ctx C = coset_ctx(A, c);
      tile_rounds<R, false, false, kQft>(A, C, T, kWsConsumers, threadIdx.x);
      tile_store<R>(A, C, T, kWsConsumers);
      __syncthreads();  // tile read out of LDS
      if (next) __syncthreads();  // next tile in LDS
    }
  }
}

// ---- fused adjoint step ---------------------------------------------------------
// One workgroup per coset undoes the pass on both adjoint states: phi's and
// lambda's tiles are loaded into two LDS tiles, the pass's rounds run on each,
// the cross densities of the layer's parameter bits are summed from the two
// resulting tiles, and both tiles are stored back -- 4 S of HBM traffic per
// layer instead of 6 S for two passes and a separate re-read of both states.
template <class R, bool kDiag, int kQft>
__global__ void __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 2 : 1)))
tile_kernel_dual(TileKArgs<R> A, cplx<R>* lam, RhoTileArgs Q,
                                                                 double* __restrict__ partials) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[rho::kRhoMaxWaves][32];
  const uint32_t M = 1u << A.m;
  cplx<R>* T0 = reinterpret_cast<cplx<R>*>(smem_raw);
  cplx<R>* T1 = T0 + lds_off(M);
  const uint32_t ntiles = gridDim.x;
  const uint32_t coset = A.order ? blockIdx.x : xcd_block(blockIdx.x, ntiles);
  const Ctx C = coset_ctx(A, coset);
  TileKArgs<R> B = A;
  B.psi = lam;
  tile_load<R>(A, C, T0);
  tile_load<R>(B, C, T1);
  __syncthreads();
  tile_rounds<R, kDiag, false, kQft>(A, C, T0, blockDim.x, threadIdx.x);
  tile_rounds<R, kDiag, false, kQft>(A, C, T1, blockDim.x, threadIdx.x);
  if (Q.nbits) rho::accumulate_tile<R>(T0, T1, M, Q, red, partials, coset, ntiles);
  tile_store<R>(A, C, T0, blockDim.x);
  tile_store<R>(B, C, T1, blockDim.x);
}

// The same step with persistent workgroups (as many as fit on the device,
// each walking the cosets c, c + G, c + 2G, ...) that issue the loads of
// their next coset's two tiles into registers before the current coset's
// rounds, cross densities and stores: HBM reads overlap the work of the step,
// which a workgroup per coset (two or four resident per CU, each loading,
// computing and storing in turn) leaves exposed.  complex64 with
// 2^m = blockDim.x * kDualPipeK * 2 (eight 16-byte accesses per thread and
// tile; checked on the host).
constexpr int kDualPipeK = 8;
template <class R, bool kDiag, int kQft>
__global__ void __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(2)))
tile_kernel_dual_pipe(TileKArgs<R> A, cplx<R>* lam, RhoTileArgs Q, double* __restrict__ partials,
                      uint32_t n_cosets) {
  static_assert(sizeof(R) == 4, "complex64 tiles only");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[rho::kRhoMaxWaves][32];
  const uint32_t M = 1u << A.m;
  cplx<R>* T0 = reinterpret_cast<cplx<R>*>(smem_raw);
  cplx<R>* T1 = T0 + lds_off(M);
  TileKArgs<R> B = A;
  B.psi = lam;
  typename PipeAccess<R>::T v0[kDualPipeK], v1[kDualPipeK];
  const uint32_t G = gridDim.x;
  uint32_t c = A.order ? blockIdx.x : xcd_block(blockIdx.x, G);
  if (c < n_cosets) {
    const Ctx C = coset_ctx(A, c);
    pipe_issue<R, 0, kDualPipeK>(A, C, v0);
    pipe_issue<R, 0, kDualPipeK>(B, C, v1);
  }
  for (; c < n_cosets; c += G) {
    const Ctx C = coset_ctx(A, c);
    __syncthreads();  // the previous coset's stores have finished reading the tiles
    pipe_to_lds<R, 0, kDualPipeK>(v0, T0);
    pipe_to_lds<R, 0, kDualPipeK>(v1, T1);
    __syncthreads();
    if (c + G < n_cosets) {
      const Ctx Cn = coset_ctx(A, c + G);
      pipe_issue<R, 0, kDualPipeK>(A, Cn, v0);
      pipe_issue<R, 0, kDualPipeK>(B, Cn, v1);
    }
    if constexpr (kDiag) {
      tile_rounds<R, kDiag, false, kQft>(A, C, T0, blockDim.x, threadIdx.x);
      tile_rounds<R, kDiag, false, kQft>(A, C, T1, blockDim.x, threadIdx.x);
    } else {
      tile_rounds<R, false, true, kQft>(A, C, T0, blockDim.x, threadIdx.x, T1);
    }
    if (Q.nbits) rho::accumulate_tile<R>(T0, T1, M, Q, red, partials, c, n_cosets);
    pipe_store<R, kDualPipeK>(A, C, T0);
    pipe_store<R, kDualPipeK>(B, C, T1);
  }
}

// A batched instance's argument block, read field by field with scalar loads.
template <class R>
__device__ __forceinline__ TileKArgs<R> load_args(const TileKArgs<R>* descs, uint32_t i) {
  const cptr<TileKArgs<R>> P = to_const(descs) + i;
  TileKArgs<R> A;
  A.psi = P->psi;
  A.rounds = P->rounds;
  A.ops = P->ops;
  A.coef = P->coef;
  A.diag = P->diag;
  A.qtab = P->qtab;
  A.L = P->L;
  A.a = P->a;
  A.h = P->h;
  A.m = P->m;
  A.n_rounds = P->n_rounds;
  A.n = P->n;
  A.scale = P->scale;
  A.norm_part = nullptr;  // batched passes never report a norm
  A.init_amp = P->init_amp;
  A.order = 0;
  return A;
}

// Many instances of one tile geometry in one grid: virtual block v (the
// XCD-aware order of the workgroups) runs coset (v & (2^shift - 1)) of
// instance (v >> shift).
template <class R, bool kDiag, int kQft>
__global__ void __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 4 : 1)))
tile_kernel_batched(const TileKArgs<R>* __restrict__ descs,
                                                                    uint32_t shift) {
  const uint32_t v = xcd_block(blockIdx.x, gridDim.x);
  tile_body<R, kDiag, false, kQft>(load_args(descs, v >> shift), v & ((1u << shift) - 1u));
}

inline uint32_t tile_threads(uint32_t m) {
  uint32_t threads = (1u << m) >> RB;
  return threads < 64 ? 64 : (threads > (uint32_t)kMaxThreads ? (uint32_t)kMaxThreads : threads);
}

template <class R, bool kDiag>
inline uint32_t tile_threads_for(uint32_t m) {
  return tile_threads(m);
}

// Dynamic LDS limit of the tile kernels: the largest tile (2^14 complex64 or
// 2^13 complex128 amplitudes with padding, 139264 bytes) plus headroom, below
// the CU's 160 KB so that the kernels' small static LDS still fits.
constexpr int kTileDynLds = 144 * 1024;

inline size_t tile_lds(uint32_t m, size_t elem) {
  const uint32_t M = 1u << m;
  return elem * (M + ((M >> 5) << 1));
}

}  // namespace

template <class R, bool kDiag, int kQft>
void launch_tile_batched_k(const TileKArgs<R>* descs_dev, uint32_t count, uint32_t n, uint32_t m, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)tile_kernel_batched<R, kDiag, kQft>, kTileDynLds, "tile_pass_batched");
    attr_set = true;
  }
  const uint32_t shift = n - m;
  QS_LAUNCH("tile_pass_batched", s, (tile_kernel_batched<R, kDiag, kQft>), dim3(count << shift), dim3(tile_threads_for<R, kDiag>(m)),
            tile_lds(m, sizeof(cplx<R>)), s, descs_dev, shift);
}

template <class R>
void launch_tile_batched(const TileKArgs<R>* descs_dev, uint32_t count, uint32_t n, uint32_t m, bool has_diag,
                         bool has_qft, hipStream_t s) {
  if (has_diag)
    has_qft ? launch_tile_batched_k<R, true, 2>(descs_dev, count, n, m, s)
            : launch_tile_batched_k<R, true, 0>(descs_dev, count, n, m, s);
  else
    has_qft ? launch_tile_batched_k<R, false, 2>(descs_dev, count, n, m, s)
            : launch_tile_batched_k<R, false, 0>(descs_dev, count, n, m, s);
}

template <class R, bool kDiag, int kQft>
void launch_tile_k(const TileKArgs<R>& A, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)tile_kernel<R, kDiag, kQft>, kTileDynLds, "tile_pass");
    attr_set = true;
  }
  // one thread per register group of a round, between 64 and 512 threads
  const uint32_t n_cosets = 1u << (A.n - A.m);
  QS_LAUNCH("tile_pass", s, (tile_kernel<R, kDiag, kQft>), dim3(n_cosets), dim3(tile_threads_for<R, kDiag>(A.m)),
            tile_lds(A.m, sizeof(cplx<R>)), s, A);
}

template <bool kDiag, bool kKeep, int kQft>
void launch_tile_c64(const TileKArgs<float>& A, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)tile_kernel_c64<kDiag, kKeep, kQft>, kTileDynLds, "tile_pass");
    attr_set = true;
  }
  QS_LAUNCH("tile_pass", s, (tile_kernel_c64<kDiag, kKeep, kQft>), dim3(1u << (A.n - A.m)), dim3(tile_threads(A.m)),
            tile_lds(A.m, sizeof(cplx<float>)), s, A);
}

// What a pass has of QFT stages picks its kernel: without their code a kernel is
// half the size with fewer scalar spills (heisenberg chain on 23 qubits, complex64:
// 2306 -> 2256 us, TFIM on 25 7835 -> 7763), and a loop over ops next to the
// straight-line rounds costs those 0.5 to 1% (30-qubit QFT and Walsh passes), in
// place of the rounds of one stage up to 4% (23-qubit complex128 QFT).
template <class R, int kQft>
void launch_tile_q(const TileKArgs<R>& A, hipStream_t s) {
  A.diag != nullptr ? launch_tile_k<R, true, kQft>(A, s) : launch_tile_k<R, false, kQft>(A, s);
}
template <int kQft>
void launch_tile_c64_q(const TileKArgs<float>& A, hipStream_t s) {
  if (A.diag != nullptr)
    A.keep ? launch_tile_c64<true, true, kQft>(A, s) : launch_tile_c64<true, false, kQft>(A, s);
  else
    A.keep ? launch_tile_c64<false, true, kQft>(A, s) : launch_tile_c64<false, false, kQft>(A, s);
}

// Workgroups of a pipelined pass: one per compute unit (at most one coset each).
inline uint32_t pipe_grid(uint32_t n_cosets) {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
  }
  return n_cosets < (uint32_t)cus ? n_cosets : (uint32_t)cus;
}

template <class R>
bool pipe_eligible(const TileKArgs<R>& A) {
  // tiles that fill the LDS, without diagonal slots (whose rounds need the
  // registers the prefetch would take)
  return A.diag == nullptr && A.init_amp == 0.0 && A.m == (sizeof(R) == 8 ? 13u : 14u) &&
         (1u << A.m) == tile_threads(A.m) * kPipeK * PipeAccess<R>::amps;
}

// complex128 tiles that fill the LDS (measured: for complex64 the pipelined
// kernel is the faster one)
template <class R>
bool ws_eligible(const TileKArgs<R>& A) {
  return sizeof(R) == 8 && pipe_eligible(A) && A.norm_part == nullptr &&
         (1u << A.m) == kWsProducers * kWsK * PipeAccess<R>::amps;
}

template <class R, int kQft>
void launch_tile_ws(const TileKArgs<R>& A, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)tile_kernel_ws<R, kQft>, kTileDynLds, "tile_pass");
    attr_set = true;
  }
  const uint32_t n_cosets = 1u << (A.n - A.m);
  QS_LAUNCH("tile_pass", s, (tile_kernel_ws<R, kQft>), dim3(pipe_grid(n_cosets)), dim3(kWsConsumers + kWsProducers),
            tile_lds(A.m, sizeof(cplx<R>)), s, A, n_cosets);
}

template <class R, int kQft>
void launch_tile_pipe(const TileKArgs<R>& A, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)tile_kernel_pipe<R, kQft>, kTileDynLds, "tile_pass");
    attr_set = true;
  }
  const uint32_t n_cosets = 1u << (A.n - A.m);
  QS_LAUNCH("tile_pass", s, (tile_kernel_pipe<R, kQft>), dim3(pipe_grid(n_cosets)), dim3(tile_threads(A.m)),
            tile_lds(A.m, sizeof(cplx<R>)), s, A, n_cosets);
}

template <class R>
void launch_tile(const TileKArgs<R>& A, hipStream_t s) {
  if (ws_eligible(A)) {
    A.qft == 2 ? launch_tile_ws<R, 2>(A, s) : launch_tile_ws<R, 1>(A, s);
    return;
  }
  if (pipe_eligible(A)) {
    A.qft == 2 ? launch_tile_pipe<R, 2>(A, s) : launch_tile_pipe<R, 1>(A, s);
    return;
  }
  if constexpr (sizeof(R) == 4) {
    A.qft == 0 ? launch_tile_c64_q<0>(A, s) : (A.qft == 1 ? launch_tile_c64_q<1>(A, s) : launch_tile_c64_q<2>(A, s));
  } else {
    A.qft == 0 ? launch_tile_q<R, 0>(A, s) : (A.qft == 1 ? launch_tile_q<R, 1>(A, s) : launch_tile_q<R, 2>(A, s));
  }
}

template <class R, bool kDiag, int kQft>
void launch_tile_dual_k(const TileKArgs<R>& A, cplx<R>* lam, const RhoTileArgs& Q, double* partials, size_t lds,
                        hipStream_t s) {
  const uint32_t n_cosets = 1u << (A.n - A.m), threads = tile_threads_for<R, kDiag>(A.m);
  if constexpr (sizeof(R) == 4) {
    if ((1u << A.m) == threads * kDualPipeK * PipeAccess<R>::amps) {
      // persistent: the workgroups that fit on the device at once (a
      // property of the kernel, its block size and LDS, looked up once each)
      static bool attr_set = false;
      static int per_cu[16] = {0};
      if (!attr_set) {
        allow_dynamic_lds((const void*)tile_kernel_dual_pipe<R, kDiag, kQft>, kTileDynLds, "tile_pass_dual");
        attr_set = true;
      }
      int& nb = per_cu[A.m & 15];
      if (nb == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)tile_kernel_dual_pipe<R, kDiag, kQft>,
                                                          (int)threads, lds) != hipSuccess ||
            nb < 1)
          nb = 1;
      }
      const uint32_t grid = std::min<uint64_t>(n_cosets, (uint64_t)nb * pipe_grid(~0u));
      QS_LAUNCH("tile_pass_dual", s, (tile_kernel_dual_pipe<R, kDiag, kQft>), dim3(grid), dim3(threads), lds, s, A, lam, Q,
                partials, n_cosets);
      return;
    }
  }
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)tile_kernel_dual<R, kDiag, kQft>, kTileDynLds, "tile_pass_dual");
    attr_set = true;
  }
  QS_LAUNCH("tile_pass_dual", s, (tile_kernel_dual<R, kDiag, kQft>), dim3(n_cosets), dim3(threads), lds, s, A, lam, Q,
            partials);
}

template <class R>
bool launch_tile_dual(const TileKArgs<R>& A, cplx<R>* lam, const RhoTileArgs& Q, double* partials, double* out,
                      hipStream_t s) {
  const size_t lds = 2 * tile_lds(A.m, sizeof(cplx<R>));
  if (lds > (size_t)kTileDynLds || Q.nbits > 32 || A.init_amp != 0.0 || A.norm_part != nullptr) return false;
  for (uint32_t k = 0; k < Q.nbits; ++k)
    if (Q.tbit[k] >= A.m) return false;
  if (A.diag != nullptr)
    A.qft ? launch_tile_dual_k<R, true, 2>(A, lam, Q, partials, lds, s)
          : launch_tile_dual_k<R, true, 0>(A, lam, Q, partials, lds, s);
  else
    A.qft ? launch_tile_dual_k<R, false, 2>(A, lam, Q, partials, lds, s)
          : launch_tile_dual_k<R, false, 0>(A, lam, Q, partials, lds, s);
  if (Q.nbits) launch_rho_finalize(partials, 1u << (A.n - A.m), 8 * Q.nbits, out, s);
  return true;
}

template bool launch_tile_dual<float>(const TileKArgs<float>&, cplx<float>*, const RhoTileArgs&, double*, double*,
                                      hipStream_t);
template bool launch_tile_dual<double>(const TileKArgs<double>&, cplx<double>*, const RhoTileArgs&, double*, double*,
                                       hipStream_t);
template void launch_tile<float>(const TileKArgs<float>&, hipStream_t);
template void launch_tile<double>(const TileKArgs<double>&, hipStream_t);
template void launch_tile_batched<float>(const TileKArgs<float>*, uint32_t, uint32_t, uint32_t, bool, bool,
                                         hipStream_t);
template void launch_tile_batched<double>(const TileKArgs<double>*, uint32_t, uint32_t, uint32_t, bool, bool,
                                         hipStream_t);

}  // namespace qs
