// Sequences of layers on states of one tile (up to 2^13 amplitudes).
//
// A pass over a state that fits one workgroup's LDS is a few microseconds of
// work behind a launch, a load, a store and cold instruction caches, and the
// gathers between passes are launches that move a few kilobytes.  Here one
// workgroup loads the state, runs a whole range of tile passes and GF(2)
// permutations on it in LDS and stores it once; the adjoint's backward sweep
// does the same with phi and lambda side by side, each on half of the threads,
// and sums every layer's cross densities on the way.
//
// Bound by the latency of the rounds (one workgroup, one to four waves per
// SIMD): 10 qubits complex64 33% of the wavefront's cycles issue vector
// instructions and 44% wait, 12 qubits complex128 22 and 53%, its backward sweep 19
// and 50%.  12-qubit, 8-layer ansatz in complex128: energy and gradient 810 us in
// 53 launches -> 620 us in seven; 10-qubit TFIM, 20 Strang steps (five passes):
// 90 -> 74 us.
#include "kernels.h"
#include "rho.h"
#include "tile_rounds.h"

namespace qs {

namespace {

constexpr uint32_t kSeqMaxThreads = 512;
constexpr int kSeqDynLds = 144 * 1024;

// Positions of a tile that a thread holds at once in permutations.
constexpr int kHold = 16;

template <class R>
__device__ __forceinline__ TileKArgs<R> step_args(cptr<SeqStep<R>> S, uint32_t n) {
  TileKArgs<R> A{};
  A.rounds = S->rounds;
  A.ops = S->ops;
  A.coef = S->coef;
  A.diag = S->diag;
  A.qtab = S->qtab;
  A.L = A.a = A.m = A.n = n;
  A.n_rounds = S->n_rounds;
  A.scale = S->scale;
  return A;
}

// Brings the plan's tables (just uploaded, or last read by another XCD) into
// this XCD's L2 while the state is loaded: the rounds read their coefficients by
// dependent scalar loads, each of which would otherwise wait for memory.
__device__ __forceinline__ void warm_tables(const void* tables, uint32_t bytes) {
  const uint4* p = reinterpret_cast<const uint4*>(tables);
  for (uint32_t i = threadIdx.x * 8u; i < bytes / 16u; i += blockDim.x * 8u) {  // one access per 128-byte line
    uint4 v = p[i];
    asm volatile("" ::"v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w));
  }
}

template <class R>
__device__ __forceinline__ void seq_load(const cplx<R>* psi, cplx<R>* T, uint32_t M, uint32_t tid, uint32_t nthr) {
  for (uint32_t p = 2u * tid; p < M; p += 2u * nthr)
    *reinterpret_cast<cplx2<R>*>(T + lds_off(p)) = *reinterpret_cast<const cplx2<R>*>(psi + p);
}

// T[y] <- T[A y ^ c'] over the whole tile; every thread of the workgroup takes
// part in the barriers.  A thread's M / nthr <= kHold2 positions go through
// registers.
template <class R, int kHold2>
__device__ __forceinline__ void seq_permute(cptr<SeqStep<R>> S, cplx<R>* T, uint32_t M, uint32_t n, uint32_t tid,
                                            uint32_t nthr) {
  // A is linear: the source of y = tid + nthr k splits into a part of the
  // thread and a uniform one
  uint32_t x0 = S->cprime;
  for (uint32_t j = 0; j < n; ++j)
    if ((tid >> j) & 1u) x0 ^= S->acol[j];
  const uint32_t lt = 31u - (uint32_t)__builtin_clz(nthr);
  cplx<R> v[kHold2];
#pragma unroll
  for (int k = 0; k < kHold2; ++k) {
    uint32_t xk = 0;
    for (uint32_t j = 0; j < 5; ++j)
      if (((uint32_t)k >> j) & 1u && lt + j < n) xk ^= S->acol[lt + j];
    if (tid + nthr * k < M) v[k] = T[lds_off(x0 ^ xk)];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kHold2; ++k)
    if (tid + nthr * k < M) T[lds_off(tid + nthr * k)] = v[k];
  __syncthreads();
}

template <class R>
__device__ __forceinline__ void seq_scale(cplx<R>* T, uint32_t M, R sc, uint32_t tid, uint32_t nthr) {
  for (uint32_t p = 2u * tid; p < M; p += 2u * nthr) {
    cplx2<R>* q = reinterpret_cast<cplx2<R>*>(T + lds_off(p));
    cplx2<R> v = *q;
    v.a = cscale(v.a, sc);
    v.b = cscale(v.b, sc);
    *q = v;
  }
}

template <class R>
__global__ void __launch_bounds__(kSeqMaxThreads) seq_kernel(cplx<R>* __restrict__ psi, uint32_t n,
                                                             const SeqStep<R>* steps, uint32_t count,
                                                             const void* tables, uint32_t table_bytes) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<R>* T = reinterpret_cast<cplx<R>*>(smem_raw);
  const uint32_t M = 1u << n, nthr = blockDim.x, tid = threadIdx.x;
  const Ctx C{0, n, n};
  warm_tables(tables, table_bytes);
  seq_load<R>(psi, T, M, tid, nthr);
  __syncthreads();
  for (uint32_t i = 0; i < count; ++i) {
    const cptr<SeqStep<R>> S = to_const(steps) + i;
    if (S->n_rounds == 0) {
      seq_permute<R, kHold>(S, T, M, n, tid, nthr);
      continue;
    }
    const TileKArgs<R> A = step_args<R>(S, n);
    tile_rounds<R, true>(A, C, T, nthr, tid);
    if (A.scale != 1.0) {
      seq_scale<R>(T, M, (R)A.scale, tid, nthr);
      __syncthreads();
    }
  }
  for (uint32_t p = 2u * tid; p < M; p += 2u * nthr)
    *reinterpret_cast<cplx2<R>*>(psi + p) = *reinterpret_cast<const cplx2<R>*>(T + lds_off(p));
}

// The adjoint's backward sweep: the steps (of the inverse plan) on phi by the
// lower half of the threads and on lambda by the upper half, the cross
// densities of step i's requested bits (bits[i], ascending) to out + slot[i]
// before the step's scale is applied.  phi and lambda are only read.
template <class R>
__global__ void __launch_bounds__(kSeqMaxThreads) seq_dual_kernel(const cplx<R>* __restrict__ phi,
                                                                  const cplx<R>* __restrict__ lam, uint32_t n,
                                                                  const SeqStep<R>* steps, SeqGrads G,
                                                                  const void* tables, uint32_t table_bytes,
                                                                  double* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[rho::kRhoMaxWaves][32];
  const uint32_t M = 1u << n, nthr = blockDim.x >> 1;
  const bool upper = threadIdx.x >= nthr;
  const uint32_t tid = upper ? threadIdx.x - nthr : threadIdx.x;
  cplx<R>* T0 = reinterpret_cast<cplx<R>*>(smem_raw);
  cplx<R>* T1 = T0 + lds_off(M);
  cplx<R>* T = upper ? T1 : T0;
  const Ctx C{0, n, n};
  warm_tables(tables, table_bytes);
  seq_load<R>(upper ? lam : phi, T, M, tid, nthr);
  __syncthreads();
  for (uint32_t i = 0; i < G.count; ++i) {
    const cptr<SeqStep<R>> S = to_const(steps) + i;
    if (S->n_rounds == 0) {
      seq_permute<R, 2 * kHold>(S, T, M, n, tid, nthr);
      continue;
    }
    const TileKArgs<R> A = step_args<R>(S, n);
    tile_rounds<R, true>(A, C, T, nthr, tid);
    const uint32_t bits = G.bits[i];
    if (bits) {
      auto tbit = [&](uint32_t k) {
        uint32_t b = bits;
        for (; k; --k) b &= b - 1u;
        return (uint32_t)__builtin_ctz(b);
      };
      rho::accumulate_bits<R>(T0, T1, M, (uint32_t)__builtin_popcount(bits), tbit, red, out + G.slot[i], 0, 1);
    }
    if (A.scale != 1.0 && i + 1 < G.count) {
      seq_scale<R>(T, M, (R)A.scale, tid, nthr);
      __syncthreads();
    }
  }
}

// (a plan's tables are a few KiB per pass; no more than a quarter of an XCD's L2)
inline uint32_t warm_bytes(size_t bytes) { return (uint32_t)(bytes < (1u << 20) ? bytes : (1u << 20)); }

inline size_t seq_tile_bytes(uint32_t n, size_t amp) {
  const uint32_t M = 1u << n;
  return amp * (M + ((M >> 5) << 1));
}

}  // namespace

bool seq_fits(int n, size_t amp_bytes, bool dual) {
  return n >= kRoundBits && n <= kSeqMaxBits && (dual ? 2 : 1) * seq_tile_bytes((uint32_t)n, amp_bytes) <= (size_t)kSeqDynLds;
}

template <class R>
void launch_seq(cplx<R>* psi, int n, const SeqStep<R>* steps, uint32_t count, const void* tables, size_t table_bytes,
                hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)seq_kernel<R>, kSeqDynLds, "seq_passes");
    attr_set = true;
  }
  const uint32_t g = (1u << n) >> kRoundBits, threads = g < 64 ? 64 : (g > kSeqMaxThreads ? kSeqMaxThreads : g);
  QS_LAUNCH("seq_passes", s, seq_kernel<R>, dim3(1), dim3(threads), seq_tile_bytes(n, sizeof(cplx<R>)), s, psi,
            (uint32_t)n, steps, count, tables, warm_bytes(table_bytes));
}

template <class R>
void launch_seq_dual(const cplx<R>* phi, const cplx<R>* lam, int n, const SeqStep<R>* steps, const SeqGrads& G,
                     const void* tables, size_t table_bytes, double* out, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)seq_dual_kernel<R>, kSeqDynLds, "seq_adjoint");
    attr_set = true;
  }
  const uint32_t g = (1u << n) >> kRoundBits;
  const uint32_t half = g < 64 ? 64 : (g > kSeqMaxThreads / 2 ? kSeqMaxThreads / 2 : g);
  QS_LAUNCH("seq_adjoint", s, seq_dual_kernel<R>, dim3(1), dim3(2 * half), 2 * seq_tile_bytes(n, sizeof(cplx<R>)), s,
            phi, lam, (uint32_t)n, steps, G, tables, warm_bytes(table_bytes), out);
}

template void launch_seq<float>(cplx<float>*, int, const SeqStep<float>*, uint32_t, const void*, size_t, hipStream_t);
template void launch_seq<double>(cplx<double>*, int, const SeqStep<double>*, uint32_t, const void*, size_t,
                                 hipStream_t);
template void launch_seq_dual<float>(const cplx<float>*, const cplx<float>*, int, const SeqStep<float>*,
                                     const SeqGrads&, const void*, size_t, double*, hipStream_t);
template void launch_seq_dual<double>(const cplx<double>*, const cplx<double>*, int, const SeqStep<double>*,
                                      const SeqGrads&, const void*, size_t, double*, hipStream_t);

}  // namespace qs
