// Pauli-sum expectations, many terms per read of the state.
//
// A term with X mask x and Z mask z needs sum_i s(i) q(i) with
// q(i) = conj(psi_i) psi_{i ^ x} (its real part when the term has an even
// number of Y factors, its imaginary part otherwise) over one index of every
// pair {i, i ^ x}, and s(i) = (-1)^popcount(i & z).  One reduction per X mask
// reads the state once per mask and pays a compensated add per term and
// amplitude; here a workgroup stages a tile of the state in LDS and takes
// windows of four tile bits: a thread forms the eight products of an X mask
// inside a window once, in FP64 registers, and contracts them with the signs
// of each of the mask's terms (s is a character of the index bits: one
// multiply-add per product folds one bit at a time, 7 per term; 15 for a Z-type
// term on the 16 probabilities).  Z factors outside the window are one parity
// per thread.
//
// Sums: the products in a thread, the lanes of a wavefront (fixed order, four
// terms at a time by register exchanges), the wavefronts in order, then
// compensated over the workgroup's tiles and over the workgroups; all in FP64.
//
// Bound by vector instructions (per 16 amplitudes about 80 per X mask, of which
// 32 are conversions to FP64, and 20 per term; 67% of the SIMDs' cycles at 26
// qubits) and nearly as many scalar ones, beside one read of the state per tile
// set.  26-qubit XXZ chain in complex64 (75 terms, 26 X masks, four
// sets): 29 reductions and host round trips 3.83 ms -> 1.00 ms; 10 qubits, 19
// terms: 12 reductions, 0.31 ms of wall time -> 0.03 ms.  The products from
// registers holding a whole window took 200 registers and 2.3 ms; 2^13 tiles
// (three sets) 0.96 ms at 26 qubits, slower from 25 down.
#include "acc.h"
#include "kernels.h"
#include "lanes.h"

namespace qs {

namespace {

constexpr uint32_t kWin = 4, kWinN = 1u << kWin;
constexpr int kThreads = 256;

__device__ __forceinline__ uint32_t lds_off(uint32_t pos) { return pos + ((pos >> 5) << 1); }

// sum_p (-1)^popcount(p & z) q[p] over 2^kBits products, one bit at a time.
template <int kBits>
__device__ __forceinline__ double contract(const double (&q)[1 << kBits], uint32_t z) {
  double u[1 << (kBits - 1)];
  double s = (z & 1u) ? -1.0 : 1.0;
#pragma unroll
  for (int p = 0; p < (1 << (kBits - 1)); ++p) u[p] = fma(s, q[2 * p + 1], q[2 * p]);
#pragma unroll
  for (int b = 1; b < kBits; ++b) {
    s = ((z >> b) & 1u) ? -1.0 : 1.0;
#pragma unroll
    for (int p = 0; p < (1 << (kBits - 1 - b)); ++p) u[p] = fma(s, u[2 * p + 1], u[2 * p]);
  }
  return u[0];
}

// Sums four values over the wavefront's lanes at once (register exchanges, no
// LDS); value r of the first cnt goes to red[(t0 + r) waves + wave].
__device__ __forceinline__ void flush4(const double (&v)[4], uint32_t cnt, uint32_t lane, double* red, uint32_t t0,
                                       uint32_t waves, uint32_t wave) {
  const double t = wave_sum4(v);
  const uint32_t r = wave_sum4_value(lane);
  if ((lane & 15u) == 0 && r < cnt) red[(t0 + r) * waves + wave] = t;
}

template <class R, bool kKeep>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
expect_tiles_kernel(ExpectArgs<R> A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const uint32_t M = 1u << A.m, waves = blockDim.x >> 6;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  cplx<R>* T = reinterpret_cast<cplx<R>*>(smem_raw);
  double* red = reinterpret_cast<double*>(T + lds_off(M));
  Acc* acc = reinterpret_cast<Acc*>(red + A.n_terms * waves);
  uint32_t* hi_tab = reinterpret_cast<uint32_t*>(acc + A.n_terms);
  for (uint32_t h = threadIdx.x; h < (1u << (A.m - A.L)); h += blockDim.x) {
    uint32_t off = 0;
    for (uint32_t j = 0; j < A.m - A.L; ++j)
      if ((h >> j) & 1u) off |= 1u << A.hi_bit[j];
    hi_tab[h] = off;
  }
  for (uint32_t t = threadIdx.x; t < A.n_terms; t += blockDim.x) acc[t] = {0.0, 0.0};
  for (uint32_t t = threadIdx.x; t < A.n_terms * waves; t += blockDim.x) red[t] = 0.0;
  const uint32_t Lmask = (1u << A.L) - 1u;
  const bool full = M == kWinN * blockDim.x, active = threadIdx.x < (M >> kWin);
  __syncthreads();
  const uint32_t my_pos = full ? 2u * threadIdx.x : 0u, my_lds = lds_off(my_pos);
  const size_t my_off = (my_pos & Lmask) | hi_tab[my_pos >> A.L];
  const uint32_t split = blockIdx.x % A.wsplit, b0 = blockIdx.x / A.wsplit, nb = gridDim.x / A.wsplit;
  for (uint32_t c = b0; c < A.n_tiles; c += nb) {
    uint32_t base = 0;
    for (uint32_t j = 0; j < A.n_free; ++j) base |= ((c >> j) & 1u) << A.free_bit[j];
    __syncthreads();  // the previous tile has been read, its sums taken
    if (full) {
      // eight pairs per thread in flight at once; the pairs of one thread are
      // a multiple of 2^5 positions apart, so both offsets split into a part
      // of the thread and a part of the access
      cplx2<R> v[8];
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k)
        v[k] = ld_state<kKeep>(reinterpret_cast<const cplx2<R>*>(A.psi + (base | A.load_off[k]) + my_off));
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k)
        *reinterpret_cast<cplx2<R>*>(T + my_lds + lds_off(2u * blockDim.x * k)) = v[k];
    } else {
      for (uint32_t p = 2u * threadIdx.x; p < M; p += 2u * blockDim.x)
        *reinterpret_cast<cplx2<R>*>(T + lds_off(p)) =
            *reinterpret_cast<const cplx2<R>*>(A.psi + (base | (p & Lmask) | hi_tab[p >> A.L]));
    }
    __syncthreads();
    for (uint32_t w = split; w < A.n_win; w += A.wsplit) {
      const uint32_t tbits = A.win[w].bits, g0 = A.win[w].g0, g1 = A.win[w].g1;
      uint32_t g = active ? threadIdx.x : 0u;
      uint32_t off[kWin];
#pragma unroll
      for (uint32_t k = 0; k < kWin; ++k) {
        const uint32_t tb = (tbits >> (8 * k)) & 0xffu;
        g = insert0(g, tb);
        off[k] = lds_off(1u << tb);
      }
      const cplx<R>* Tg = T + lds_off(g);
      const uint32_t gi = base | (g & Lmask) | hi_tab[g >> A.L];  // window bits clear
      // terms four at a time through v; a term's masks are read one term ahead
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      uint32_t t = A.grp[g0].t0;
      uint32_t z = A.term[t].z, zw = A.term[t].zw;
      auto emit = [&](double part) {  // term t's value from its signed sum
        const double val =
            __hiloint2double(__double2hiint(part) ^ (int)((uint32_t)popc(gi & z) << 31), __double2loint(part));
        switch (t & 3u) {
          case 0: v[0] = val; break;
          case 1: v[1] = val; break;
          case 2: v[2] = val; break;
          default:
            v[3] = val;
            flush4(v, 4, lane, red, t - 3u, waves, wave);
            break;
        }
      };
      for (uint32_t e = g0; e < g1; ++e) {
        const uint32_t x = A.grp[e].x, t1 = A.grp[e].t1;
        uint32_t have = ~0u;  // signs of part: a group's terms come in order of zw
        double part = 0.0;
        if (x == 0) {
          double q[kWinN];
#pragma unroll
          for (uint32_t j = 0; j < kWinN; ++j) {
            const cplx<R> a = Tg[((j & 1) ? off[0] : 0u) + ((j & 2) ? off[1] : 0u) + ((j & 4) ? off[2] : 0u) +
                                 ((j & 8) ? off[3] : 0u)];
            q[j] = abs2_d(a);
          }
          if (!full && !active) {
#pragma unroll
            for (uint32_t j = 0; j < kWinN; ++j) q[j] = 0.0;
          }
          for (; t < t1; ++t) {
            const uint32_t zn = A.term[t + 1].z, zwn = A.term[t + 1].zw;
            if (zw != have) part = contract<4>(q, have = zw);
            emit(part);
            z = zn;
            zw = zwn;
          }
        } else {
          // the pairs {i, i ^ x}: i over the window bits other than x's highest
          // (offset o[k] each), its partner at the offsets' complement on x
          const uint32_t H = 31u - (uint32_t)__builtin_clz(x);
          uint32_t o[3];
          int d[3], oj = (int)off[0];
          oj = (int)(H == 1 ? off[1] : H == 2 ? off[2] : H == 3 ? off[3] : off[0]);
#pragma unroll
          for (uint32_t k = 0; k < 3; ++k) {
            const uint32_t b = k < H ? k : k + 1;
            o[k] = k < H ? off[k] : off[k + 1];
            const bool in = (x >> b) & 1u;
            d[k] = in ? -(int)o[k] : (int)o[k];
            oj += in ? (int)o[k] : 0;
          }
          const bool imag = A.grp[e].imag != 0;
          cplx<R> ai[8], aj[8];
#pragma unroll
          for (int p = 0; p < 8; ++p) {
            ai[p] = Tg[((p & 1) ? o[0] : 0u) + ((p & 2) ? o[1] : 0u) + ((p & 4) ? o[2] : 0u)];
            aj[p] = Tg[oj + ((p & 1) ? d[0] : 0) + ((p & 2) ? d[1] : 0) + ((p & 4) ? d[2] : 0)];
          }
          double q[8];
          if (imag) {
#pragma unroll
            for (int p = 0; p < 8; ++p)
              q[p] = fma((double)ai[p].re, (double)aj[p].im, -(double)ai[p].im * (double)aj[p].re);
          } else {
#pragma unroll
            for (int p = 0; p < 8; ++p)
              q[p] = fma((double)ai[p].re, (double)aj[p].re, (double)ai[p].im * (double)aj[p].im);
          }
          if (!full && !active) {
#pragma unroll
            for (int p = 0; p < 8; ++p) q[p] = 0.0;
          }
          for (; t < t1; ++t) {
            const uint32_t zn = A.term[t + 1].z, zwn = A.term[t + 1].zw;
            if (zw != have) part = contract<3>(q, have = zw);
            emit(part);
            z = zn;
            zw = zwn;
          }
        }
      }
      if (t & 3u) flush4(v, t & 3u, lane, red, t & ~3u, waves, wave);
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < A.n_terms; t += blockDim.x) {
      double v = 0.0;
      for (uint32_t k = 0; k < waves; ++k) v += red[t * waves + k];
      Acc a = acc[t];
      nadd(a, v);
      acc[t] = a;
    }
  }
  for (uint32_t t = threadIdx.x; t < A.n_terms; t += blockDim.x) {
    const Acc a = acc[t];
    A.partials[((size_t)blockIdx.x * A.n_terms + t) * 2] = a.s;
    A.partials[((size_t)blockIdx.x * A.n_terms + t) * 2 + 1] = a.c;
  }
}

// One wavefront per term of every set folds its workgroups' sums, compensated
// and in a fixed order.
__global__ void __launch_bounds__(64) expect_fold_kernel(ExpectFold F, double* __restrict__ out) {
  uint32_t t = blockIdx.x, s = 0;
  while (s + 1 < F.n_sets && t >= F.n_terms[s]) t -= F.n_terms[s++];
  const double* P = F.partials + F.off[s];
  Acc a = {0.0, 0.0};
  for (uint32_t b = threadIdx.x; b < F.n_blocks[s]; b += 64) {
    const size_t e = ((size_t)b * F.n_terms[s] + t) * 2;
    a = ncombine(a, Acc{P[e], P[e + 1]});
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    const Acc o{__shfl_xor(a.s, d, 64), __shfl_xor(a.c, d, 64)};
    a = ncombine(a, o);
  }
  if (threadIdx.x == 0) out[blockIdx.x] = a.s + a.c;
}

inline uint32_t expect_threads(uint32_t m) {
  const uint32_t t = (1u << m) >> kWin;
  return t < 64 ? 64 : t;
}

}  // namespace

template <class R, bool kKeep>
void launch_expect_tiles_k(const ExpectArgs<R>& A, uint32_t blocks, hipStream_t s) {
  constexpr int kMaxLds = 96 * 1024;
  static bool attr_set = false;
  if (!attr_set) {
    allow_dynamic_lds((const void*)expect_tiles_kernel<R, kKeep>, kMaxLds, "expect_tiles");
    attr_set = true;
  }
  const uint32_t M = 1u << A.m, threads = expect_threads(A.m), waves = threads / 64;
  const size_t lds = sizeof(cplx<R>) * (M + ((M >> 5) << 1)) + sizeof(double) * A.n_terms * waves + sizeof(Acc) * A.n_terms +
                     sizeof(uint32_t) * ((size_t)1 << (A.m - A.L));
  QS_LAUNCH("expect_tiles", s, (expect_tiles_kernel<R, kKeep>), dim3(blocks), dim3(threads), lds, s, A);
}
template <class R>
void launch_expect_tiles(const ExpectArgs<R>& A, uint32_t blocks, hipStream_t s) {
  // three terms on 25 complex64 qubits 75 us, streaming 83; XXZ on 24 complex128
  // qubits 394 and 432
  if (keep_resident((uint64_t)sizeof(cplx<R>) << (A.m + A.n_free), 0, 0))
    launch_expect_tiles_k<R, true>(A, blocks, s);
  else
    launch_expect_tiles_k<R, false>(A, blocks, s);
}

void launch_expect_fold(const ExpectFold& F, double* out, hipStream_t s) {
  uint32_t n = 0;
  for (uint32_t k = 0; k < F.n_sets; ++k) n += F.n_terms[k];
  QS_LAUNCH("expect_fold", s, expect_fold_kernel, dim3(n), dim3(64), 0, s, F, out);
}

template void launch_expect_tiles<float>(const ExpectArgs<float>&, uint32_t, hipStream_t);
template void launch_expect_tiles<double>(const ExpectArgs<double>&, uint32_t, hipStream_t);

}  // namespace qs
