// Read-out from the device state: shot sampling of the basis-state
// distribution p_i = |psi_i|^2 / ||psi||^2 and marginal distributions over a
// subset of qubits (the paper's measurement and sampling workloads, Sections
// "State Management" and "Algorithm Implementations").
//
// Sampling, for caller-provided uniform numbers u in [0, 1): the drawn index
// is the first i whose cumulative probability mass exceeds u ||psi||^2.  The
// cumulative sums are hierarchical and FP64 with a fixed order everywhere:
// 64-amplitude sub-block sums (one wavefront each), block sums over 2^14
// amplitudes, an exclusive scan of the block sums by one workgroup; then one
// wavefront per sample searches the block prefixes, scans the block's
// sub-block sums and finally the sub-block's 64 probabilities.
#include "kernels.h"
#include "lanes.h"

#include <mutex>
#include <string>

#include "planner.h"

namespace qs {

void check_hip(hipError_t e, const char* what);

namespace {

constexpr int kSampThreads = 256;
constexpr int kScanThreads = 1024;

template <class R>
__device__ __forceinline__ double prob(const cplx<R>& a) {
  const double x = (double)a.re, y = (double)a.im;
  return x * x + y * y;
}

// Fixed-order inclusive scan across a wavefront.
__device__ __forceinline__ double wave_scan(double x, uint32_t lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double y = __shfl_up(x, d, 64);
    if (lane >= (uint32_t)d) x += y;
  }
  return x;
}
// One workgroup per block: sub[s] = the probability of sub-block s (sub_len <=
// 64 amplitudes, one per lane), blk[b] = the sum of the block's sub-block sums
// in order.  A wavefront takes eight sub-blocks at a time, their loads in
// flight together and their sums taken four at a time.
// Bound by the read of the state: 26 qubits complex64, sums of sub-blocks one
// by one through LDS and a second kernel over them 200 us, this one 120 us.
template <class R>
__global__ void __launch_bounds__(kSampThreads) block_masses_kernel(const cplx<R>* __restrict__ psi, uint64_t n_blk,
                                                                    uint32_t subs_per_block, uint32_t sub_len,
                                                                    double* __restrict__ sub, double* __restrict__ blk) {
  __shared__ double s_sub[256];
  constexpr uint32_t kWaves = kSampThreads / 64, kU = 8;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  for (uint64_t b = blockIdx.x; b < n_blk; b += gridDim.x) {
    const uint64_t s0 = b * subs_per_block;
    for (uint32_t j = wave * kU; j < subs_per_block; j += kWaves * kU) {
      cplx<R> a[kU];
#pragma unroll
      for (uint32_t k = 0; k < kU; ++k) {
        a[k] = cplx<R>{R(0), R(0)};
        if (j + k < subs_per_block && lane < sub_len) a[k] = ld_nt(psi + (s0 + j + k) * sub_len + lane);
      }
#pragma unroll
      for (uint32_t h = 0; h < kU; h += 4) {
        const double p[4] = {prob(a[h]), prob(a[h + 1]), prob(a[h + 2]), prob(a[h + 3])};
        const double t = wave_sum4(p);
        const uint32_t o = j + h + wave_sum4_value(lane);
        if ((lane & 15u) == 0 && o < subs_per_block) s_sub[o] = t;
      }
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < subs_per_block; j += kSampThreads) sub[s0 + j] = s_sub[j];
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (uint32_t j0 = 0; j0 < subs_per_block; j0 += 16) {
        double v[16];
#pragma unroll
        for (uint32_t k = 0; k < 16; ++k) v[k] = j0 + k < subs_per_block ? s_sub[j0 + k] : 0.0;
#pragma unroll
        for (uint32_t k = 0; k < 16; ++k) t += v[k];
      }
      blk[b] = t;
    }
    __syncthreads();
  }
}

// P[0..n] = exclusive prefix of blk[0..n) (P[n] = total); one workgroup.
__global__ void __launch_bounds__(kScanThreads) block_scan_kernel(const double* __restrict__ blk, uint64_t n,
                                                                  double* __restrict__ P) {
  __shared__ double tot[kScanThreads];
  const uint64_t chunk = (n + kScanThreads - 1) / kScanThreads;
  const uint64_t b0 = threadIdx.x * chunk, b1 = b0 + chunk < n ? b0 + chunk : n;
  double t = 0.0;
  for (uint64_t b = b0; b < b1; b += 8) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = b + k < b1 ? blk[b + k] : 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) t += v[k];
  }
  tot[threadIdx.x] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    // one chain of additions, its operands read 16 ahead
    double run = 0.0;
    for (int k0 = 0; k0 < kScanThreads; k0 += 16) {
      double v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = tot[k0 + k];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double x = v[k];
        v[k] = run;
        run += x;
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) tot[k0 + k] = v[k];
    }
    P[n] = run;
  }
  __syncthreads();
  double run = tot[threadIdx.x];
  for (uint64_t b = b0; b < b1; b += 8) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = b + k < b1 ? blk[b + k] : 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (b + k < b1) P[b + k] = run;
      run += v[k];
    }
  }
}

// One wavefront per sample.
template <class R>
__global__ void __launch_bounds__(kSampThreads) sample_kernel(const cplx<R>* __restrict__ psi,
                                                              const double* __restrict__ sub,
                                                              const double* __restrict__ P, uint64_t n_blk,
                                                              uint32_t subs_per_block, uint32_t sub_len,
                                                              const double* __restrict__ u, uint64_t count,
                                                              uint64_t* __restrict__ out) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t k = blockIdx.x * (uint64_t)(kSampThreads / 64) + (threadIdx.x >> 6);
  if (k >= count) return;
  const double total = P[n_blk];
  double t = u[k] * total;
  // block: last b with P[b] <= t (P is non-decreasing, P[0] = 0); requiring
  // P[b] < total as well keeps a product u total that rounded up to total in
  // the last block with mass
  uint64_t lo = 0, hi = n_blk - 1;
  while (lo < hi) {
    const uint64_t mid = (lo + hi + 1) / 2;
    if (P[mid] <= t && P[mid] < total) lo = mid;
    else hi = mid - 1;
  }
  const uint64_t b = lo;
  t -= P[b];
  // sub-block: subs_per_block <= 256 sums, 4 per lane, scanned in order
  double s4[4], run = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t idx = lane * 4 + j;
    s4[j] = idx < subs_per_block ? sub[b * subs_per_block + idx] : 0.0;
    run += s4[j];
  }
  const double incl = wave_scan(run, lane);
  double excl = incl - run;
  // the first sub-block whose inclusive sum exceeds t; if rounding leaves t at
  // or past the block's total, the last sub-block with mass
  int pick = -1, last = -1;
  double before = 0.0, before_last = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int idx = (int)(lane * 4 + j);
    if (s4[j] > 0.0) {
      if (pick < 0 && excl + s4[j] > t) {
        pick = idx;
        before = excl;
      }
      last = idx;
      before_last = excl;
    }
    excl += s4[j];
  }
  // the smallest lane holding a pick wins; else the largest lane holding mass
  const uint64_t hit = __ballot(pick >= 0);
  uint32_t sb;
  double sbefore;
  if (hit) {
    const int src = __builtin_ctzll(hit);
    sb = (uint32_t)__shfl(pick, src, 64);
    sbefore = __shfl(before, src, 64);
  } else {
    const uint64_t has = __ballot(last >= 0);
    const int src = has ? 63 - __builtin_clzll(has) : 0;
    sb = has ? (uint32_t)__shfl(last, src, 64) : 0u;
    sbefore = has ? __shfl(before_last, src, 64) : 0.0;
  }
  t -= sbefore;
  // amplitude within the sub-block
  const uint64_t base = (b * subs_per_block + sb) * sub_len;
  const double p = lane < sub_len ? prob(psi[base + lane]) : 0.0;
  const double pin = wave_scan(p, lane);
  const uint64_t over = __ballot(p > 0.0 && pin > t);
  const uint64_t mass = __ballot(p > 0.0);
  uint32_t idx;
  if (over) idx = (uint32_t)__builtin_ctzll(over);
  else idx = mass ? (uint32_t)(63 - __builtin_clzll(mass)) : 0u;
  if (lane == 0) out[k] = base + idx;
}

// Marginal.  Rows of 2^row consecutive amplitudes, one pair per thread: the
// selected bits below `row` follow from the thread and the pair's half, those
// above it (hsel) from the workgroup, so reads are whole rows whatever is
// selected.  Workgroup (hb, c) sums the rows of chunk c of high bin hb, then
// folds its pairs into the low bins; partial[(hb chunks + c) 2^kl + lb].
// Bound by the read of the state: 26 qubits, 8 of them selected, 168 us with
// an index deposit per amplitude, 91 us.
template <class R>
__global__ void __launch_bounds__(kSampThreads) marginal_kernel(const cplx<R>* __restrict__ psi, MarginalArgs A,
                                                                double* __restrict__ partials) {
  __shared__ double red[2 * kSampThreads];
  const uint32_t hb = blockIdx.x / A.chunks, c = blockIdx.x % A.chunks;
  const bool active = 2u * threadIdx.x < (1u << A.row);
  // state index bits above the row, selected ones fixed to hb's, the others
  // counting: (i | hsel) + 2^row carries over the selected bits
  uint32_t fixed = 0, i = 0;
  for (uint32_t j = 0, m = A.hsel; m; ++j, m &= m - 1u)
    if ((hb >> j) & 1u) fixed |= m & (0u - m);
  for (uint32_t j = 0, m = A.hfree; m; ++j, m &= m - 1u)
    if (((uint64_t)c * A.chunk_rows >> j) & 1u) i |= m & (0u - m);
  double s0 = 0.0, s1 = 0.0;
  constexpr uint32_t kU = 8;
  const cplx2<R>* p2 = reinterpret_cast<const cplx2<R>*>(psi) + threadIdx.x;
  if (active) {
    for (uint32_t r = 0; r < A.chunk_rows; r += kU) {
      cplx2<R> v[kU];
#pragma unroll
      for (uint32_t k = 0; k < kU; ++k) {
        v[k] = cplx2<R>{{R(0), R(0)}, {R(0), R(0)}};
        if (r + k < A.chunk_rows) {
          v[k] = ld_nt(p2 + ((i | fixed) >> 1));
          i = ((i | ~A.hfree) + 1u) & A.hfree;
        }
      }
#pragma unroll
      for (uint32_t k = 0; k < kU; ++k) {
        s0 += prob(v[k].a);
        s1 += prob(v[k].b);
      }
    }
  }
  red[2 * threadIdx.x] = s0;
  red[2 * threadIdx.x + 1] = s1;
  __syncthreads();
  // fold the row's unselected bits away, the highest first (a fixed order);
  // what is left sits at the positions made of selected bits alone
  const uint32_t rest = ((1u << A.row) - 1u) & ~A.lsel;
  for (uint32_t bit = 1u << 8, folded = 0; bit; bit >>= 1) {
    if (!(rest & bit)) continue;
    folded |= bit;
    for (uint32_t p = threadIdx.x; p < (1u << A.row); p += kSampThreads)
      if (!(p & folded)) red[p] += red[p | bit];
    __syncthreads();
  }
  const uint32_t kl = (uint32_t)__builtin_popcount(A.lsel);
  for (uint32_t lb = threadIdx.x; lb < (1u << kl); lb += kSampThreads) {
    uint32_t at = 0;
    for (uint32_t j = 0, m = A.lsel; m; ++j, m &= m - 1u)
      if ((lb >> j) & 1u) at |= m & (0u - m);
    partials[((size_t)blockIdx.x << kl) + lb] = red[at];
  }
}

// One wavefront per bin adds its chunks: lanes strided, then a fixed butterfly.
__global__ void __launch_bounds__(kSampThreads) marginal_finalize(const double* __restrict__ partials,
                                                                  uint32_t bins, uint32_t chunks, uint32_t kl,
                                                                  double* __restrict__ out) {
  const uint32_t lane = threadIdx.x & 63u, waves = gridDim.x * (kSampThreads / 64);
  for (uint32_t b = blockIdx.x * (kSampThreads / 64) + (threadIdx.x >> 6); b < bins; b += waves) {
    const double* p = partials + ((size_t)(b >> kl) * chunks << kl) + (b & ((1u << kl) - 1u));
    double t = 0.0;
    for (uint32_t c = lane; c < chunks; c += 64) t += p[(size_t)c << kl];
    t = wave_sum_fixed(t);
    if (lane == 0) out[b] = t;
  }
}

inline unsigned grid_of(uint64_t work, int per_block, unsigned cap) {
  uint64_t g = (work + per_block - 1) / per_block;
  return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace

SampleGeom sample_geometry(int n) {
  SampleGeom G;
  G.sub_len = n >= 6 ? 64u : (1u << n);
  const uint32_t blk_len = n >= 14 ? (1u << 14) : (1u << n);
  G.subs_per_block = blk_len / G.sub_len;
  G.n_blk = (1ull << n) / blk_len;
  G.n_sub = G.n_blk * G.subs_per_block;
  return G;
}

size_t sample_scratch_doubles(int n) {
  const SampleGeom G = sample_geometry(n);
  return G.n_sub + G.n_blk + (G.n_blk + 1);
}

template <class R>
void launch_sample(const cplx<R>* psi, int n, const double* u_dev, uint64_t count, uint64_t* out_dev,
                   double* work, hipStream_t s) {
  const SampleGeom G = sample_geometry(n);
  double* sub = work;
  double* blk = sub + G.n_sub;
  double* P = blk + G.n_blk;
  QS_LAUNCH("sample_masses", s, block_masses_kernel<R>, dim3(grid_of(G.n_blk, 1, 1u << 20)), dim3(kSampThreads), 0, s,
            psi, G.n_blk, G.subs_per_block, G.sub_len, sub, blk);
  QS_LAUNCH("sample_scan", s, block_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, blk, G.n_blk, P);
  if (count)
    QS_LAUNCH("sample_draw", s, sample_kernel<R>, dim3(grid_of(count, kSampThreads / 64, 1u << 30)),
              dim3(kSampThreads), 0, s, psi, sub, P, G.n_blk, G.subs_per_block, G.sub_len, u_dev, count,
              out_dev);
}

// ---- allocation-free sampling ----------------------------------------------
// Static scratch of qs_sample_noalloc, one copy per GPU (kept until the
// process ends): nothing in it needs clearing, since every region is written
// before it is read within a call.  Calls that overlap on one GPU share it.
namespace {
constexpr size_t kNaSumDoubles = ((size_t)1 << (kNoAllocSampleMaxQubits - 6)) +
                                 2 * ((size_t)1 << (kNoAllocSampleMaxQubits - 14)) + 1;
constexpr size_t kNaDoubles = kNaSumDoubles + 2 * kNoAllocSampleMaxDraws;
constexpr int kNaMaxDevices = 64;
std::mutex g_na_mu;
double* g_na_ptr[kNaMaxDevices] = {};
}  // namespace

static __device__ __align__(256) double scratch[kNaDoubles];

NoAllocSampleScratch noalloc_sample_scratch(int device) {
  if (device < 0 || device >= kNaMaxDevices) fail(QS_EINVAL, "device ordinal out of range");
  double* base;
  {
    std::lock_guard<std::mutex> lk(g_na_mu);
    if (!g_na_ptr[device]) {
      // the array's address differs per device: look it up with that device current
      int prev = 0;
      check_hip(hipGetDevice(&prev), "hipGetDevice");
      if (prev != device) check_hip(hipSetDevice(device), "hipSetDevice");
      void* p = nullptr;
      const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (prev != device) (void)hipSetDevice(prev);
      check_hip(e, "hipGetSymbolAddress(scratch)");
      g_na_ptr[device] = (double*)p;
    }
    base = g_na_ptr[device];
  }
  NoAllocSampleScratch S;
  S.sums = base;
  S.u = S.sums + kNaSumDoubles;
  S.out = (uint64_t*)(S.u + kNoAllocSampleMaxDraws);
  return S;
}

size_t marginal_partials(const MarginalArgs& A) { return ((size_t)1 << A.k) * A.chunks; }

MarginalArgs marginal_geometry(int n, const int* sel_bits, int k) {
  MarginalArgs A{};
  A.k = (uint32_t)k;
  A.row = (uint32_t)(n < 9 ? n : 9);  // 2 kSampThreads amplitudes
  uint32_t sel = 0;
  for (int j = 0; j < k; ++j) sel |= 1u << sel_bits[j];
  const uint32_t row_mask = (1u << A.row) - 1u, all = n >= 32 ? 0xffffffffu : (1u << n) - 1u;
  A.lsel = sel & row_mask;
  A.hsel = sel & ~row_mask;
  A.hfree = all & ~row_mask & ~sel;
  const uint32_t rows = 1u << __builtin_popcount(A.hfree), hbins = 1u << __builtin_popcount(A.hsel);
  // about 4096 workgroups in all, at least eight rows (the loads in flight) each
  uint32_t chunks = hbins < 4096u ? 4096u / hbins : 1u;
  while (chunks > 1 && rows / chunks < 8) chunks >>= 1;
  A.chunks = chunks;
  A.chunk_rows = rows / chunks;
  return A;
}

template <class R>
void launch_marginal(const cplx<R>* psi, const MarginalArgs& A, double* partials, double* out, hipStream_t s) {
  const uint32_t bins = 1u << A.k, kl = (uint32_t)__builtin_popcount(A.lsel);
  QS_LAUNCH("marginal", s, marginal_kernel<R>, dim3((bins >> kl) * A.chunks), dim3(kSampThreads), 0, s, psi, A,
            partials);
  QS_LAUNCH("marginal_finalize", s, marginal_finalize, dim3(grid_of(bins, kSampThreads / 64, 4096)),
            dim3(kSampThreads), 0, s, partials, bins, A.chunks, kl, out);
}

template void launch_sample<float>(const cplx<float>*, int, const double*, uint64_t, uint64_t*, double*, hipStream_t);
template void launch_sample<double>(const cplx<double>*, int, const double*, uint64_t, uint64_t*, double*,
                                    hipStream_t);
template void launch_marginal<float>(const cplx<float>*, const MarginalArgs&, double*, double*, hipStream_t);
template void launch_marginal<double>(const cplx<double>*, const MarginalArgs&, double*, double*, hipStream_t);

}  // namespace qs
