// Dense k-qubit blocks (k = 4, 5, 6) on the matrix cores.
//
// A block applies a 2^k x 2^k complex matrix U to the k target bits of every
// basis index: for each assignment of the other bits (a column), the 2^k
// amplitudes along the targets are multiplied by U.  That is a complex matrix
// product Y = U X with X of shape 2^k x (number of columns); the paper names
// generic matrix fusion of such windows as its next extension (Section
// "Limitations and Future Work"), and it is the one layer here whose
// arithmetic intensity (8 2^k flop per amplitude, 2^(k-1) flop per byte in
// complex64) reaches the matrix cores' ridge.
//
// Tiles: the target bits plus the c lowest non-target bits (the columns).
// Every tile bit below the c-th non-target bit is in the tile, so the tile's
// low L >= c bits are the state's low bits and loads/stores move runs of
// 2^L >= 16 consecutive amplitudes; the remaining tile bits are targets.  A
// workgroup (4 waves) stages a tile in LDS; wave w takes 16-column blocks w,
// w + 4, ...; each block's product is 4 real MFMA 16x16x4 chains per 16-row tile
// of U:
//   Yr += Ur Xr + Ui (-Xi),   Yi += Ur Xi + Ui Xr,
// with U's fragments held in registers for the whole kernel and X's read from
// LDS.  Results go back to the same LDS columns (each column block is read and
// written by one wave only, or, for k = 6, by one pair of waves that each
// compute half of its rows, with a barrier between their reads and writes), then
// the tile is stored.
//
// What bounds them: HBM, and for k = 6 (complex128 also k = 5) the matrix cores.
// Address arithmetic is kept off the tile loop (it cost up to a third of it): a
// thread's state and LDS offsets are a lane part plus uniform parts, held in
// registers.  us per block with FP32 products for complex64 k = 5 and 6, deposits
// and tables in the tile loop and 2048 workgroups, and now:
//             complex64                      complex128
//   n      k=4       k=5       k=6       k=4       k=5        k=6
//   16   5.4 4.1   8.1 6.7  15.3 11.1  6.4 5.0  10.1 7.1   20.6 14.3
//   22    20  15    30  18    42   27    30  24    49  32     85   52
//   25   108  83   123  90   194  133   204 179   250 198    451  308
//   27   440 375   446 393   681  527   857 743   933 822   1633 1206
// (27 qubits complex64: 2.1 GB moved, 5.7, 5.5 and 4.1 TB/s; a copy of this
// size reaches 5.65.)
//
// Operand layouts of V_MFMA_{F32,F64}_16X16X4 (wave64): A[i][kk] in lane
// i + 16 kk, B[kk][j] in lane j + 16 kk; D[i][j] in lane j + 16 (i / 4),
// register i % 4 for F32, and in lane j + 16 (i % 4), register i / 4 for F64
// (checked by a one-hot probe of both builtins).
#include "kernels.h"
#include "lanes.h"

#include <type_traits>

namespace qs {

namespace {

constexpr int kDenseThreads = 256;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <class R>
struct Acc4;
template <>
struct Acc4<float> {
  typedef f32x4 T;
};
template <>
struct Acc4<double> {
  typedef f64x4 T;
};

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mfma16(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// LDS element of tile position pos (two pad elements every 32).
__device__ __forceinline__ uint32_t dense_lds_off(uint32_t pos) { return pos + ((pos >> 5) << 1); }

// First state index of tile t: zeros inserted at the tile's bits, [0, L) and
// hi_bit (ascending).
__device__ __forceinline__ uint32_t dense_tile_base(uint32_t t, const DenseGeom& G) {
  uint32_t base = t << G.L;
#pragma unroll
  for (uint32_t j = 0; j < 6; ++j)
    if (j < G.n_hi) {
      const uint32_t b = G.hi_bit[j];
      base = ((base >> b) << b << 1) | (base & ((1u << b) - 1u));
    }
  return base;
}

// A thread's kN accesses of W adjacent amplitudes to each tile of at most
// W NT kN amplitudes: positions W (tid + NT k), modulo the tile where it is
// smaller (several threads then move the same amplitudes: a branch here would
// make a wait for the next tile's loads one for this tile's stores as well).
// The state offset of a position is the thread's part (one pointer for the
// whole kernel) and a uniform part of k and the tile, so an access costs one
// address addition.  All of a tile's loads are issued before the first is
// waited for.
template <class R, int W, int kN, uint32_t NT>
struct DenseIO {
  typedef typename std::conditional<W == 2, cplx2<R>, cplx<R>>::type V;
  cplx<R>* lane;
  uint32_t uni[kN];        // state offsets of the uniform parts
  uint32_t tid_lds, uni_lds[kN];
  __device__ __forceinline__ static uint32_t offset(uint32_t p, const DenseGeom& G) {
    uint32_t off = p & ((1u << G.L) - 1u);
#pragma unroll
    for (uint32_t j = 0; j < 6; ++j) off |= ((p >> (G.L + j)) & 1u) << G.hi_bit[j];
    return off;
  }
  __device__ __forceinline__ DenseIO(cplx<R>* psi, const DenseGeom& G) {
    const uint32_t wrap = (1u << G.m) - 1u;
    lane = psi + offset((W * threadIdx.x) & wrap, G);
    tid_lds = dense_lds_off((W * threadIdx.x) & wrap);
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      uni[k] = offset((W * NT * k) & wrap, G);
      uni_lds[k] = dense_lds_off((W * NT * k) & wrap);
    }
  }
  template <bool kKeep>
  __device__ __forceinline__ void issue(uint32_t base, V (&v)[kN]) const {
#pragma unroll
    for (int k = 0; k < kN; ++k) v[k] = ld_state<kKeep>(reinterpret_cast<const V*>(lane + (base | uni[k])));
  }
  __device__ __forceinline__ void issue(bool keep, uint32_t base, V (&v)[kN]) const {
    if (keep) issue<true>(base, v);
    else issue<false>(base, v);
  }
  __device__ __forceinline__ void put(cplx<R>* T, const V (&v)[kN]) const {
#pragma unroll
    for (int k = 0; k < kN; ++k) *reinterpret_cast<V*>(T + tid_lds + uni_lds[k]) = v[k];
  }
  __device__ __forceinline__ void load(bool keep, uint32_t base, cplx<R>* T) const {
    V v[kN];
    issue(keep, base, v);
    put(T, v);
  }
  __device__ __forceinline__ void store(uint32_t base, const cplx<R>* T) const {
    V v[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) v[k] = *reinterpret_cast<const V*>(T + tid_lds + uni_lds[k]);
#pragma unroll
    for (int k = 0; k < kN; ++k) st_nt(reinterpret_cast<V*>(lane + (base | uni[k])), v[k]);
  }
};

// LDS offsets of the single target (row) and column bits, in increasing order;
// the offset of several bits is their sum.
struct DenseBits {
  uint32_t row[6], col[6];
  __device__ __forceinline__ explicit DenseBits(const DenseGeom& G) {
    uint32_t r = G.rowmask, c = ((1u << G.m) - 1u) & ~G.rowmask;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      row[j] = dense_lds_off(r & (0u - r));
      r &= r - 1u;
      col[j] = dense_lds_off(c & (0u - c));
      c &= c - 1u;
    }
  }
  // row bits from `at` on of v < 2^nb
  __device__ __forceinline__ uint32_t rows(uint32_t v, int at, int nb) const {
    uint32_t o = 0;
#pragma unroll
    for (int j = 0; j < nb; ++j) o += (v >> j) & 1u ? row[at + j] : 0u;
    return o;
  }
  // column 16 cb + li: a lane's part and a uniform one
  __device__ __forceinline__ uint32_t col_lane(uint32_t li) const {
    uint32_t o = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) o += (li >> j) & 1u ? col[j] : 0u;
    return o;
  }
  __device__ __forceinline__ uint32_t col_block(uint32_t cb) const {
    return (cb & 1u ? col[4] : 0u) + (cb & 2u ? col[5] : 0u);
  }
};

template <class R, int K>
__global__ void __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(3)))
dense_kernel(cplx<R>* __restrict__ psi, const cplx<R>* U_, DenseGeom G) {
  constexpr int KS = K / 4;   // 4-deep steps of the contraction
  constexpr int RT = K / 16;  // 16-row tiles of U
  typedef typename Acc4<R>::T acc_t;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<R>* T = reinterpret_cast<cplx<R>*>(smem_raw);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t li = lane & 15u, lk = lane >> 4;

  // U fragments: A[i][kk] = U[16 rt + i][4 ks + kk]
  const cptr<cplx<R>> U = to_const(U_);
  R ur[RT][KS], ui[RT][KS];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint32_t e = (16u * rt + li) * K + 4u * ks + lk;
      ur[rt][ks] = U[e].re;
      ui[rt][ks] = U[e].im;
    }
  // rows a lane reads, 4 ks + lk, and writes, 16 rt + (4 lk + v or lk + 4 v)
  const DenseBits B(G);
  constexpr int kV = sizeof(R) == 4 ? 0 : 2;  // the row bits of register v in D
  const uint32_t rd = B.col_lane(li) + B.rows(lk, 0, 2), wr = B.col_lane(li) + B.rows(lk, 2 - kV, 2);
  const uint32_t ncb = (1u << G.c) >> 4;
  // complex128: one 16-byte amplitude per lane and access (in pairs, a wave's
  // access covers every other 16 bytes of its lines: k = 5 at 27 qubits 1380
  // against 810 us).  No prefetch of the next tile: at k = 4 and 5 it gains
  // nothing or loses.
  constexpr int W = sizeof(R) == 8 ? 1 : 2;
  const DenseIO<R, W, K * 64 / (W * kDenseThreads), kDenseThreads> io(psi, G);
  for (uint32_t t = blockIdx.x; t < G.n_tiles; t += gridDim.x) {
    const uint32_t base = dense_tile_base(t, G);
    io.load(G.keep, base, T);
    __syncthreads();
    for (uint32_t cb = wave; cb < ncb; cb += 4u) {
      const uint32_t colp = B.col_block(cb);
      acc_t yr[RT], yi[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        yr[rt] = acc_t{0, 0, 0, 0};
        yi[rt] = acc_t{0, 0, 0, 0};
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const cplx<R> x = T[rd + colp + B.rows(ks, 2, 3)];
        const R nxi = -x.im;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          yr[rt] = mfma16(ur[rt][ks], x.re, yr[rt]);
          yr[rt] = mfma16(ui[rt][ks], nxi, yr[rt]);
          yi[rt] = mfma16(ur[rt][ks], x.im, yi[rt]);
          yi[rt] = mfma16(ui[rt][ks], x.re, yi[rt]);
        }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          T[wr + colp + B.rows(v, kV, 2) + B.rows(rt, 4, 1)] = cplx<R>{yr[rt][v], yi[rt][v]};
    }
    __syncthreads();
    io.store(base, T);
    __syncthreads();
  }
}

// ---- complex64 k = 5 and 6 on the bf16 matrix cores ----------------------------
// The FP32 matrix cores make k = 6 compute-bound (27 qubits, this tile loop: 575
// us, against the 380 that the state's traffic takes) and k = 5 nearly so (405).
// A float is the exact sum h + m + l of three bf16 numbers (8 significant bits
// each, signs absorbing the rest), so U X = sum_ij U_i X_j with products that are
// exact in FP32; the six with i + j <= 4 are taken, the three left out are below
// 2^-24 of |u| |x| in all and of random sign.  Six bf16 products cost 6 / 16 of
// an FP32 one, and 32 of them enter an accumulator per instruction instead of 4.
//
// V_MFMA_F32_16X16X32_BF16: lane l holds row (A) or column (B) l % 16 and the
// eight depths of its quarter l / 16 (A and B alike, so the contraction does not
// depend on their order); D as for the FP32 16x16 forms.  What it rounds (probed
// with single products): a quarter's eight products are cut, towards zero, at
// 2^-24 of the largest one and added; the sum enters the accumulator with one
// rounding to nearest, a smaller accumulator first being cut there too, downwards.
// Beside a product with an entry of U near one, those with U's small entries so
// lose their last bits, and with the same sign each time: a window near the
// identity, applied again and again as Trotter steps do, had an error that grew
// with the number of steps.  U's heads h are therefore taken in two, the large
// ones (from an eighth of U's largest entry on) and the others, each with
// products, and the large ones with accumulators, of their own: seven products.
//
// Error (2-norm) against complex128, FP32 forms, six products, now, for 1, 40 and
// 400 applications, 1e-7:
//   k = 5  window within 1e-3 of 1   1.5  17  91   0.9  25  233   0.3  7.3  71
//          random unitary            1.5 9.3  34   0.5 3.7   21   0.5  3.1  20
//   k = 6  window within 1e-3 of 1   2.1  26 119   1.2  31  265   0.3  7.0  68
//          random unitary            2.0  13  43   1.2 7.4   26   0.6  3.6  16
// (what is left near the identity is U's rounding to float).  27 qubits: k = 5 379
// us with six products, 393 now, k = 6 487 and 527.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// x = h + m + l, eight numbers at a time (converted in pairs).
struct Split8 {
  bf16x8 h, m, l;
};
__device__ __forceinline__ uint32_t to_bf16x2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ void split8(const float (&x)[8], Split8& S) {
  u32x4 h, m, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    h[e] = to_bf16x2(x[2 * e], x[2 * e + 1]);
    const float r0 = x[2 * e] - __uint_as_float(h[e] << 16);
    const float r1 = x[2 * e + 1] - __uint_as_float(h[e] & 0xffff0000u);
    m[e] = to_bf16x2(r0, r1);
    l[e] = to_bf16x2(r0 - __uint_as_float(m[e] << 16), r1 - __uint_as_float(m[e] & 0xffff0000u));
  }
  S.h = __builtin_bit_cast(bf16x8, h);
  S.m = __builtin_bit_cast(bf16x8, m);
  S.l = __builtin_bit_cast(bf16x8, l);
}
// U's numbers: h in two, the large ones (from `large` on) and the others.
struct SplitU8 {
  u32x4 big, rest, m, l;
  __device__ __forceinline__ SplitU8() = default;
  __device__ __forceinline__ SplitU8(const float (&u)[8], float large) {
    Split8 S;
    split8(u, S);
    const u32x4 h = __builtin_bit_cast(u32x4, S.h);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t keep = (fabsf(u[2 * e]) >= large ? 0xffffu : 0u) | (fabsf(u[2 * e + 1]) >= large ? 0xffff0000u : 0u);
      big[e] = h[e] & keep;
      rest[e] = h[e] & ~keep;
    }
    m = __builtin_bit_cast(u32x4, S.m);
    l = __builtin_bit_cast(u32x4, S.l);
  }
  // h, put together where it is used: `never`, a zero that the compiler cannot know,
  // keeps it from holding h in registers as well
  __device__ __forceinline__ u32x4 head(uint32_t never) const { return (big ^ never) | rest; }
};
__device__ __forceinline__ f32x4 mfma_bf16(const u32x4& a, const bf16x8& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), b, c, 0, 0, 0);
}
__device__ __forceinline__ void negate(Split8& S) {
  S.h = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, S.h) ^ 0x80008000u);
  S.m = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, S.m) ^ 0x80008000u);
  S.l = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, S.l) ^ 0x80008000u);
}
// A lane mask folded over the four lanes l, l + 16, ... of a column: 16 bits.
__device__ __forceinline__ uint32_t fold_or16(uint64_t m) {
  const uint32_t w = (uint32_t)m | (uint32_t)(m >> 32);
  return (w | w >> 16) & 0xffffu;
}
__device__ __forceinline__ uint32_t fold_xor16(uint64_t m) {
  const uint32_t w = (uint32_t)m ^ (uint32_t)(m >> 32);
  return w ^ w >> 16;
}
// The split's range.  Below 2^-109 or so l's last bits are under bf16's range, where
// the matrix cores take zero (a state of amplitudes around 2^-115 had an error of
// 1.6e-6, around 2^-120 5e-5), and the first steps of an evolution from a basis
// state are full of such columns: columns whose first 32 rows all lie below
// kTinyColumn are multiplied by 2^64 (exact), their results by 2^-64.  What the
// others lose is below 2^-60 of their largest number.  The finite floats from
// kSplitMax on round to infinity in bf16, and an infinity's remainder is no number: a
// tile with such a number (scaled, if it is), or a matrix with one or of tiny
// entries only, takes the FP32 forms.
constexpr float kSplitMax = 0x1.ffp127f, kTinyColumn = 0x1p-60f, kTinyMatrix = 0x1p-96f;
constexpr float kLargeU = 0x1p-3f;  // of U's largest entry
// max(m, |a|, |b|) in one instruction (fmaxf first canonicalises each operand)
__device__ __forceinline__ float max3_abs(float m, float a, float b) {
  asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
  return m;
}

// k = 6: the two waves of a pair take the same column blocks, each two of U's
// four 16-row tiles, with a barrier between a block's reads and its in-place
// writes; k = 5: a wave takes whole column blocks.  At k = 6 the next tile's
// loads are issued before this tile's contraction (two waves per SIMD hold them
// and U's parts; three spill).
template <int K>
__global__ void __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(K == 64 ? 2 : 3)))
dense_split_kernel(cplx<float>* __restrict__ psi, const cplx<float>* U_, DenseGeom G) {
  constexpr int kSlabs = K / 32, RT = 2;
  constexpr bool kPair = K == 64;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<float>* T = reinterpret_cast<cplx<float>*>(smem_raw);
  uint32_t* unfit = reinterpret_cast<uint32_t*>(smem_raw + sizeof(cplx<float>) * dense_lds_off(1u << G.m));
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t li = lane & 15u, lk = lane >> 4;
  const uint32_t rt0 = kPair ? 2u * (wave & 1u) : 0u;
  const uint32_t cb0 = kPair ? wave >> 1 : wave, cbs = kPair ? 2u : 4u;
  const DenseIO<float, 2, K / 8, kDenseThreads> io(psi, G);
  cplx2<float> pre[K / 8];
  if (kPair && blockIdx.x < G.n_tiles) io.issue(G.keep, dense_tile_base(blockIdx.x, G), pre);
  SplitU8 ur[RT][kSlabs], ui[RT][kSlabs];
  bool u_unfit;
  {
    float re[RT][kSlabs][8], im[RT][kSlabs][8], m = 0.0f;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int sl = 0; sl < kSlabs; ++sl) {
        const cplx<float>* u = U_ + (16u * (rt0 + rt) + li) * K + 32u * sl + 8u * lk;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          re[rt][sl][e] = u[e].re;
          im[rt][sl][e] = u[e].im;
          m = max3_abs(m, re[rt][sl][e], im[rt][sl][e]);
        }
      }
    m = wave_max(m);
    u_unfit = m >= kSplitMax || m < kTinyMatrix;
    const float large = m * kLargeU;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int sl = 0; sl < kSlabs; ++sl) {
        ur[rt][sl] = SplitU8(re[rt][sl], large);
        ui[rt][sl] = SplitU8(im[rt][sl], large);
      }
  }
  // rows a lane reads, 32 sl + 8 lk + e, and writes, 16 (rt0 + rt) + 4 lk + v
  const DenseBits B(G);
  const uint32_t rd = B.col_lane(li) + B.rows(lk, 3, 2);
  const uint32_t wr = B.col_lane(li) + B.rows(lk, 2, 2) + (rt0 ? B.row[5] : 0u);
  const uint32_t ncb = (1u << G.c) >> 4;
  const uint32_t trips = (ncb + cbs - 1u) / cbs;  // uniform: barriers inside
  for (uint32_t t = blockIdx.x; t < G.n_tiles; t += gridDim.x) {
    const uint32_t base = dense_tile_base(t, G);
    if (threadIdx.x == 0) *unfit = 0u;
    if constexpr (kPair) {
      io.put(T, pre);
      if (t + gridDim.x < G.n_tiles) io.issue(G.keep, dense_tile_base(t + gridDim.x, G), pre);
    } else {
      io.load(G.keep, base, T);
    }
    __syncthreads();
    bool bad = u_unfit;
    for (uint32_t it = 0; it < trips; ++it) {
      const uint32_t cb = cb0 + it * cbs;
      const bool on = cb < ncb;
      const uint32_t colp = B.col_block(cb);
      // real and imaginary: the products of U's large heads with heads, and the others
      f32x4 hr[RT], hi[RT], sr[RT], si[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) hr[rt] = hi[rt] = sr[rt] = si[rt] = f32x4{0, 0, 0, 0};
      float scale = 1.0f;
      if (on) {
        uint32_t never = 0u;
        asm volatile("" : "+s"(never));
        float m = 0.0f;
#pragma unroll
        for (int sl = 0; sl < kSlabs; ++sl) {
          float re[8], im[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const cplx<float> x = T[rd + colp + B.rows(e, 0, 3) + (sl ? B.row[5] : 0u)];
            re[e] = x.re;
            im[e] = x.im;
            m = max3_abs(m, x.re, x.im);
          }
          // Half of the columns are multiplied as -X and negated again, by a bit of
          // the data and one of a hash of the place: with one sign, what is cut
          // downwards would add up over the amplitudes (a transform circuit of dense
          // windows on 20 qubits: 5.6e-5 of a mean amplitude in one output instead of
          // 2e-6) and over the applications of a window.
          if (sl == 0) {
            uint32_t hash = (4u * t + cb) * 0x85ebca6bu;
            hash = (hash ^ (hash >> 13)) * 0xc2b2ae35u;
            const uint64_t odd = __ballot(__float_as_uint(m) & 1u);
            const uint32_t col = fold_xor16(odd) ^ (uint32_t)((int32_t)hash >> 31);
            const uint32_t sgn = (col >> li) << 31;
            const uint32_t tiny = (~fold_or16(__ballot(m >= kTinyColumn)) >> li & 1u) << 29;  // 64 in the exponent
            scale = __uint_as_float(0x3f800000u + tiny | sgn);
          }
          {
// (as multiply-adds with the split's first differences, the unscaled numbers would
// stay in registers)
#pragma clang fp contract(off)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              re[e] *= scale;
              im[e] *= scale;
            }
          }
          Split8 x;
          // h and s += u x, of s the smallest products first
          auto mul = [&](const SplitU8& u, f32x4& h, f32x4& s) {
            const u32x4 uh = u.head(never);
            s = mfma_bf16(u.l, x.h, s);
            s = mfma_bf16(uh, x.l, s);
            s = mfma_bf16(u.m, x.m, s);
            s = mfma_bf16(u.m, x.h, s);
            s = mfma_bf16(uh, x.m, s);
            s = mfma_bf16(u.rest, x.h, s);
            h = mfma_bf16(u.big, x.h, h);
          };
          split8(re, x);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            mul(ur[rt][sl], hr[rt], sr[rt]);
            mul(ui[rt][sl], hi[rt], si[rt]);
          }
          split8(im, x);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) mul(ur[rt][sl], hi[rt], si[rt]);
          negate(x);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) mul(ui[rt][sl], hr[rt], sr[rt]);
        }
        bad = bad || __any(fabsf(m * scale) >= kSplitMax);
      }
      if constexpr (kPair) __syncthreads();
      if (on) {
        const float unscale = __uint_as_float(0x7f000000u - __float_as_uint(scale));  // 1 / scale
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            T[wr + colp + B.rows(v, 0, 2) + B.rows(rt, 4, 1)] =
                cplx<float>{unscale * (hr[rt][v] + sr[rt][v]), unscale * (hi[rt][v] + si[rt][v])};
      }
    }
    if (bad && lane == 0) *unfit = 1u;
    __syncthreads();
    if (__builtin_expect(*unfit, 0u)) {
      io.load(false, base, T);  // the state still holds the tile
      __syncthreads();
      for (uint32_t it = 0; it < trips; ++it) {
        const uint32_t cb = cb0 + it * cbs;
        const uint32_t colp = cb < ncb ? B.col_block(cb) : 0u;
        f32x4 yr[RT], yi[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) yr[rt] = yi[rt] = f32x4{0, 0, 0, 0};
#pragma unroll 1
        for (uint32_t ks = 0; ks < (uint32_t)K / 4u; ++ks) {
          const cplx<float> x = T[B.col_lane(li) + colp + B.rows(lk, 0, 2) + B.rows(ks, 2, 4)];
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            const cplx<float> u = U_[(16u * (rt0 + rt) + li) * K + 4u * ks + lk];
            yr[rt] = mfma16(u.re, x.re, yr[rt]);
            yr[rt] = mfma16(u.im, -x.im, yr[rt]);
            yi[rt] = mfma16(u.re, x.im, yi[rt]);
            yi[rt] = mfma16(u.im, x.re, yi[rt]);
          }
        }
        if constexpr (kPair) __syncthreads();
        if (cb < ncb) {
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              T[wr + colp + B.rows(v, 0, 2) + B.rows(rt, 4, 1)] = cplx<float>{yr[rt][v], yi[rt][v]};
        }
      }
      __syncthreads();
    }
    io.store(base, T);
    __syncthreads();
  }
}

// complex128 k = 6: the 64 x 64 matrix (64 KB) does not fit the register
// file, so it is staged in LDS next to the tile and each wave reads its A
// fragments from there; otherwise as dense_kernel (f64 MFMA, D[i][j] in lane
// j + 16 (i % 4), register i / 4).  The staged rows are kUsStride = 65
// entries apart: the 16 rows a fragment read touches then fall in 16
// different bank groups (at 64 they would all share one).
constexpr int kUsStride = 65;
constexpr uint32_t kThreads6 = 512;
__global__ void __launch_bounds__(kThreads6) dense_kernel_k6_c128(cplx<double>* __restrict__ psi,
                                                                  const cplx<double>* U_, DenseGeom G) {
  // 512 threads, two waves per SIMD: the waves of a pair take the same
  // column block, each two of U's four 16-row tiles (as the complex64 k = 6
  // split), with a barrier between a column block's reads and its in-place
  // writes
  constexpr int K = 64, RT = 2, KS = K / 4;
  constexpr uint32_t NT = kThreads6;
  typedef f64x4 acc_t;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<double>* T = reinterpret_cast<cplx<double>*>(smem_raw);
  cplx<double>* Us = T + dense_lds_off(1u << G.m);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t li = lane & 15u, lk = lane >> 4;
  const uint32_t rt0 = 2u * (wave & 1u), cb0 = wave >> 1, cbs = NT / 128u;
  // the next tile's loads are issued before this tile's contraction (one
  // workgroup per CU: tile and matrix fill the LDS); one amplitude per lane and
  // access (1236 us at 27 qubits, in pairs 1350)
  const DenseIO<double, 1, 8, NT> io(psi, G);
  cplx<double> pre[8];
  if (blockIdx.x < G.n_tiles) io.issue(G.keep, dense_tile_base(blockIdx.x, G), pre);
  for (uint32_t e = threadIdx.x; e < (uint32_t)(K * K); e += NT) Us[(e / K) * kUsStride + e % K] = U_[e];
  const DenseBits B(G);
  const uint32_t rd = B.col_lane(li) + B.rows(lk, 0, 2);
  const uint32_t wr = rd + (rt0 ? B.row[5] : 0u);
  const uint32_t ncb = (1u << G.c) >> 4;
  const uint32_t trips = (ncb + cbs - 1u) / cbs;
  for (uint32_t t = blockIdx.x; t < G.n_tiles; t += gridDim.x) {
    const uint32_t base = dense_tile_base(t, G);
    io.put(T, pre);
    __syncthreads();
    if (t + gridDim.x < G.n_tiles) io.issue(G.keep, dense_tile_base(t + gridDim.x, G), pre);
    for (uint32_t it = 0; it < trips; ++it) {
      const uint32_t cb = cb0 + it * cbs;
      const bool active = cb < ncb;
      const uint32_t colp = B.col_block(cb);
      acc_t yr[RT], yi[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        yr[rt] = acc_t{0, 0, 0, 0};
        yi[rt] = acc_t{0, 0, 0, 0};
      }
      if (active) {
#pragma unroll 4
        for (int ks = 0; ks < KS; ++ks) {
          const cplx<double> x = T[rd + colp + B.rows(ks, 2, 4)];
          const double nxi = -x.im;
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            const cplx<double> u = Us[(16u * (rt0 + rt) + li) * kUsStride + 4u * ks + lk];
            yr[rt] = mfma16(u.re, x.re, yr[rt]);
            yr[rt] = mfma16(u.im, nxi, yr[rt]);
            yi[rt] = mfma16(u.re, x.im, yi[rt]);
            yi[rt] = mfma16(u.im, x.re, yi[rt]);
          }
        }
      }
      __syncthreads();  // both waves of the pair have read the column block
      if (active) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            T[wr + colp + B.rows(v, 2, 2) + B.rows(rt, 4, 1)] = cplx<double>{yr[rt][v], yi[rt][v]};
      }
    }
    __syncthreads();
    io.store(base, T);
    __syncthreads();
  }
}

}  // namespace

bool dense_supported(int n, int k, bool complex128) {
  (void)complex128;  // complex128 k = 6 stages its matrix in LDS
  return k >= 4 && k <= 6 && n - k >= 4 && n <= 32;
}

DenseGeom dense_geometry(int n, int k, const int* bits_sorted) {
  DenseGeom G{};
  uint32_t tmask = 0;
  for (int j = 0; j < k; ++j) tmask |= 1u << bits_sorted[j];
  const int c = n - k < 6 ? n - k : 6;
  // tile bits: the targets plus the c lowest other bits
  uint32_t bmask = tmask;
  for (int b = 0, got = 0; b < n && got < c; ++b)
    if (!((tmask >> b) & 1u)) {
      bmask |= 1u << b;
      ++got;
    }
  int L = 0;
  while (L < n && ((bmask >> L) & 1u)) ++L;
  G.m = (uint32_t)(k + c);
  G.c = (uint32_t)c;
  G.L = (uint32_t)L;
  // tile position of every tile bit = its rank in bmask
  uint32_t rowmask = 0, pos = 0;
  for (int b = 0; b < n; ++b)
    if ((bmask >> b) & 1u) {
      if ((tmask >> b) & 1u) rowmask |= 1u << pos;
      if ((int)pos >= L) G.hi_bit[G.n_hi++] = (uint32_t)b;
      ++pos;
    }
  G.rowmask = rowmask;
  G.n_tiles = 1u << (n - k - c);
  return G;
}

template <class R>
bool launch_dense(cplx<R>* psi, int n, int k, const int* bits_sorted, const cplx<R>* U_dev, hipStream_t s,
                  uint64_t others) {
  if (!dense_supported(n, k, sizeof(R) == 8)) return false;
  DenseGeom G = dense_geometry(n, k, bits_sorted);
  // cached reads, streamed writes (a ladder's 24-qubit window passes 65 against
  // 71 us; cached writes 81, the tiles' short runs evicting each other)
  G.keep = keep_resident((uint64_t)sizeof(cplx<R>) << n, others);
  const uint32_t M = 1u << G.m;
  const size_t lds = sizeof(cplx<R>) * (M + ((M >> 5) << 1)) + sizeof(uint32_t);
  // Two workgroups per CU.  With more, those in flight walk the state further
  // apart and U is read and split more often (27 qubits: complex128 k = 4 756 us,
  // with 2048 825); with one, loads are too few.  Exceptions, measured the same
  // way: complex64 k = 4 (8 KB tiles) three (375 us, two 416), and k = 5 up to 2^16
  // tiles (22 qubits 17.7 us, two 19.1; 25 qubits 90.0 and 90.9; 27 qubits 393 and
  // 389; 28 qubits 791 and 761); complex128 k = 6 one, what the LDS holds (21 qubits
  // 27 us, two 32); complex64 k = 6 more once a workgroup would take over 16 tiles
  // (28 qubits: 1030 us, two 1034).
  uint32_t wgs = 512u;
  if (sizeof(R) == 4 && (k == 4 || (k == 5 && G.n_tiles <= 1u << 16))) wgs = 768u;
  if (sizeof(R) == 4 && k == 6 && G.n_tiles / 16u > wgs) wgs = G.n_tiles / 16u;
  if (sizeof(R) == 8 && k == 6) wgs = 256u;
  const uint32_t grid = G.n_tiles < wgs ? G.n_tiles : wgs;
  if (k == 4) {
    QS_LAUNCH("dense_k4", s, (dense_kernel<R, 16>), dim3(grid), dim3(kDenseThreads), lds, s, psi, U_dev, G);
  } else if (k == 5) {
    if constexpr (sizeof(R) == 4)
      QS_LAUNCH("dense_k5", s, dense_split_kernel<32>, dim3(grid), dim3(kDenseThreads), lds, s, psi, U_dev, G);
    else
      QS_LAUNCH("dense_k5", s, (dense_kernel<R, 32>), dim3(grid), dim3(kDenseThreads), lds, s, psi, U_dev, G);
  } else if constexpr (sizeof(R) == 4) {
    QS_LAUNCH("dense_k6", s, dense_split_kernel<64>, dim3(grid), dim3(kDenseThreads), lds, s, psi, U_dev, G);
  } else {
    // the tile, the 64 x 64 complex128 matrix (rows padded): ~134 KB
    const size_t lds6 = sizeof(cplx<double>) * (M + ((M >> 5) << 1)) + sizeof(cplx<double>) * 64 * kUsStride;
    static bool attr_set = false;
    if (!attr_set) {
      allow_dynamic_lds((const void*)dense_kernel_k6_c128, (int)lds6, "dense_k6");
      attr_set = true;
    }
    QS_LAUNCH("dense_k6", s, dense_kernel_k6_c128, dim3(grid), dim3(kThreads6), lds6, s, psi, U_dev, G);
  }
  return true;
}

template bool launch_dense<float>(cplx<float>*, int, int, const int*, const cplx<float>*, hipStream_t, uint64_t);
template bool launch_dense<double>(cplx<double>*, int, int, const int*, const cplx<double>*, hipStream_t, uint64_t);

}  // namespace qs
