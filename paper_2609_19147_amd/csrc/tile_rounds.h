// The rounds of a tile pass on a tile in LDS: register patterns, their loops
// and the dispatch over a pass's rounds.  Shared by the passes over HBM
// (k_tile.hip) and the sequences of passes on states of one tile (k_seq.hip).
#pragma once
#include "kernels.h"

namespace qs {

namespace {

constexpr int RB = kRoundBits;
constexpr int RN = 1 << RB;

// LDS element of tile position pos (two pad elements every 32).
__device__ __forceinline__ uint32_t lds_off(uint32_t pos) { return pos + ((pos >> 5) << 1); }

struct Ctx {
  uint32_t base;  // coset bits (tile bits zero)
  uint32_t L, a;
  __device__ __forceinline__ uint32_t dep(uint32_t pos) const {
    return (pos & ((1u << L) - 1u)) | ((pos >> L) << a);
  }
};

// u x + v y as one multiply-add chain per component (four instructions each,
// against five for two complex products and an add).
template <class R>
__device__ __forceinline__ cplx<R> cmul2(cplx<R> u, cplx<R> x, cplx<R> v, cplx<R> y) {
  return {fma(u.re, x.re, fma(-u.im, x.im, fma(v.re, y.re, -v.im * y.im))),
          fma(u.re, x.im, fma(u.im, x.re, fma(v.re, y.im, v.im * y.re)))};
}

template <int S, class R>
__device__ __forceinline__ void op_mat(cplx<R>* a, cptr<cplx<R>> u) {
  const cplx<R> u00 = ldc(u, 0), u01 = ldc(u, 1), u10 = ldc(u, 2), u11 = ldc(u, 3);
#pragma unroll
  for (int j = 0; j < RN; ++j) {
    if (j & (1 << S)) continue;
    const cplx<R> x = a[j], y = a[j | (1 << S)];
    a[j] = cmul2(u00, x, u01, y);
    a[j | (1 << S)] = cmul2(u10, x, u11, y);
  }
}

template <int S, class R>
__device__ __forceinline__ void op_diag(cplx<R>* a, cptr<cplx<R>> u) {
  const cplx<R> d0 = ldc(u, 0), d1 = ldc(u, 1);
#pragma unroll
  for (int j = 0; j < RN; ++j) a[j] = cmul((j & (1 << S)) ? d1 : d0, a[j]);
}

// Unscaled Hadamard butterfly (the pass applies 2^(-k/2) at the store).
template <int S, class R>
__device__ __forceinline__ void op_h(cplx<R>* a) {
#pragma unroll
  for (int j = 0; j < RN; ++j) {
    if (j & (1 << S)) continue;
    const cplx<R> x = a[j], y = a[j | (1 << S)];
    a[j] = cadd(x, y);
    a[j | (1 << S)] = csub(x, y);
  }
}

// Unscaled QFT stage on register bit S: a1' = (a0 - a1) t_k with t_k = w E[k],
// w the group twiddle (bits outside the round) and E[k] the intra-round
// factor of the register bits below S.  The inverse stage undoes it:
// a1 <- a1 conj(t_k), then the butterfly.
// kThenH: the Hadamard of bit S follows at once (no later stage of a round
// acts on bit S or is controlled by it): with u = a0 + a1 and
// v = t_k (a0 - a1), a0' = u + v and a1' = 2u - a0' (five multiply-adds and
// four adds per pair instead of twelve operations).
// kSym: E[k + 2^(S-1)] = i E[k], so the upper half of the t_k is the lower
// half times i (register moves and sign flips, no multiplies).
template <int S, class R, bool kInv, bool kThenH = false, bool kSym = false>
__device__ __forceinline__ void op_qft(cplx<R>* a, cplx<R> w, cptr<cplx<R>> E) {
  static_assert(!(kInv && kThenH), "the inverse stage has no fused Hadamard");
  constexpr int K = 1 << S;
  cplx<R> tw[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (kSym && k >= K / 2 && K >= 2)
      tw[k] = {-tw[k - K / 2].im, tw[k - K / 2].re};
    else
      tw[k] = k == 0 ? w : cmul(w, ldc(E, k));
  }
  // pairs (j, j | 2^S) with j = k + hi * 2^(S+1): the twiddle depends on k only
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const cplx<R> t = tw[k];
#pragma unroll
    for (int hi = 0; hi < (RN >> (S + 1)); ++hi) {
      const int j = k + (hi << (S + 1));
      const cplx<R> x = a[j], y = a[j | (1 << S)];
      if constexpr (kInv) {
        const cplx<R> yt = cmulc(y, t);
        a[j] = cadd(x, yt);
        a[j | (1 << S)] = csub(x, yt);
      } else if constexpr (kThenH) {
        const cplx<R> u = cadd(x, y), d = csub(x, y);
        const cplx<R> s0 = {fma(t.re, d.re, fma(-t.im, d.im, u.re)), fma(t.re, d.im, fma(t.im, d.re, u.im))};
        a[j] = s0;
        a[j | (1 << S)] = {fma(R(2), u.re, -s0.re), fma(R(2), u.im, -s0.im)};
      } else {
        a[j] = cadd(x, y);
        a[j | (1 << S)] = cmul(csub(x, y), t);
      }
    }
  }
}

// Twiddle numerator of a stage on bit p of a register whose lowest bit is
// base: the index bits in [base, p).
__device__ __forceinline__ uint32_t stage_low(uint32_t g, int p, int base) {
  return g & ((1u << p) - 1u) & ~((1u << base) - 1u);
}

// ---- straight-line round patterns -------------------------------------------
// Group twiddle of a stage with stage bit p: exp(i pi (g mod 2^p) / 2^p), or the
// square of the previous stage's (bit p + 1 of the same round) when flagged.
template <class R>
__device__ __forceinline__ cplx<R> qft_w(cptr<TileOp> op, uint32_t gglobal, cplx<R> wprev) {
  if (op->square) return cmul(wprev, wprev);
  const int p = op->sbit;
  return cispi<R>(stage_low(gglobal, p, op->base), p);
}

// The four stages of a QFT round; kThenH: each followed by its Hadamard.
template <class R, bool kThenH, bool kSym>
__device__ __forceinline__ void round_qft4(cplx<R>* a, cptr<TileOp> ops, cptr<cplx<R>> coef, uint32_t gglobal) {
  cplx<R> w = qft_w<R>(ops + 0, gglobal, cplx<R>{R(1), R(0)});
  op_qft<3, R, false, kThenH, kSym>(a, w, coef + ops[0].coef);
  w = qft_w<R>(ops + 1, gglobal, w);
  op_qft<2, R, false, kThenH, kSym>(a, w, coef + ops[1].coef);
  w = qft_w<R>(ops + 2, gglobal, w);
  op_qft<1, R, false, kThenH, kSym>(a, w, coef + ops[2].coef);
  w = qft_w<R>(ops + 3, gglobal, w);
  op_qft<0, R, false, kThenH, kSym>(a, w, coef + ops[3].coef);
}

template <class R>
__device__ __forceinline__ void round_h4(cplx<R>* a) {
  op_h<3>(a);
  op_h<2>(a);
  op_h<1>(a);
  op_h<0>(a);
}

template <class R>
__device__ __forceinline__ void round_mat4(cplx<R>* a, cptr<cplx<R>> c) {
  op_mat<0>(a, c);
  op_mat<1>(a, c + 4);
  op_mat<2>(a, c + 8);
  op_mat<3>(a, c + 12);
}

// [[x, -i y], [-i y, x]] with real (x, y) = c: 2 real multiply-adds per output component.
template <int S, class R>
__device__ __forceinline__ void op_rx(cplx<R>* a, cplx<R> c) {
#pragma unroll
  for (int j = 0; j < RN; ++j) {
    if (j & (1 << S)) continue;
    const cplx<R> x = a[j], y = a[j | (1 << S)];
    a[j] = {c.re * x.re + c.im * y.im, c.re * x.im - c.im * y.re};
    a[j | (1 << S)] = {c.re * y.re + c.im * x.im, c.re * y.im - c.im * x.re};
  }
}
// [[x, -y], [y, x]] with real (x, y) = c.
template <int S, class R>
__device__ __forceinline__ void op_ry(cplx<R>* a, cplx<R> c) {
#pragma unroll
  for (int j = 0; j < RN; ++j) {
    if (j & (1 << S)) continue;
    const cplx<R> x = a[j], y = a[j | (1 << S)];
    a[j] = {c.re * x.re - c.im * y.re, c.re * x.im - c.im * y.im};
    a[j | (1 << S)] = {c.im * x.re + c.re * y.re, c.im * x.im + c.re * y.im};
  }
}
// Factored rotations, the common factor applied at the store: [[1, -i t],
// [-i t, 1]] and [[1, -t], [t, 1]], one multiply-add per output component.
template <int S, class R>
__device__ __forceinline__ void op_rxf(cplx<R>* a, R t) {
#pragma unroll
  for (int j = 0; j < RN; ++j) {
    if (j & (1 << S)) continue;
    const cplx<R> x = a[j], y = a[j | (1 << S)];
    a[j] = {fma(t, y.im, x.re), fma(-t, y.re, x.im)};
    a[j | (1 << S)] = {fma(t, x.im, y.re), fma(-t, x.re, y.im)};
  }
}
template <int S, class R>
__device__ __forceinline__ void op_ryf(cplx<R>* a, R t) {
#pragma unroll
  for (int j = 0; j < RN; ++j) {
    if (j & (1 << S)) continue;
    const cplx<R> x = a[j], y = a[j | (1 << S)];
    a[j] = {fma(-t, y.re, x.re), fma(-t, y.im, x.im)};
    a[j | (1 << S)] = {fma(t, x.re, y.re), fma(t, x.im, y.im)};
  }
}

// A general single-qubit round as D2 T D1 (RT_ZYZ4 and its two reduced forms).
template <class R, bool kD1, bool kD2>
struct FZyz4 {
  cptr<cplx<R>> c;  // D1[16] if kD1, then D2[16] if kD2, then t[4] as (t, 0)
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const {
    constexpr int o2 = kD1 ? 16 : 0, ot = o2 + (kD2 ? 16 : 0);
    if constexpr (kD1) {
#pragma unroll
      for (int j = 0; j < RN; ++j) a[j] = cmul(a[j], ldc(c, j));
    }
    op_ryf<0>(a, c[ot + 0].re);
    op_ryf<1>(a, c[ot + 1].re);
    op_ryf<2>(a, c[ot + 2].re);
    op_ryf<3>(a, c[ot + 3].re);
    if constexpr (kD2) {
#pragma unroll
      for (int j = 0; j < RN; ++j) a[j] = cmul(a[j], ldc(c, o2 + j));
    }
  }
};

// ---- round patterns as functors: f(a, g) transforms the 16 registers of the
// group whose smallest index is g (index bits outside the round).
template <class R, bool kThenH4, bool kSym>
struct FQft4 {
  cptr<TileOp> ops;
  cptr<cplx<R>> coef;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t g) const {
    round_qft4<R, kThenH4, kSym>(a, ops, coef, g);
  }
};
template <class R>
struct FH4 {
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const { round_h4<R>(a); }
};
template <class R>
struct FMat4 {
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const { round_mat4<R>(a, c); }
};
template <class R>
struct FRx4 {
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const {
    op_rx<0>(a, ldc(c, 0));
    op_rx<1>(a, ldc(c, 1));
    op_rx<2>(a, ldc(c, 2));
    op_rx<3>(a, ldc(c, 3));
  }
};
template <class R>
struct FRx4F {
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const {
    op_rxf<0>(a, c[0].re);
    op_rxf<1>(a, c[1].re);
    op_rxf<2>(a, c[2].re);
    op_rxf<3>(a, c[3].re);
  }
};
template <class R>
struct FRy4F {
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const {
    op_ryf<0>(a, c[0].re);
    op_ryf<1>(a, c[1].re);
    op_ryf<2>(a, c[2].re);
    op_ryf<3>(a, c[3].re);
  }
};
template <class R>
struct FRy4 {
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const {
    op_ry<0>(a, ldc(c, 0));
    op_ry<1>(a, ldc(c, 1));
    op_ry<2>(a, ldc(c, 2));
    op_ry<3>(a, ldc(c, 3));
  }
};
template <int S, class R>
struct FH1 {
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const { op_h<S>(a); }
};
template <int S, class R>
struct FDiag1 {
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const { op_diag<S>(a, c); }
};
template <int S, class R>
struct FMat1 {
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t) const { op_mat<S>(a, c); }
};
// One QFT stage (stage bit p) on register bit S, optionally followed by the
// Hadamard of the same bit.  A lone stage always evaluates its twiddle.
template <int S, class R, bool kThenH, bool kInv>
struct FQft1 {
  cptr<cplx<R>> E;
  int p, base;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t g) const {
    const cplx<R> w = cispi<R>(stage_low(g, p, base), p);
    op_qft<S, R, kInv, kThenH>(a, w, E);
  }
};

// Any sequence of ops on the round's register bits, one after the other on the
// registers (RT_CHAIN).  A QFT stage and the Hadamard
// of its bit behind it run as one; every stage evaluates its twiddle.
template <class R>
struct FChain {
  cptr<TileOp> ops;
  int n;
  cptr<cplx<R>> coef;
  template <int S>
  __device__ __forceinline__ static void run(cplx<R>* a, int kind, cplx<R> w, cptr<cplx<R>> c) {
    switch (kind) {
      case OP_H: op_h<S>(a); break;
      case OP_DIAG: op_diag<S>(a, c); break;
      case OP_QFT: op_qft<S, R, false>(a, w, c); break;
      case OP_QFT_INV: op_qft<S, R, true>(a, w, c); break;
      case kQftH: op_qft<S, R, false, true>(a, w, c); break;
      default: op_mat<S>(a, c); break;
    }
  }
  static constexpr int kQftH = -1;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t g) const {
#pragma unroll 1
    for (int k = 0; k < n;) {
      const cptr<TileOp> op = ops + k;
      const int rbit = op->rbit;
      int kind = op->kind, step = 1;
      cplx<R> w = {R(1), R(0)};
      if (kind == OP_QFT || kind == OP_QFT_INV) {
        w = cispi<R>(stage_low(g, op->sbit, op->base), op->sbit);
        if (kind == OP_QFT && k + 1 < n && op[1].kind == OP_H && op[1].rbit == rbit) {
          kind = kQftH;
          step = 2;
        }
      }
      const cptr<cplx<R>> c = coef + op->coef;
      switch (rbit & 3) {
        case 0: run<0>(a, kind, w, c); break;
        case 1: run<1>(a, kind, w, c); break;
        case 2: run<2>(a, kind, w, c); break;
        default: run<3>(a, kind, w, c); break;
      }
      k += step;
    }
  }
};

// Diagonal slot d of a pass (uniform): its descriptor read with scalar loads.
__device__ __forceinline__ DiagDev diag_slot(const DiagDev* slots, int d) {
  const cptr<DiagDev> S = to_const(slots) + d;
  DiagDev D;
  D.terms = S->terms;
  D.groups = S->groups;
  D.lut = S->lut;
  D.n_groups = S->n_groups;
  D.conj = S->conj;
  D.theta = S->theta;
  D.global = S->global;
  return D;
}

template <class R>
struct RoundLoop {
  const Ctx& C;
  cptr<TileRound> R_;
  cplx<R>* T;
  uint32_t ngroups, nthr, tid;

  template <class F>
  __device__ __forceinline__ void operator()(const F& f) const {
    const int t0 = R_->tbit[0], t1 = R_->tbit[1], t2 = R_->tbit[2], t3 = R_->tbit[3];
    uint32_t loff[RN];
#pragma unroll
    for (int j = 0; j < RN; ++j) loff[j] = R_->loff[j];
    auto place = [&](uint32_t g) {
      g = insert0(g, t0);
      g = insert0(g, t1);
      g = insert0(g, t2);
      return insert0(g, t3);
    };
    for (uint32_t g = tid; g < ngroups; g += nthr) {
      const uint32_t gpos = place(g);
      cplx<R>* Tg = T + lds_off(gpos);
      cplx<R> a[RN];
#pragma unroll
      for (int j = 0; j < RN; ++j) a[j] = Tg[loff[j]];
      f(a, C.base | C.dep(gpos));
#pragma unroll
      for (int j = 0; j < RN; ++j) Tg[loff[j]] = a[j];
    }
  }
};

// The same loop over two tiles at once (the fused adjoint step's phi and
// lambda): one set of LDS addresses and one barrier per round for both.
template <class R>
struct RoundLoop2 {
  const Ctx& C;
  cptr<TileRound> R_;
  cplx<R>* T;
  cplx<R>* T1;
  uint32_t ngroups, nthr, tid;

  template <class F>
  __device__ __forceinline__ void operator()(const F& f) const {
    const int t0 = R_->tbit[0], t1 = R_->tbit[1], t2 = R_->tbit[2], t3 = R_->tbit[3];
    uint32_t loff[RN];
#pragma unroll
    for (int j = 0; j < RN; ++j) loff[j] = R_->loff[j];
    for (uint32_t g = tid; g < ngroups; g += nthr) {
      uint32_t gpos = insert0(g, t0);
      gpos = insert0(gpos, t1);
      gpos = insert0(gpos, t2);
      gpos = insert0(gpos, t3);
      cplx<R>* Ta = T + lds_off(gpos);
      cplx<R>* Tb = T1 + lds_off(gpos);
      cplx<R> a[RN], b[RN];
#pragma unroll
      for (int j = 0; j < RN; ++j) a[j] = Ta[loff[j]];
#pragma unroll
      for (int j = 0; j < RN; ++j) b[j] = Tb[loff[j]];
      const uint32_t gg = C.base | C.dep(gpos);
      f(a, gg);
      f(b, gg);
#pragma unroll
      for (int j = 0; j < RN; ++j) Ta[loff[j]] = a[j];
#pragma unroll
      for (int j = 0; j < RN; ++j) Tb[loff[j]] = b[j];
    }
  }
};
template <class R, bool kTwo>
struct LoopOf {
  using type = RoundLoop<R>;
  __device__ static type make(const Ctx& C, cptr<TileRound> R_, cplx<R>* T, cplx<R>*, uint32_t ng, uint32_t nt,
                              uint32_t tid) {
    return type{C, R_, T, ng, nt, tid};
  }
};
template <class R>
struct LoopOf<R, true> {
  using type = RoundLoop2<R>;
  __device__ static type make(const Ctx& C, cptr<TileRound> R_, cplx<R>* T, cplx<R>* T1, uint32_t ng, uint32_t nt,
                              uint32_t tid) {
    return type{C, R_, T, T1, ng, nt, tid};
  }
};

// RT_DIAG rounds: register j of the group at index g holds index g | b_j with
// b_j the subset j of the round's state bits b[0..3].
template <class R, bool kConj>
struct FDiagLut {
  DiagDev D;
  cptr<int32_t> qt;
  uint32_t b[4];
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t g) const { diag_lut_round<R, kConj>(a, g, b, D, qt); }
};
template <class R, bool kConj>
struct FDiagPair {
  DiagDev D;
  cptr<int32_t> row;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t g) const { diag_pair_round<R, kConj>(a, g, D, row); }
};
template <class R, bool kConj, bool kFactored>
struct FDiagPairRx4 {
  DiagDev D;
  cptr<int32_t> row;
  cptr<cplx<R>> c;
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t g) const {
    diag_pair_round<R, kConj>(a, g, D, row);
    if constexpr (kFactored) {
      op_rxf<0>(a, c[0].re);
      op_rxf<1>(a, c[1].re);
      op_rxf<2>(a, c[2].re);
      op_rxf<3>(a, c[3].re);
    } else {
      op_rx<0>(a, ldc(c, 0));
      op_rx<1>(a, ldc(c, 1));
      op_rx<2>(a, ldc(c, 2));
      op_rx<3>(a, ldc(c, 3));
    }
  }
};
template <class R>
struct FDiagAngles {
  DiagDev D;
  const cplx<R>* qp;
  uint32_t b[4];
  __device__ __forceinline__ void operator()(cplx<R>* a, uint32_t g) const {
    diag_apply_angles<R>(a, g, b[0], b[1], b[2], b[3], D, qp);
  }
};

// kDiag: the pass carries diagonal layers.  Passes without them use an
// instantiation that has no phase-evaluation code at all, which keeps the
// butterfly rounds' register allocation and schedule tight.
// Coset `coset` of the pass's tile bits: its index bits outside the tile.
template <class R>
__device__ __forceinline__ Ctx coset_ctx(const TileKArgs<R>& A, uint32_t coset) {
  Ctx C;
  C.L = A.L;
  C.a = A.a;
  const uint32_t nlo = A.a - A.L;  // coset bits placed at [L, a)
  const uint32_t top = A.a + A.h;  // first coset bit above the high tile range
  C.base = ((coset & ((1u << nlo) - 1u)) << A.L) | (top >= 32 ? 0u : ((coset >> nlo) << top));
  return C;
}

// kTwo: the rounds run on T and T1 together (RoundLoop2).  kQft: 0 the pass
// has no QFT stages and their code is left out, 1 it has, none in an RT_CHAIN,
// 2 any (rounds of one stage run as chains of one).
template <class R, bool kDiag, bool kTwo = false, int kQft = 2>
__device__ __forceinline__ void tile_rounds(const TileKArgs<R>& A, const Ctx& C, cplx<R>* T, uint32_t nthr,
                                            uint32_t tid, cplx<R>* T1 = nullptr) {
  // threads tid < nthr take the register groups; every thread of the workgroup
  // takes part in the barrier after each round
  const uint32_t M = 1u << A.m;
  // the pattern is uniform per round, so the dispatch sits
  // outside the per-thread group loop and every pattern runs its own loop
  // (registers loaded, transformed and stored with no value crossing a join)
  const uint32_t ngroups = M >> RB;
  const cptr<TileRound> rounds = to_const(A.rounds);
  const cptr<TileOp> ops = to_const(A.ops);
  const cptr<cplx<R>> coef = to_const(A.coef);
  for (uint32_t r = 0; r < A.n_rounds; ++r) {
    const cptr<TileRound> R_ = rounds + r;
    const auto L = LoopOf<R, kTwo>::make(C, R_, T, T1, ngroups, nthr, tid);
    switch (R_->type) {
      case RT_DIAG:
        if constexpr (kDiag) {
          const DiagDev D = diag_slot(A.diag, R_->diag);
          const uint32_t b[4] = {C.dep(1u << R_->tbit[0]), C.dep(1u << R_->tbit[1]), C.dep(1u << R_->tbit[2]),
                                 C.dep(1u << R_->tbit[3])};
          if (R_->qcoef >= 0)
            L(FDiagAngles<R>{D, A.coef + R_->qcoef, {b[0], b[1], b[2], b[3]}});
          else if (D.conj)
            L(FDiagLut<R, true>{D, to_const(A.qtab) + R_->qoff, {b[0], b[1], b[2], b[3]}});
          else
            L(FDiagLut<R, false>{D, to_const(A.qtab) + R_->qoff, {b[0], b[1], b[2], b[3]}});
        }
        break;
      case RT_DIAG_PAIR:
        if constexpr (kDiag) {
          const DiagDev D = diag_slot(A.diag, R_->diag);
          if (D.conj)
            L(FDiagPair<R, true>{D, to_const(A.qtab) + R_->qoff});
          else
            L(FDiagPair<R, false>{D, to_const(A.qtab) + R_->qoff});
        }
        break;
      case RT_DIAG_PAIR_RX:
      case RT_DIAG_PAIR_RXF:
        if constexpr (kDiag) {
          const DiagDev D = diag_slot(A.diag, R_->diag);
          const cptr<int32_t> row = to_const(A.qtab) + R_->qoff;
          const cptr<cplx<R>> c = coef + R_->coef4;
          if (R_->type == RT_DIAG_PAIR_RXF) {
            if (D.conj)
              L(FDiagPairRx4<R, true, true>{D, row, c});
            else
              L(FDiagPairRx4<R, false, true>{D, row, c});
          } else {
            if (D.conj)
              L(FDiagPairRx4<R, true, false>{D, row, c});
            else
              L(FDiagPairRx4<R, false, false>{D, row, c});
          }
        }
        break;
      case RT_QFT4:
        if constexpr (kQft > 0) L(FQft4<R, false, false>{ops + R_->op_begin, coef});
        break;
      case RT_QFT4_H4:
        if constexpr (kQft > 0) L(FQft4<R, true, false>{ops + R_->op_begin, coef});
        break;
      case RT_QFT4S:
        if constexpr (kQft > 0) L(FQft4<R, false, true>{ops + R_->op_begin, coef});
        break;
      case RT_QFT4S_H4:
        if constexpr (kQft > 0) L(FQft4<R, true, true>{ops + R_->op_begin, coef});
        break;
      case RT_H4:
        L(FH4<R>{});
        break;
      case RT_MAT4:
        L(FMat4<R>{coef + R_->coef4});
        break;
      case RT_MAT4_RX:
        L(FRx4<R>{coef + R_->coef4});
        break;
      case RT_MAT4_RY:
        L(FRy4<R>{coef + R_->coef4});
        break;
      case RT_ZYZ4:
        L(FZyz4<R, true, true>{coef + R_->coef4});
        break;
      case RT_YZ4:
        L(FZyz4<R, false, true>{coef + R_->coef4});
        break;
      case RT_ZY4:
        L(FZyz4<R, true, false>{coef + R_->coef4});
        break;
      case RT_MAT4_RXF:
        L(FRx4F<R>{coef + R_->coef4});
        break;
      case RT_MAT4_RYF:
        L(FRy4F<R>{coef + R_->coef4});
        break;
      case RT_OP1: {
        const cptr<TileOp> op = ops + R_->op_begin;
        const cptr<cplx<R>> c = coef + op->coef;
        const int kind = op->kind == OP_H ? 0 : (op->kind == OP_DIAG ? 1 : 2);
        switch (kind * 4 + (op->rbit & 3)) {
          case 0: L(FH1<0, R>{}); break;
          case 1: L(FH1<1, R>{}); break;
          case 2: L(FH1<2, R>{}); break;
          case 3: L(FH1<3, R>{}); break;
          case 4: L(FDiag1<0, R>{c}); break;
          case 5: L(FDiag1<1, R>{c}); break;
          case 6: L(FDiag1<2, R>{c}); break;
          case 7: L(FDiag1<3, R>{c}); break;
          case 8: L(FMat1<0, R>{c}); break;
          case 9: L(FMat1<1, R>{c}); break;
          case 10: L(FMat1<2, R>{c}); break;
          default: L(FMat1<3, R>{c}); break;
        }
        break;
      }
      case RT_QH1:
        if constexpr (kQft == 1) {
          const cptr<TileOp> op = ops + R_->op_begin;
          const cptr<cplx<R>> E = coef + op->coef;
          const int p = op->sbit, base = op->base;
          switch (op->rbit & 3) {
            case 0: L(FQft1<0, R, true, false>{E, p, base}); break;
            case 1: L(FQft1<1, R, true, false>{E, p, base}); break;
            case 2: L(FQft1<2, R, true, false>{E, p, base}); break;
            default: L(FQft1<3, R, true, false>{E, p, base}); break;
          }
          break;
        }
        [[fallthrough]];
      case RT_QFT1:
        if constexpr (kQft == 1) {
          const cptr<TileOp> op = ops + R_->op_begin;
          const cptr<cplx<R>> E = coef + op->coef;
          const int p = op->sbit, base = op->base;
          switch ((op->kind == OP_QFT_INV ? 4 : 0) + (op->rbit & 3)) {
            case 0: L(FQft1<0, R, false, false>{E, p, base}); break;
            case 1: L(FQft1<1, R, false, false>{E, p, base}); break;
            case 2: L(FQft1<2, R, false, false>{E, p, base}); break;
            case 3: L(FQft1<3, R, false, false>{E, p, base}); break;
            case 4: L(FQft1<0, R, false, true>{E, p, base}); break;
            case 5: L(FQft1<1, R, false, true>{E, p, base}); break;
            case 6: L(FQft1<2, R, false, true>{E, p, base}); break;
            default: L(FQft1<3, R, false, true>{E, p, base}); break;
          }
          break;
        }
        [[fallthrough]];
      default:  // RT_CHAIN
        if constexpr (kQft == 2) L(FChain<R>{ops + R_->op_begin, R_->op_end - R_->op_begin, coef});
        break;
    }
    __syncthreads();
  }

}

}  // namespace

}  // namespace qs
