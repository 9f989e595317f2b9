// Expectations of Pauli sums: terms sorted into tile sets that share a read of
// the state (k_expect.hip); X masks of more than four bits, states of fewer than
// four qubits, and a few terms of one mask take one reduction per mask.
#include <algorithm>
#include <cmath>
#include <map>

#include "runtime.h"

namespace qs {

namespace {

struct Term {
  uint32_t x, z;  // state bits
  int ny;         // Y factors mod 4
  size_t index;   // in the caller's list
};

// Terms of one X mask (and one parity of Y factors) that share their products.
struct Piece {
  uint32_t x;
  bool imag;
  std::vector<const Term*> terms;
};

struct TileSet {
  uint32_t bits = 0;
  std::vector<const Piece*> pieces;
  size_t n_slots = 0;
  static size_t slots(const Piece& p) { return (p.terms.size() + 3) & ~size_t(3); }
  bool room(const Piece& p) const {
    return pieces.size() < kExpectMaxGroups && n_slots + slots(p) <= kExpectMaxTerms;
  }
  void add(const Piece& p) {
    pieces.push_back(&p);
    n_slots += slots(p);
    bits |= p.x;
  }
};

constexpr int kLowBits = 5;            // contiguous low bits of every tile: runs of 32 amplitudes
constexpr uint32_t kBlocks = 1024;     // resident workgroups (four per compute unit)
constexpr size_t kZPieceTerms = 64;    // Z-type terms per window; eight where windows are spread over workgroups

uint32_t bits_of(int k) { return k >= 32 ? 0xffffffffu : (1u << k) - 1u; }

// First fit in order of the X masks: neighbouring bonds share a set.
std::vector<TileSet> make_sets(int n, uint32_t m, const std::vector<Piece>& pieces) {
  std::vector<TileSet> sets;
  std::vector<char> taken(pieces.size(), 0);
  size_t left = pieces.size();
  while (left) {
    TileSet S;
    S.bits = bits_of(std::min(n, kLowBits));
    for (size_t k = 0; k < pieces.size(); ++k) {
      if (taken[k] || !S.room(pieces[k]) || (uint32_t)__builtin_popcount(S.bits | pieces[k].x) > m) continue;
      S.add(pieces[k]);
      taken[k] = 1;
      --left;
    }
    for (int b = 0; b < n && (uint32_t)__builtin_popcount(S.bits) < m; ++b) S.bits |= 1u << b;
    sets.push_back(std::move(S));
  }
  return sets;
}

// Kernel arguments of a set; order receives the set's terms in kernel order
// (null where a window's last slots stay free).
template <class R>
ExpectArgs<R> set_args(int n, const TileSet& S, std::vector<const Term*>& order) {
  ExpectArgs<R> A{};
  A.m = (uint32_t)__builtin_popcount(S.bits);
  A.L = 0;
  while (A.L < A.m && ((S.bits >> A.L) & 1u)) ++A.L;
  uint32_t pos[32] = {0}, tile_bit[32] = {0}, p = 0;
  for (int b = 0; b < n; ++b) {
    if ((S.bits >> b) & 1u) {
      if (p >= A.L) A.hi_bit[p - A.L] = (uint8_t)b;
      tile_bit[p] = (uint32_t)b;
      pos[b] = p++;
    } else {
      A.free_bit[A.n_free++] = (uint8_t)b;
    }
  }
  A.n_tiles = 1u << A.n_free;
  for (uint32_t k = 0; k < 8; ++k)
    for (uint32_t j = 0; j < 3; ++j)
      if ((k >> j) & 1u) A.load_off[k] |= 1u << tile_bit[A.m - 3 + j];
  uint32_t ng = 0, nt = 0;
  for (size_t k0 = 0; k0 < S.pieces.size();) {
    // a window: consecutive pieces whose X masks cover at most four bits; a
    // Z-type piece has its own
    uint32_t w = S.pieces[k0]->x;
    size_t k1 = k0 + 1;
    while (w != 0 && k1 < S.pieces.size() && S.pieces[k1]->x != 0 && __builtin_popcount(w | S.pieces[k1]->x) <= 4)
      w |= S.pieces[k1++]->x;
    for (uint32_t q = A.m; q-- > 0 && __builtin_popcount(w) < 4;) w |= 1u << tile_bit[q];
    ExpectWindow& W = A.win[A.n_win++];
    uint32_t wb[4], c = 0;
    for (int b = 0; b < n; ++b)
      if ((w >> b) & 1u) {
        W.bits |= pos[b] << (8 * c);
        wb[c++] = (uint32_t)b;
      }
    W.g0 = ng;
    for (size_t k = k0; k < k1; ++k) {
      const Piece& P = *S.pieces[k];
      ExpectGroup& G = A.grp[ng++];
      for (uint32_t j = 0; j < 4; ++j) G.x |= ((P.x >> wb[j]) & 1u) << j;
      G.imag = P.imag;
      G.t0 = nt;
      const uint32_t top = G.x ? 31u - (uint32_t)__builtin_clz(G.x) : 4u;
      std::vector<std::pair<uint32_t, const Term*>> by_zw;
      for (const Term* t : P.terms) {
        uint32_t zw = 0;
        for (uint32_t j = 0, o = 0; j < 4; ++j)
          if (j != top) zw |= ((t->z >> wb[j]) & 1u) << o++;
        by_zw.push_back({zw, t});
      }
      std::stable_sort(by_zw.begin(), by_zw.end(), [](const auto& a, const auto& b) { return a.first < b.first; });
      for (const auto& e : by_zw) {
        A.term[nt++] = {e.second->z, e.first};
        order.push_back(e.second);
      }
      G.t1 = nt;
    }
    W.g1 = ng;
    for (; nt & 3u; ++nt) order.push_back(nullptr);
    k0 = k1;
  }
  A.n_terms = nt;
  return A;
}

// One reduction per X mask, eight terms at a time.
void expect_by_mask(qs_state& s, const std::vector<Term>& terms, std::vector<double>& out) {
  s.ensure_red();
  for (size_t t0 = 0; t0 < terms.size();) {
    size_t t1 = t0 + 1;
    while (t1 < terms.size() && t1 - t0 < (size_t)kMaxTermsPerLaunch && terms[t1].x == terms[t0].x) ++t1;
    const int nt = (int)(t1 - t0);
    uint32_t zz[kMaxTermsPerLaunch];
    int yy[kMaxTermsPerLaunch];
    for (int k = 0; k < nt; ++k) {
      zz[k] = terms[t0 + k].z;
      yy[k] = terms[t0 + k].ny;
    }
    const uint32_t x = terms[t0].x;
    if (x == 0) {
      if (s.dtype == QS_C64)
        launch_expect_z<float>((const cplx<float>*)s.cur_ptr(), s.n, zz, nt, s.red_partials, s.red_out, s.stream);
      else
        launch_expect_z<double>((const cplx<double>*)s.cur_ptr(), s.n, zz, nt, s.red_partials, s.red_out, s.stream);
    } else {
      if (s.dtype == QS_C64)
        launch_expect_x<float>((const cplx<float>*)s.cur_ptr(), s.n, x, zz, yy, nt, s.red_partials, s.red_out,
                               s.stream);
      else
        launch_expect_x<double>((const cplx<double>*)s.cur_ptr(), s.n, x, zz, yy, nt, s.red_partials, s.red_out,
                                s.stream);
    }
    double o[kMaxTermsPerLaunch];
    check_hip(hipMemcpyAsync(o, s.red_out, sizeof o, hipMemcpyDeviceToHost, s.stream), "hipMemcpyAsync");
    s.sync();
    for (int k = 0; k < nt; ++k) out[terms[t0 + k].index] = o[k];
    t0 = t1;
  }
}

template <class R>
void expect_tiled(qs_state& s, const std::vector<Term>& terms, std::vector<double>& out) {
  const int n = s.n;
  const uint32_t m = std::min<uint32_t>((uint32_t)n, expect_tile_bits(sizeof(R) == 8));
  const uint32_t n_tiles = 1u << (n - m);
  const size_t zmax = n_tiles < kBlocks ? (size_t)8 : kZPieceTerms;
  std::vector<Piece> pieces;
  for (const Term& t : terms) {  // sorted by (x, imaginary)
    const bool imag = (t.ny & 1) != 0;
    if (pieces.empty() || pieces.back().x != t.x || pieces.back().imag != imag ||
        pieces.back().terms.size() >= (t.x ? kZPieceTerms : zmax))
      pieces.push_back({t.x, imag, {}});
    pieces.back().terms.push_back(&t);
  }
  const std::vector<TileSet> sets = make_sets(n, m, pieces);
  for (size_t s0 = 0, ns = 0; s0 < sets.size(); s0 += ns) {
    ExpectFold F{};
    std::vector<ExpectArgs<R>> args;
    std::vector<const Term*> order;
    uint64_t doubles = 0;
    // as many sets as one launch folds and the kept scratch holds (a set's partials
    // are 4 MiB at most)
    for (ns = 0; ns < kExpectMaxSets && s0 + ns < sets.size(); ++ns) {
      const size_t terms_before = order.size();
      ExpectArgs<R> A = set_args<R>(n, sets[s0 + ns], order);
      const uint32_t nb = std::min(A.n_tiles, kBlocks);
      A.wsplit = std::min(A.n_win, kBlocks / nb);
      const uint64_t add = 2ull * nb * A.wsplit * A.n_terms;
      if (ns && (order.size() + doubles + add) * sizeof(double) > kKeptScratch) {
        order.resize(terms_before);
        break;
      }
      F.n_terms[ns] = A.n_terms;
      F.n_blocks[ns] = nb * A.wsplit;
      F.off[ns] = doubles;
      doubles += add;
      args.push_back(A);
    }
    F.n_sets = (uint32_t)ns;
    double* buf = nullptr;
    try {
      buf = (double*)s.ensure_scratch((order.size() + doubles) * sizeof(double));
    } catch (const Error&) {
      // a device without room for it: the reductions need next to none
      (void)hipGetLastError();
      std::vector<Term> left;
      for (size_t k = s0; k < sets.size(); ++k)
        for (const Piece* p : sets[k].pieces)
          for (const Term* t : p->terms) left.push_back(*t);
      std::stable_sort(left.begin(), left.end(), [](const Term& a, const Term& b) { return a.x < b.x; });
      expect_by_mask(s, left, out);
      return;
    }
    F.partials = buf + order.size();
    for (size_t k = 0; k < ns; ++k) {
      args[k].psi = (const cplx<R>*)s.cur_ptr();
      args[k].partials = buf + order.size() + F.off[k];
      launch_expect_tiles<R>(args[k], F.n_blocks[k], s.stream);
    }
    launch_expect_fold(F, buf, s.stream);
    std::vector<double> r(order.size());
    check_hip(hipMemcpyAsync(r.data(), buf, r.size() * sizeof(double), hipMemcpyDeviceToHost, s.stream),
              "hipMemcpyAsync");
    s.sync();
    for (size_t k = 0; k < order.size(); ++k) {
      if (!order[k]) continue;
      // both indices of a pair contribute alike; i^ny's sign for two or three Y factors
      const double f = order[k]->x == 0 ? 1.0 : (order[k]->ny >= 2 ? -2.0 : 2.0);
      out[order[k]->index] = f * r[k];
    }
  }
}

}  // namespace

std::vector<double> state_expect(qs_state& s, const qs_pauli* terms, size_t n_terms) {
  const int n = s.n;
  std::vector<double> out(n_terms, 0.0);
  std::vector<Term> tiled, rest;
  for (size_t t = 0; t < n_terms; ++t) {
    const qs_pauli& P = terms[t];
    if (!std::isfinite(P.coeff)) fail(QS_EINVAL, "non-finite Pauli coefficient");
    if (n < 64 && ((P.x_mask >> n) || (P.z_mask >> n))) fail(QS_EINVAL, "Pauli mask out of range");
    Term T{0, 0, 0, t};
    for (int q = 0; q < n; ++q) {
      if ((P.x_mask >> q) & 1) T.x |= 1u << (n - 1 - q);
      if ((P.z_mask >> q) & 1) T.z |= 1u << (n - 1 - q);
    }
    T.ny = __builtin_popcount(T.x & T.z) & 3;
    (n >= 4 && __builtin_popcount(T.x) <= 4 ? tiled : rest).push_back(T);
  }
  std::stable_sort(tiled.begin(), tiled.end(), [](const Term& a, const Term& b) {
    return a.x != b.x ? a.x < b.x : (a.ny & 1) < (b.ny & 1);
  });
  // A few terms of one X mask are one reduction, whose single read of a large state
  // is faster than the tiles' (one term in us, reduction and tiles: complex64 23
  // qubits 41 and 44, 25 68 and 74; complex128 24 67 and 71, 26 199 and 267), until
  // its sums term by term cost more (complex64, 24 qubits: two Z-type terms 51 and
  // 54, three 55 and 55, two of an X mask 54 and 55; complex128, 26 qubits: eight
  // Z-type 238 and 276, four of an X mask 210 and 271, eight 297 and 275).  Below 64
  // MiB both wait for their launches.
  if (!tiled.empty() && s.state_bytes() >= (64u << 20) && tiled.front().x == tiled.back().x) {
    const size_t few = s.dtype == QS_C64 ? (tiled.front().x ? 1 : 2) : (tiled.front().x ? 4 : 8);
    if (tiled.size() <= few) {
      rest.insert(rest.end(), tiled.begin(), tiled.end());
      tiled.clear();
    }
  }
  std::stable_sort(rest.begin(), rest.end(), [](const Term& a, const Term& b) { return a.x < b.x; });
  if (!tiled.empty()) {
    if (s.dtype == QS_C64) expect_tiled<float>(s, tiled, out);
    else expect_tiled<double>(s, tiled, out);
  }
  if (!rest.empty()) expect_by_mask(s, rest, out);
  for (size_t t = 0; t < n_terms; ++t) out[t] *= terms[t].coeff;
  return out;
}

}  // namespace qs
