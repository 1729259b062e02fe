// The RNS engine's host tables (csrc/rns_host.hpp) and the steps of its output
// conversion (k_rns_from in csrc/kernels_rns.hip) on the CPU, one element at a
// time, for tests/test_rns_host.py.
#include <cstdint>
#include <cstring>
#include <vector>

#include "../paper_2601_14980_amd/csrc/rns_host.hpp"

using pc2h::Limbs;

extern "C" {

// Tile count of a modulus of `bits` bits.
int sim_tiles(int bits) { return pc2h::rns_tiles(bits); }

// x (nl words, below N) through the residues of base B and back: nw words at
// out, `pad` words of the value `poison` behind the limbs (where the kernel's
// next array stands).  mont: x leaves Montgomery form on the way.  -1: the engine
// does not take N.
int sim_from(const uint32_t* N0, int nn, const uint32_t* x0, int nx, int T, int mont, int nw,
             uint32_t poison, uint32_t* out) {
  const pc2h::RnsBase& R = pc2h::rns_base(T);
  Limbs N(N0, N0 + nn), x(x0, x0 + nx);
  std::vector<uint32_t> E, cst;
  if (!pc2h::rns_e1(R, N, &E, &cst)) return -1;
  const pc2h::RnsFromHost C = pc2h::rns_from(R, N, mont != 0);
  std::vector<int64_t> w(R.n);
  for (int j = 0; j < R.n; ++j)
    w[j] = pc2h::centred((int64_t)pc2h::mod_small(x, R.b[j]) * R.s[j], R.b[j]);
  int64_t s = 0;
  for (int j = 0; j < R.n; ++j) s += w[j] * C.F[j];
  const int64_t beta = (s + ((int64_t)1 << 35)) >> 36;
  const int SB = 8 * C.nblk, pad = nw + 8;
  std::vector<uint32_t> limb(SB + pad, poison);
  std::vector<int64_t> cy(C.nblk);
  for (int k = 0; k < C.nblk; ++k) {
    int64_t carry = 0;
    for (int c = 0; c < 8; ++c) {
      int64_t v = beta * C.D[k * 8 + c] + C.O[k * 8 + c] + carry;
      for (int j = 0; j < R.n; ++j) v += w[j] * (int64_t)C.C[((size_t)k * R.n + j) * 8 + c];
      limb[k * 8 + c] = (uint32_t)v & 0xFFFFFFFu;
      carry = v >> 28;
    }
    cy[k] = carry;
  }
  int64_t carry = 0;
  for (int k = 0; k < C.nblk; ++k) {
    for (int c = 0; c < 8; ++c) {
      const int64_t v = (int64_t)limb[k * 8 + c] + carry;
      limb[k * 8 + c] = (uint32_t)v & 0xFFFFFFFu;
      carry = v >> 28;
    }
    carry += cy[k];
  }
  double top = 0.0;
  for (int i = C.S - 1; i >= C.S - 4 && i >= 0; --i) top = top * 268435456.0 + (double)limb[i];
  const double qd = top * C.ntop_inv - 0.001;
  const int64_t q = qd > 0.0 ? (int64_t)qd : 0;
  auto subtract = [&](int64_t f) {
    int64_t c = 0;
    for (int i = 0; i < C.S; ++i) {
      const int64_t v = (int64_t)limb[i] - f * (int64_t)C.N28[i] + c;
      limb[i] = (uint32_t)v & 0xFFFFFFFu;
      c = v >> 28;
    }
  };
  subtract(q);
  int c = 0;
  for (int i = C.S - 1; i >= 0 && c == 0; --i)
    if (limb[i] != C.N28[i]) c = limb[i] > C.N28[i] ? 1 : -1;
  if (c >= 0) subtract(1);
  for (int j = 0; j < nw; ++j) out[j] = pc2k::rns_word28(limb.data(), SB, 1, j);
  return 0;
}

// Whether the bounds on 32-bit sums hold for tile count T with mt tiles a wavefront
// (0: the compiled ones).
int sim_bounds(int T, int mt) { return pc2h::make_rns_base(T, mt ? mt : pc2k::rns_mt(T)).ok; }

// The digits of a block of a constant (RnsDigits): for each its shift, width, and the
// table entries of its values 1 and 2^width - 1; returns the entries of a column.
int sim_digits(int ebits, int n, int nblk, int32_t* out) {
  const pc2k::RnsDigits d = pc2k::RnsDigits::of(ebits, n, nblk);
  for (int t = 0; t < n; ++t) {
    out[4 * t] = d.shift(t);
    out[4 * t + 1] = d.width(t);
    out[4 * t + 2] = (int32_t)(d.before(t) + 1);
    out[4 * t + 3] = (int32_t)(d.before(t) + ((1u << d.width(t)) - 1));
  }
  return (int)d.entries();
}

// MA of a tile count (its words; returns how many)
int sim_ma(int T, uint32_t* out) {
  const Limbs& m = pc2h::rns_base(T).MA;
  std::memcpy(out, m.data(), m.size() * 4);
  return (int)m.size();
}
}
