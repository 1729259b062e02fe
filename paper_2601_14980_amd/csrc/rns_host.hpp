// Host-side constants of the RNS engine (rns_mont.hpp): the channel moduli and
// everything that depends on them alone, once per tile count, and a modulus'
// own matrices and conversion tables, once per key.
#pragma once
#include <array>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <vector>

#include "host_bn.hpp"
#include "rns_types.hpp"

namespace pc2h {

inline uint32_t mod_small(const Limbs& x, uint32_t m) {
  uint64_t r = 0;
  for (size_t i = x.size(); i-- > 0;) r = ((r << 32) | x[i]) % m;
  return (uint32_t)r;
}
inline Limbs div_small(const Limbs& x, uint32_t m) {  // exact or floor
  Limbs q(x.size(), 0);
  uint64_t r = 0;
  for (size_t i = x.size(); i-- > 0;) {
    r = (r << 32) | x[i];
    q[i] = (uint32_t)(r / m);
    r %= m;
  }
  trim(q);
  return q;
}
inline Limbs mul_small(const Limbs& x, uint32_t m) {
  Limbs r(x.size() + 1, 0);
  uint64_t c = 0;
  for (size_t i = 0; i < x.size(); ++i) {
    c += (uint64_t)x[i] * m;
    r[i] = (uint32_t)c;
    c >>= 32;
  }
  r[x.size()] = (uint32_t)c;
  return r;
}
inline uint32_t inv_small(uint32_t a, uint32_t m) {  // a^-1 mod m, 0 if not invertible
  int64_t r0 = m, r1 = a % m, t0 = 0, t1 = 1;
  while (r1) {
    const int64_t q = r0 / r1;
    int64_t t = r0 - q * r1;
    r0 = r1;
    r1 = t;
    t = t0 - q * t1;
    t0 = t1;
    t1 = t;
  }
  if (r0 != 1) return 0;
  return (uint32_t)(t0 < 0 ? t0 + m : t0);
}

// Residues modulo a channel's m of |v| < 2^50: in [0, m), and centred in
// (-m/2, m/2].  The quotient in double is exact to +-1; a key's tables take some
// 10^5 of these, which the division instruction made half of its creation.
struct Mod {
  int64_t m;
  double inv;
  explicit Mod(uint32_t m_) : m(m_), inv(1.0 / (double)m_) {}
  uint32_t operator()(int64_t v) const {
    int64_t r = v - m * (int64_t)((double)v * inv);
    r += r < 0 ? m : 0;
    r -= r >= m ? m : 0;
    return (uint32_t)r;
  }
  int32_t centred(int64_t v) const {
    const int64_t r = (*this)(v);
    return (int32_t)(2 * r > m ? r - m : r);
  }
};
inline int32_t centred(int64_t v, uint32_t m) { return Mod(m).centred(v); }

// largest prime allowed per tile count: small enough for the bounds on the
// 32-bit sums, large enough that 16 T of them hold the modulus and 2^30
inline uint32_t rns_top(int T) {
  return T >= 34 ? 49000 : T >= 26 ? 38500 : T >= 17 ? 46341 : T >= 13 ? 36000 : 32768;
}

// What depends on the tile count alone.
struct RnsBase {
  int T = 0, n = 0;
  std::vector<uint32_t> a, b;      // channel moduli
  Limbs MA, MB;
  std::vector<uint32_t> s;         // MA^-1 mod b_j
  std::vector<uint32_t> iMAi;      // (MA / a_i)^-1 mod a_i
  std::vector<uint32_t> ia;        // [j][i] a_i^-1 mod b_j
  std::vector<int32_t> g;          // MA (MB / b_j)^-1 mod b_j, centred
  std::vector<uint32_t> E2;        // fragments (T T 256 words)
  std::vector<uint32_t> c2, kb, ka;
  bool ok = false;
};

// E[row channel][column channel] (centred mod m_row) -> fragments, initial sums
// (128 sum_i E) and the check of the bounds: |sum| + extra_row < 2^31 for all
// inputs with |r_col| < 0.52 m_col + 128.
inline bool rns_pack(const std::vector<int32_t>& E, const std::vector<uint32_t>& mrow,
                     const std::vector<uint32_t>& mcol, bool square, std::vector<uint32_t>* frag,
                     std::vector<uint32_t>* cst) {
  const int n = (int)mrow.size(), T = n / 16;
  frag->assign((size_t)T * T * 256, 0);
  cst->assign((size_t)T * 16, 0);
  uint8_t* out = reinterpret_cast<uint8_t*>(frag->data());
  bool ok = true;
  for (int j = 0; j < n; ++j) {
    const int t = j / 16, H = (j >> 3) & 1, u = j & 7;
    int64_t sum = 0, bound = 0;
    const Mod M(mrow[j]);
    for (int i = 0; i < n; ++i) {
      const int32_t e = E[(size_t)j * n + i];
      const int32_t f = M.centred((int64_t)e * 256);
      sum += e;
      const int64_t hmax = (int64_t)((0.52 * mcol[i] + 128) / 256) + 1;
      bound += 128 * (int64_t)std::abs(e) + hmax * std::abs(f);
      const int c = i / 16, Hk = (i >> 3) & 1, s0 = 2 * (i & 7);
      for (int k = 0; k < 2; ++k) {
        const int32_t v = k ? f : e;
        const int32_t lo = (int32_t)(int8_t)(v & 255), hi = (v - lo) >> 8;
        if (hi < -128 || hi > 127) ok = false;
        for (int part = 0; part < 2; ++part) {
          const int r = 2 * u + part, rho = 8 * (r >> 2) + 4 * H + (r & 3);
          out[(((size_t)t * T + c) * 64 + 32 * Hk + rho) * 16 + s0 + k] =
              (uint8_t)(part ? hi : lo);
        }
      }
    }
    const int32_t c0 = centred(128 * sum, mrow[j]);
    (*cst)[(size_t)(t * 2 + H) * 8 + u] = (uint32_t)c0;
    const double sq = 0.52 * mrow[j];
    const double extra = square ? sq * sq : (double)(1 << 27);
    if ((double)bound + std::abs(c0) + extra + (1 << 24) >= 2147483648.0) ok = false;
  }
  return ok;
}

inline uint32_t float_bits(float f) {
  uint32_t u;
  static_assert(sizeof(u) == sizeof(f), "");
  __builtin_memcpy(&u, &f, 4);
  return u;
}
inline uint32_t pair16(int32_t lo, int32_t hi) {
  return ((uint32_t)lo & 0xFFFFu) | ((uint32_t)hi << 16);
}

// mt: tiles a wavefront owns, at most
inline RnsBase make_rns_base(int T, int mt) {
  RnsBase R;
  R.T = T;
  const int n = R.n = 16 * T;
  std::vector<uint32_t> ps;
  for (uint32_t x = rns_top(T) | 1; (int)ps.size() < 2 * n; x -= 2) {
    if (x >= rns_top(T)) continue;
    bool prime = true;
    for (uint32_t d = 3; d * d <= x && prime; d += 2) prime = x % d != 0;
    if (prime) ps.push_back(x);
  }
  R.a.assign(ps.begin(), ps.begin() + n);
  R.b.assign(ps.begin() + n, ps.end());
  R.MA = R.MB = Limbs{1};
  for (int i = 0; i < n; ++i) {
    R.MA = mul_small(R.MA, R.a[i]);
    R.MB = mul_small(R.MB, R.b[i]);
  }
  trim(R.MA);
  trim(R.MB);
  // products of a base's other moduli, and of the other base, per channel
  auto prod_mod = [](const std::vector<uint32_t>& v, uint32_t m, int skip) {
    const Mod M(m);
    uint32_t r = 1;
    for (int i = 0; i < (int)v.size(); ++i)
      if (i != skip) r = M((int64_t)r * v[i]);
    return r;
  };
  R.s.resize(n);
  R.iMAi.resize(n);
  R.g.resize(n);
  R.ia.resize((size_t)n * n);
  std::vector<uint32_t> pre(n + 1);
  for (int i = 0; i < n; ++i) R.iMAi[i] = inv_small(prod_mod(R.a, R.a[i], i), R.a[i]);
  for (int j = 0; j < n; ++j) {
    const uint32_t m = R.b[j];
    const Mod M(m);
    pre[0] = 1;
    for (int i = 0; i < n; ++i) pre[i + 1] = M((int64_t)pre[i] * R.a[i]);
    R.s[j] = inv_small(pre[n], m);
    uint32_t run = R.s[j];
    for (int i = n; i-- > 0;) {  // inverse of every a_i from one inverse of their product
      R.ia[(size_t)j * n + i] = M((int64_t)run * pre[i]);
      run = M((int64_t)run * R.a[i]);
    }
    R.g[j] = centred((int64_t)((uint64_t)pre[n] * inv_small(prod_mod(R.b, m, j), m) % m), m);
  }
  std::vector<int32_t> E2((size_t)n * n);
  for (int i = 0; i < n; ++i) {
    const uint32_t m = R.a[i];
    const Mod M(m);
    std::vector<uint32_t> suf(n + 1);
    suf[n] = 1;
    for (int j = n; j-- > 0;) suf[j] = M((int64_t)suf[j + 1] * R.b[j]);
    uint32_t p = 1;
    for (int j = 0; j < n; ++j) {
      E2[(size_t)i * n + j] = M.centred((int64_t)M((int64_t)p * suf[j + 1]) * R.g[j]);
      p = M((int64_t)p * R.b[j]);
    }
  }
  R.ok = rns_pack(E2, R.a, R.b, false, &R.E2, &R.c2);
  R.kb.assign((size_t)T * 48, 0);
  R.ka.assign((size_t)T * 48, 0);
  for (int c = 0; c < n; ++c) {
    const size_t at = (size_t)(c / 8) * 24;
    const int u = c & 7;
    R.kb[at + u] = float_bits(1.0f / (float)R.b[c]);
    R.kb[at + 8 + u] = 0u - R.b[c];
    R.ka[at + u] = float_bits(1.0f / (float)R.a[c]);
    R.ka[at + 8 + u] = 0u - R.a[c];
    // beta = lo + 4096 hi: -MB and -4096 MB mod a_i
    const uint32_t mb = mod_small(R.MB, R.a[c]);
    R.ka[at + 16 + u] = pair16(centred(-(int64_t)mb, R.a[c]), centred(-4096ll * mb, R.a[c]));
    if (R.a[c] >= 60000 || R.b[c] >= 60000) R.ok = false;
  }
  std::vector<std::array<double, 2>> beta(2 * T, {0.0, 0.0});  // by tile half
  for (int c = 0; c < n; c += 2) {  // g_j / b_j = F1 2^-12 + F2 2^-25
    int32_t f1[2], f2[2];
    for (int k = 0; k < 2; ++k) {
      const double x = (double)R.g[c + k] / (double)R.b[c + k];
      f1[k] = (int32_t)std::nearbyint(x * 4096.0);
      f2[k] = (int32_t)std::nearbyint((x - f1[k] / 4096.0) * 33554432.0);
    }
    const size_t at = (size_t)(c / 8) * 24;
    const int u = (c & 7) / 2;
    R.kb[at + 16 + u] = pair16(f1[0], f1[1]);
    R.kb[at + 20 + u] = pair16(f2[0], f2[1]);
    for (int k = 0; k < 2; ++k) {
      // a lane's part of beta (s1, s2 of finish_b): its half of mt tiles, |w| < 0.52 b
      const double z = 0.52 * R.b[c + k];
      beta[c / 8][0] += z * std::abs(f1[k]);
      beta[c / 8][1] += z * std::abs(f2[k]);
    }
  }
  for (int h = 0; h < 2; ++h)
    for (int t = 0; t + mt <= T; ++t)
      for (int i = 0; i < 2; ++i) {
        double sum = 0;
        for (int m = 0; m < mt; ++m) sum += beta[2 * (t + m) + h][i];
        if (sum >= 2147483648.0) R.ok = false;
      }
  return R;
}

// The tables of a tile count, made once per process.
inline const RnsBase& rns_base(int T) {
  static std::once_flag once[64];
  static RnsBase* made[64];
  std::call_once(once[T], [T] { made[T] = new RnsBase(make_rns_base(T, pc2k::rns_mt(T))); });
  return *made[T];
}

// Smallest compiled tile count whose bases hold a modulus of `bits` bits with
// 2^30 to spare, or 0.
inline int rns_tiles(int bits) {
  for (int T : pc2k::RNS_T) {
    if (256 * T < bits) continue;  // 16 T channels of less than 16 bits
    const RnsBase& R = rns_base(T);
    if (R.ok && bitlen(R.MA) > bits + 31 && bitlen(R.MB) > bits + 31) return T;
  }
  return 0;
}

// The first extension's matrix of modulus N; false if N shares a factor with
// a channel modulus or a bound does not hold.
inline bool rns_e1(const RnsBase& R, const Limbs& N, std::vector<uint32_t>* frag,
                   std::vector<uint32_t>* cst) {
  const int n = R.n;
  std::vector<int32_t> E((size_t)n * n);
  std::vector<int64_t> ki(n);  // centred, as q's bound wants
  for (int i = 0; i < n; ++i) {
    const uint32_t a = R.a[i], inv = inv_small(mod_small(N, a), a);
    if (!inv) return false;
    ki[i] = centred((int64_t)(a - inv) * R.iMAi[i], a);
  }
  for (int j = 0; j < n; ++j) {
    const uint32_t m = R.b[j];
    const uint64_t Nj = mod_small(N, m);
    if (!Nj) return false;
    const Mod M(m);
    const int64_t f = M((int64_t)(Nj * R.s[j]));
    for (int i = 0; i < n; ++i) {
      E[(size_t)j * n + i] = M.centred(ki[i] * M.centred(f * R.ia[(size_t)j * n + i]));
    }
  }
  return rns_pack(E, R.b, R.a, true, frag, cst);
}

// Input conversion by the constant f (RnsTo): V_(2 i) = 2^(16 i) f mod N for
// each of nhalf 16-bit halves, V_(2 i + 1) = 256 V_(2 i), so that the value is
// below 2^16 nhalf N; add_one: plus 1.
struct RnsToHost {
  std::vector<uint32_t> E, cst;
  int nchunk = 0;
};
inline RnsToHost rns_to(const RnsBase& R, const Limbs& N0, const Limbs& f, int nhalf,
                        bool add_one) {
  RnsToHost o;
  Limbs N = N0;
  trim(N);
  const int n = R.n, T = R.T, KC = o.nchunk = (nhalf + 15) / 16;
  o.E.assign((size_t)2 * T * KC * 256, 0);
  o.cst.assign((size_t)(KC + 1) * 2 * n, 0);
  uint8_t* E = reinterpret_cast<uint8_t*>(o.E.data());
  std::vector<uint32_t> r(2 * n), Nm(2 * n), sc(2 * n), x(2 * n);
  std::vector<int64_t> sum(2 * n, 0);
  std::vector<Mod> Ms;
  for (int c = 0; c < 2 * n; ++c) Ms.emplace_back(c < n ? R.b[c] : R.a[c - n]);  // base B first
  Limbs v = mod(f, N);
  for (int c = 0; c < 2 * n; ++c) {
    r[c] = mod_small(v, (uint32_t)Ms[c].m);
    Nm[c] = mod_small(N, (uint32_t)Ms[c].m);
    sc[c] = c < n ? R.s[c] : 1u;
  }
  auto constants = [&](int chunks) {
    for (int c = 0; c < 2 * n; ++c)
      o.cst[(size_t)chunks * 2 * n + c] =
          (uint32_t)Ms[c].centred(128 * sum[c] + (add_one ? (int64_t)sc[c] : 0));
  };
  constants(0);
  const size_t nl = N.size();
  const double Ntop = (double)N[nl - 1] * 4294967296.0 + (nl > 1 ? N[nl - 2] : 0);
  for (int i = 0; i < nhalf; ++i) {
    for (int c = 0; c < 2 * n; ++c) x[c] = Ms[c]((int64_t)r[c] * sc[c]);
    for (int c = 0; c < 2 * n; ++c) {
      const int row = c >> 4, u = c & 7, H = (c >> 3) & 1;
      for (int k = 0; k < 2; ++k) {
        const int32_t e = Ms[c].centred((int64_t)x[c] << (8 * k));
        const int32_t lo = (int32_t)(int8_t)(e & 255), hi = (e - lo) >> 8;
        sum[c] += e;
        const int at = 2 * i + k;  // input byte
        for (int part = 0; part < 2; ++part) {
          const int q = 2 * u + part, rho = 8 * (q >> 2) + 4 * H + (q & 3);
          E[(((size_t)row * KC + at / 32) * 64 + 32 * ((at >> 4) & 1) + rho) * 16 + (at & 15)] =
              (uint8_t)(part ? hi : lo);
        }
      }
    }
    if (i % 16 == 15 || i + 1 == nhalf) constants(i / 16 + 1);
    if (i + 1 == nhalf) break;
    // v <- 2^16 v mod N, on the limbs and on the residues
    Limbs w(nl + 1, 0);
    for (size_t l = 0; l < nl; ++l) {
      w[l] |= v[l] << 16;
      w[l + 1] |= v[l] >> 16;
    }
    const double wtop = ((double)w[nl] * 4294967296.0 + w[nl - 1]) * 4294967296.0 +
                        (nl > 1 ? w[nl - 2] : 0);
    int64_t q = (int64_t)(wtop / Ntop);
    Limbs qn = resized(mul_small(N, (uint32_t)q), nl + 1);
    if (cmp(qn, w) > 0) {
      --q;
      qn = resized(mul_small(N, (uint32_t)q), nl + 1);
    }
    w = sub(w, qn);
    if (cmp(w, N) >= 0) {
      ++q;
      w = sub(w, N);
    }
    v = resized(w, nl);
    for (int c = 0; c < 2 * n; ++c) r[c] = Ms[c]((int64_t)r[c] * 65536 - q * (int64_t)Nm[c]);
  }
  return o;
}

// v mod N as one entry: 16-bit residues by base B's channels (times s_j), then
// base A's, centred.
inline std::vector<uint32_t> rns_entry(const RnsBase& R, const Limbs& N, const Limbs& v0) {
  const Limbs v = mod(v0, N);
  std::vector<uint32_t> o;
  for (int p = 0; p < 2; ++p)
    for (int c = 0; c < R.n; c += 2) {
      int32_t r[2];
      for (int k = 0; k < 2; ++k) {
        const uint32_t m = p ? R.a[c + k] : R.b[c + k];
        r[k] = centred((int64_t)mod_small(v, m) * (p ? 1 : R.s[c + k]), m);
      }
      o.push_back(pair16(r[0], r[1]));
    }
  return o;
}

// Output conversion; mont: of values in Montgomery form (divides by MA).
struct RnsFromHost {
  std::vector<uint32_t> C, D, O, N28;
  std::vector<int64_t> F;
  int S = 0, nblk = 0;
  double ntop_inv = 0;
};
inline std::vector<uint32_t> limbs28(const Limbs& v, int S) {
  std::vector<uint32_t> out(S, 0);
  for (int i = 0; i < S; ++i) {
    const long bit = 28l * i;
    const size_t w = bit / 32;
    const uint64_t lo = w < v.size() ? v[w] : 0, hi = w + 1 < v.size() ? v[w + 1] : 0;
    out[i] = (uint32_t)(((hi << 32) | lo) >> (bit % 32)) & ((1u << 28) - 1u);
  }
  return out;
}
inline RnsFromHost rns_from(const RnsBase& R, const Limbs& N0, bool mont) {
  RnsFromHost o;
  Limbs N = N0;
  trim(N);
  const int n = R.n;
  o.S = (bitlen(N) + 27 + 27) / 28;
  o.nblk = (o.S + 7) / 8;
  const int SB = 8 * o.nblk;
  // x / a mod N, exactly divided after adding the multiple of N that makes it
  // divisible
  auto div_mod = [&](const Limbs& x, uint32_t a) {
    const uint64_t ninv = inv_small(mod_small(N, a), a);
    const uint32_t t = (uint32_t)((a - mod_small(x, a)) * ninv % a);
    return div_small(add(mul_small(N, t), x), a);
  };
  Limbs f = mod(R.MB, N);  // MB, or MB / MA
  if (mont)
    for (int i = 0; i < n; ++i) f = div_mod(f, R.a[i]);
  o.C.assign((size_t)o.nblk * n * 8, 0);
  for (int j = 0; j < n; ++j) {  // g_j f / b_j
    Limbs c = mod(mul_small(div_mod(f, R.b[j]), (uint32_t)std::abs(R.g[j])), N);
    if (R.g[j] < 0 && !is_zero(c)) c = sub(N, c);
    const std::vector<uint32_t> l = limbs28(c, SB);
    for (int i = 0; i < SB; ++i) o.C[((size_t)(i / 8) * n + j) * 8 + i % 8] = l[i];
    o.F.push_back((int64_t)std::nearbyintl((long double)R.g[j] / (long double)R.b[j] *
                                           68719476736.0L));
  }
  o.D = limbs28(is_zero(f) ? f : sub(N, f), SB);
  Limbs off(N.size() + 1, 0);
  off = resized(mul_small(N, 1u << 26), N.size() + 1);
  o.O = limbs28(off, SB);
  o.N28 = limbs28(N, SB);
  double top = 0;
  for (int i = o.S - 1; i >= o.S - 4 && i >= 0; --i) top = top * 268435456.0 + o.N28[i];
  o.ntop_inv = 1.0 / top;
  return o;
}

// The program of x^e (sliding-window schedule `sched` of width w), closed by
// the product with the second input if gm.
inline std::vector<uint32_t> rns_program(const std::vector<uint32_t>& sched, int w, bool gm) {
  using namespace pc2k;
  std::vector<uint32_t> p;
  const uint32_t half = 1u << (w - 1);  // entry j < half: x^(2 j + 1); entry half: x^2
  p.push_back(rns_op(RNS_LOAD, 0, RNS_NODST));
  p.push_back(rns_op(RNS_MUL, RNS_SQ, half));
  p.push_back(rns_op(RNS_MUL, 0, 1));
  for (uint32_t j = 2; j < half; ++j) p.push_back(rns_op(RNS_MUL, half, j));
  p.push_back(rns_op(RNS_LOAD, (sched[0] & 0xFFFFu) >> 1, RNS_NODST));
  for (size_t i = 1; i < sched.size(); ++i) {
    for (uint32_t k = sched[i] >> 16; k; --k) p.push_back(rns_op(RNS_MUL, RNS_SQ, RNS_NODST));
    const uint32_t d = sched[i] & 0xFFFFu;
    if (d) p.push_back(rns_op(RNS_MUL, d >> 1, RNS_NODST));
  }
  if (gm) p.push_back(rns_op(RNS_MUL, RNS_GM, RNS_NODST));
  if (p.back() >> 16 != RNS_MUL) return {};  // the power is a table entry: not a key's exponent
  p.back() = rns_op(RNS_MUL, p.back() & 0xFFu, RNS_OUT);
  p.push_back(rns_op(RNS_END, 0, RNS_NODST));
  return p;
}

}  // namespace pc2h
