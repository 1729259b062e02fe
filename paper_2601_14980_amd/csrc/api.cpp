// C ABI of libpc2 (declared in include/pc2.h): contexts, keys, argument
// validation, scratch sizing and kernel launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/pc2.h"
#include "host_bn.hpp"
#include "launch.hpp"
#include "pc2_types.hpp"
#include "rns_host.hpp"
#include "rns_launch.hpp"

using pc2h::Limbs;

// Launch shape of k_rns_pow for one call (rns_plan).
struct RnsPlan {
  int T = 0, nb = 0, grid = 0, w = 0;
  bool wide = false;
  size_t ngroups = 0, group_bytes = 0, table_bytes = 0;
  double cost = 0;  // of a product, over all rounds of workgroups (rns_plan)
  size_t stage_bytes() const { return ngroups * group_bytes; }  // one input, one modulus
};

struct pc2_ctx {
  int device = 0;
  int cus = 0;
  int* err = nullptr;          // device word, latched error bits
  uint32_t* scratch = nullptr; // per-tile tables and per-call staging
  size_t scratch_bytes = 0;    // sized by the key constructors and pc2_ctx_reserve
  hipEvent_t done = nullptr;   // recorded after the last call that used the scratch
  void* done_stream = nullptr; // ... on this stream
  bool done_valid = false;
  int window = 0;              // 0 = automatic
  int modmul = PC2_MODMUL_AUTO;
  int tile = 0;                // PC2_OPT_TILE: 0 automatic, 1 wide, else lanes per ciphertext
  int occ[pc2k::NUM_GEOS][pc2k::OP_COUNT] = {};    // workgroups per CU (0 = not queried)
  int tuned[pc2k::NUM_GEOS][pc2k::OP_COUNT] = {};  // autotuned windows (0 = none)
  int tuned_geo[pc2k::NUM_CLASSES] = {-1, -1, -1, -1, -1, -1, -1, -1, -1};  // encryption tile
  int rocc[2][pc2k::RNS_NT][pc2k::RNS_NBMAX + 1] = {};  // RNS powering (wide): workgroups per CU
  int gocc[pc2k::RNS_NGATHER][pc2k::RNS_NT][pc2k::RNS_NBMAX + 1] = {};  // and the gather kernels'
};

// One key's jobs of a batch or runner launch on the RNS engine.
struct RnsPart {
  const pc2_pk* pk = nullptr;  // encryption
  const pc2_sk* sk = nullptr;  // decryption
  RnsPlan plan;
  pc2k::RnsJobs jobs{};
  bool side = false;           // batches: runs beside the others
};

struct pc2_runner {
  pc2_ctx* ctx = nullptr;
  int op = 0, max_cls = 0;
  size_t max_jobs = 0, max_groups = 0, max_ptrs = 0;
  size_t slot_words = 0;
  int grid_cap = 0;
  int ls = 0;            // largest prime (limbs) the decryption staging holds
  void* dev = nullptr;   // jobs | items | pointers | queue
  void* host = nullptr;  // pinned staging, same layout
  size_t jobs_b = 0, items_b = 0, ptr_b = 0;
  uint32_t* scratch = nullptr;
  uint32_t* stage = nullptr;  // decryption: CRT halves of one launch's groups
  uint8_t* mscratch = nullptr;  // encryption on the matrix cores: tables of the widest grid
  size_t mscratch_bytes = 0;
  uint8_t* rscratch = nullptr;  // the RNS engine's tables and staging
  size_t rscratch_bytes = 0, rjobs_b = 0;
  int mocc[pc2k::NUM_CLASSES] = {};  // resident workgroups per CU of k_batch_mfma per class
  hipEvent_t copied = nullptr;
  bool pending = false;
};

struct pc2_admm {
  pc2_ctx* ctx = nullptr;
  const double* A = nullptr;
  int N = 0, B = 0, K = 0;
  double rho = 1.0;
  double* buf = nullptr;  // W (K B B) | aty (K N) | w (K N) | t (K B) | s (K B)
  double *W = nullptr, *aty = nullptr, *w = nullptr, *t = nullptr, *s = nullptr;
};

struct pc2_batch {
  pc2_ctx* ctx = nullptr;
  int op = 0, pair = 0, grid = 0, nitems = 0;
  int w_a = 5, w_b = 5;
  size_t slot_words = 0;
  void* dev = nullptr;  // jobs, items, pointer/length arrays, queue
  pc2k::BatchJob* jobs = nullptr;
  pc2k::BatchItem* items = nullptr;
  int* queue = nullptr;
  uint32_t* scratch = nullptr;
  uint32_t* stage = nullptr;  // decryption: CRT halves of every job's elements
  // encryption jobs of up to two key classes that run on the matrix cores:
  // per class its own items (after the others), queue, grid and window; one
  // table scratch for both (the launches run in order on one stream)
  struct MPart {
    int cls = -1, grid = 0, nitems = 0, w = 6, sub = 1;  // sub: largest group of its jobs
    pc2k::BatchItem* items = nullptr;
    int* queue = nullptr;
  } mp[2];
  uint8_t* mscratch = nullptr;
  // jobs on the RNS engine, one part per key: its jobs and plan.  The parts run
  // one after another on the caller's stream (one scratch for all), or two of
  // them side by side, the second on `side` (rns_parts_pair)
  std::vector<RnsPart> rparts;
  uint8_t *rscratch = nullptr, *rscratch2 = nullptr;
  hipStream_t side = nullptr;
  hipEvent_t forked = nullptr, joined = nullptr;
  hipGraphExec_t exec = nullptr;
  void* graph_stream = nullptr;
};

struct pc2_matvec {
  pc2_ctx* ctx = nullptr;
  const pc2_pk* pk = nullptr;
  int w = 0, nw = 0, ebits = 0;
  size_t cols = 0, table_bytes = 0;
  uint32_t* tab = nullptr;    // fixed-base tables [cols][nw][2^w - 1] entries
  uint32_t* parts = nullptr;  // partial products of row chunks [chunks][rows][2L]
  size_t parts_bytes = 0;
  int cap_table = 1, cap_apply = 1;  // resident workgroups of the two kernels
  bool loaded = false;
  // on the RNS engine (rdg.n > 0): the digits of the constants, whose entries are
  // in tab; the running values of rblocks blocks of 32 rows, and a flag per row
  pc2k::RnsDigits rdg{};
  uint8_t* rstage = nullptr;
  size_t rstage_bytes = 0;
  uint32_t* rbad = nullptr;
  size_t rblocks = 0;
  hipEvent_t done = nullptr;  // after the last call that used them, on done_stream
  void* done_stream = nullptr;
  bool done_valid = false;
};

struct pc2_colsplit {
  pc2_ctx* ctx = nullptr;
  const pc2_sk* sk = nullptr;
  int M = 0, N = 0, K = 0, Nk = 0, k = 0;
  double rho = 1.0;
  const uint32_t* r_pool = nullptr;
  size_t r_count = 0, iter = 0;
  std::vector<pc2_matvec*> mv;  // one plan per node over Gamma_2(rho B_k)
  void* dev = nullptr;          // per-node constants, then per-iteration staging
  double *alpha = nullptr, *rhoB = nullptr;       // [K][Nk], [K][Nk][Nk]
  uint64_t *G = nullptr, *R = nullptr;            // [K][Nk][Nk], [K][Nk]
  uint32_t* ahat = nullptr;                       // [K][Nk][2L] Enc(Gamma_1(alpha_k))
  uint64_t *w = nullptr, *S = nullptr;            // [2][N] Gamma_2(z), Gamma_2(-v); [K]
  uint32_t *cw = nullptr, *c = nullptr, *xhat = nullptr, *P = nullptr;  // [2N][2L], [N][2L] x2, [N][L]
  uint32_t* g1 = nullptr;                         // [K][Nk][4] Gamma_1(alpha_k)
};

struct pc2_pk {
  pc2_ctx* ctx = nullptr;
  int device = 0;
  uint32_t nbits = 0;
  int L = 0;
  int cls = 0;
  void* dev = nullptr;  // one allocation holding every constant
  pc2k::PkConst c{};
  pc2k::PkConst alt{};  // n^2 constants in the alternative tile (ALT_GEO[cls] >= 0)
  pc2k::RnsKey rn{};    // modulo n^2, power n (T = 0: not on the RNS engine)
};

struct pc2_sk {
  pc2_ctx* ctx = nullptr;
  pc2_pk pk;            // the public part (owns nothing; dev below owns all)
  void* dev = nullptr;
  pc2k::SkConst c{};
  bool crt_ok = false;  // p < 2 q: the key-holder encryption's inputs fit mod q^2
  pc2k::RnsKey dec[2]{};  // modulo p^2, q^2: power s - 1, output times MA^-1
  pc2k::RnsKey enc[2]{};  // ... power n mod s (s - 1), 1 + m n
};

namespace {

// ------------------------------------------------------------ helpers
struct DevBuf {
  std::vector<uint32_t> words;
  // append words, 16-byte aligned; returns the word offset
  size_t add(const std::vector<uint32_t>& w) {
    size_t off = words.size();
    words.insert(words.end(), w.begin(), w.end());
    while (words.size() % 4) words.push_back(0);
    return off;
  }
};

// value -> chunked D-digit layout for geometry (D, K, T)
std::vector<uint32_t> to_chunk(const Limbs& v, int D, int K, int T) {
  const int K4 = (K + 3) & ~3;
  std::vector<uint32_t> out((size_t)T * K4, 0);
  const int S = K * T;
  for (int g = 0; g < S; ++g) {
    long bit = (long)g * D;
    size_t w = bit / 32;
    int s = bit % 32;
    uint64_t lo = w < v.size() ? v[w] : 0, hi = w + 1 < v.size() ? v[w + 1] : 0;
    uint32_t d = (uint32_t)(((hi << 32) | lo) >> s) & ((1u << D) - 1u);
    out[(size_t)(g / K) * K4 + (g % K)] = d;
  }
  return out;
}


// Montgomery constants of odd N in geometry (D, K, T), appended to buf.
struct ModOffsets {
  size_t N, R1, R2, R3, ONE, Nl;
  uint32_t nprime;
  int nl;
};
ModOffsets add_modulus(DevBuf& buf, const Limbs& N0, int D, int K, int T, int nl) {
  Limbs N = N0;
  pc2h::trim(N);
  const int S = K * T;
  const uint64_t RB = (uint64_t)D * S;  // R = 2^RB
  ModOffsets o{};
  Limbs r1 = pc2h::pow2_mod(RB, N);
  Limbs r2 = pc2h::shl_mod(r1, RB, N);
  Limbs r3 = pc2h::shl_mod(r2, RB, N);
  o.N = buf.add(to_chunk(N, D, K, T));
  o.R1 = buf.add(to_chunk(r1, D, K, T));
  o.R2 = buf.add(to_chunk(r2, D, K, T));
  o.R3 = buf.add(to_chunk(r3, D, K, T));
  o.ONE = buf.add(to_chunk(Limbs{1}, D, K, T));
  o.Nl = buf.add(pc2h::resized(N, nl));
  uint32_t inv = pc2h::inv32(N[0]);
  o.nprime = (0u - inv) & ((1u << D) - 1u);
  o.nl = nl;
  return o;
}
pc2k::ModConst mod_const(const uint32_t* base, const ModOffsets& o) {
  pc2k::ModConst m{};
  m.N = base + o.N;
  m.R1 = base + o.R1;
  m.R2 = base + o.R2;
  m.R3 = base + o.R3;
  m.ONE = base + o.ONE;
  m.Nl = base + o.Nl;
  m.nprime = o.nprime;
  m.nl = o.nl;
  return m;
}


// Left-to-right sliding-window schedule of e > 0 (see pc2k::Sched)
std::vector<uint32_t> sliding_schedule(const Limbs& e0, int w) {
  Limbs e = e0;
  pc2h::trim(e);
  auto bit = [&](int i) -> uint32_t { return (e[i / 32] >> (i % 32)) & 1u; };
  std::vector<uint32_t> out;
  int i = pc2h::bitlen(e) - 1;
  uint32_t sq = 0;
  bool first = true;
  while (i >= 0) {
    if (!bit(i)) {
      ++sq;
      --i;
      continue;
    }
    int j = std::max(i - w + 1, 0);
    while (!bit(j)) ++j;
    uint32_t d = 0;
    for (int k = i; k >= j; --k) d = (d << 1) | bit(k);
    if (!first) sq += (uint32_t)(i - j + 1);
    out.push_back((sq << 16) | d);
    first = false;
    sq = 0;
    i = j - 1;
  }
  if (sq) out.push_back(sq << 16);
  return out;
}

struct SchedOffsets {
  size_t off[pc2k::SCHED_WMAX - pc2k::SCHED_WMIN + 1];
  int n[pc2k::SCHED_WMAX - pc2k::SCHED_WMIN + 1];
};
SchedOffsets add_schedules(DevBuf& buf, const Limbs& e) {
  SchedOffsets o{};
  for (int w = pc2k::SCHED_WMIN; w <= pc2k::SCHED_WMAX; ++w) {
    std::vector<uint32_t> sc = sliding_schedule(e, w);
    o.off[w - pc2k::SCHED_WMIN] = buf.add(sc);
    o.n[w - pc2k::SCHED_WMIN] = (int)sc.size();
  }
  return o;
}
pc2k::Sched sched_const(const uint32_t* base, const SchedOffsets& o) {
  pc2k::Sched c{};
  for (int i = 0; i <= pc2k::SCHED_WMAX - pc2k::SCHED_WMIN; ++i) {
    c.p[i] = base + o.off[i];
    c.n[i] = o.n[i];
  }
  return c;
}

struct GeoOffsets {  // the n^2 constants that depend on the digit geometry
  ModOffsets n2;
  size_t nR, Rk;
};
struct PkOffsets {
  GeoOffsets g, alt;  // alt: only for classes with an alternative tile
  size_t n;
  size_t mN, mNp, mR2, mnR, mRk, mN28;  // matrix-core product constants
  int mS;
  SchedOffsets nsch;
};

// v -> D = 4 S forward 7-bit digits, one per byte after 64 zero bytes, with
// a zero tail to 64 + D8 + 16 bytes (D8 = D rounded up to 16)
std::vector<uint32_t> to_digits7(const Limbs& v, int S) {
  const int D = 4 * S, FB = 64 + ((D + 15) & ~15) + 16;
  std::vector<uint32_t> out(FB / 4, 0);
  for (int i = 0; i < D; ++i) {
    const long bit = (long)i * 7;
    const size_t w = bit / 32;
    const int sh = bit % 32;
    const uint64_t lo = w < v.size() ? v[w] : 0, hi = w + 1 < v.size() ? v[w + 1] : 0;
    const uint32_t d = (uint32_t)(((hi << 32) | lo) >> sh) & 0x7Fu;
    out[(64 + i) / 4] |= d << (8 * (i % 4));
  }
  return out;
}

// v -> S limbs of 28 bits
std::vector<uint32_t> to_limbs28(const Limbs& v, int S) {
  std::vector<uint32_t> out(S, 0);
  for (int i = 0; i < S; ++i) {
    const long bit = (long)i * 28;
    const size_t w = bit / 32;
    const int sh = bit % 32;
    const uint64_t lo = w < v.size() ? v[w] : 0, hi = w + 1 < v.size() ? v[w + 1] : 0;
    out[i] = (uint32_t)(((hi << 32) | lo) >> sh) & ((1u << 28) - 1u);
  }
  return out;
}

// n^2, n R and the powers R^k mod n^2 in the digit geometry `geo`
GeoOffsets add_geo(DevBuf& buf, const Limbs& n, const Limbs& n2, int geo, int L) {
  const pc2k::ClassGeo g = pc2k::CLASS_GEO[geo];
  GeoOffsets o{};
  o.n2 = add_modulus(buf, n2, g.nD, g.nK, g.nT, 2 * L);
  const uint64_t RB = (uint64_t)g.nD * g.nK * g.nT;
  Limbs nR = pc2h::shl_mod(n, RB, n2);
  o.nR = buf.add(to_chunk(nR, g.nD, g.nK, g.nT));
  // R^k mod n^2, k = 0..RK_MAX, by Montgomery products with 32-bit limbs
  pc2h::Mont32 M(n2);
  Limbs r1m = M.to(pc2h::pow2_mod(RB, n2));
  Limbs rkm = M.to(Limbs{1});
  std::vector<uint32_t> tab;
  for (int k = 0; k <= pc2k::RK_MAX; ++k) {
    std::vector<uint32_t> ch = to_chunk(M.from(rkm), g.nD, g.nK, g.nT);
    tab.insert(tab.end(), ch.begin(), ch.end());
    rkm = M.mm(rkm, r1m);
  }
  o.Rk = buf.add(tab);
  return o;
}

PkOffsets add_public(DevBuf& buf, const Limbs& n, int cls, int L) {
  Limbs n2 = pc2h::mul(n, n);
  PkOffsets o{};
  o.g = add_geo(buf, n, n2, cls, L);
  if (pc2k::ALT_GEO[cls] >= 0) o.alt = add_geo(buf, n, n2, pc2k::ALT_GEO[cls], L);
  o.n = buf.add(pc2h::resized(n, L));
  // matrix-core form: R = 2^(28 S), N' = -N^-1 mod R
  const int S = pc2k::MFMA_S[cls];
  const uint64_t RBm = 28ull * S;
  Limbs N = n2;
  pc2h::trim(N);
  const size_t nw = (RBm + 31) / 32;
  Limbs inv = pc2h::inv_pow2(N, nw);
  Limbs Rm = pc2h::resized(Limbs{}, nw + 1);
  Rm[RBm / 32] |= 1u << (RBm % 32);  // 2^RBm (RBm < 32 nw + 32)
  Limbs invR = pc2h::resized(inv, nw);
  if (RBm % 32) invR[nw - 1] &= (1u << (RBm % 32)) - 1u;  // inv mod 2^RBm
  pc2h::trim(invR);
  Limbs np = pc2h::sub(Rm, invR);  // 2^RBm - inv (inv != 0 for odd N)
  pc2h::trim(np);
  o.mS = S;
  o.mN = buf.add(to_digits7(N, S));
  o.mNp = buf.add(to_digits7(np, S));
  o.mR2 = buf.add(to_digits7(pc2h::pow2_mod(2 * RBm, N), S));
  o.mnR = buf.add(to_digits7(pc2h::shl_mod(n, RBm, N), S));
  {  // R^k mod n^2, k = 0..RK_MAX (R = 2^RBm), by Montgomery products with 32-bit limbs
    pc2h::Mont32 M(N);
    const Limbs r1m = M.to(pc2h::pow2_mod(RBm, N));
    Limbs rkm = M.to(Limbs{1});
    std::vector<uint32_t> tab;
    for (int k = 0; k <= pc2k::RK_MAX; ++k) {
      const std::vector<uint32_t> d = to_digits7(M.from(rkm), S);
      tab.insert(tab.end(), d.begin(), d.end());
      rkm = M.mm(rkm, r1m);
    }
    o.mRk = buf.add(tab);
  }
  o.mN28 = buf.add(to_limbs28(N, S));
  o.nsch = add_schedules(buf, n);
  return o;
}

pc2k::PkConst pk_const(const uint32_t* base, const PkOffsets& o, int L, int nbits) {
  pc2k::PkConst c{};
  c.n2 = mod_const(base, o.g.n2);
  c.nR = base + o.g.nR;
  c.Rk = base + o.g.Rk;
  c.n = base + o.n;
  c.L = L;
  c.nbits = nbits;
  c.mf.N = (const uint8_t*)(base + o.mN);
  c.mf.Np = (const uint8_t*)(base + o.mNp);
  c.mf.R2 = (const uint8_t*)(base + o.mR2);
  c.mf.nR = (const uint8_t*)(base + o.mnR);
  c.mf.Rk = (const uint8_t*)(base + o.mRk);
  c.mf.N28 = base + o.mN28;
  c.mf.S = o.mS;
  c.nsch = sched_const(base, o.nsch);
  return c;
}

// the same key with the n^2 constants of the alternative tile
pc2k::PkConst pk_const_alt(const uint32_t* base, const PkOffsets& o, const pc2k::PkConst& c) {
  pc2k::PkConst a = c;
  a.n2 = mod_const(base, o.alt.n2);
  a.nR = base + o.alt.nR;
  a.Rk = base + o.alt.Rk;
  return a;
}

// ---------------------------------------------------------- RNS engine keys
struct RnsOffsets {
  int T = 0;
  size_t E1, E2, c2, kb, ka;
  struct To { size_t E = 0, cst = 0; int nchunk = 0; } x, gm, c;
  size_t one;
  struct From { size_t C, D, O, N28, F; int S, nblk; double ntop_inv; } from;
  size_t ops[5];
};
size_t add_aligned(DevBuf& buf, const std::vector<uint32_t>& w) {
  while (buf.words.size() % 64) buf.words.push_back(0);  // 256 bytes
  return buf.add(w);
}
RnsOffsets::To add_rns_to(DevBuf& buf, const pc2h::RnsToHost& h) {
  return {add_aligned(buf, h.E), add_aligned(buf, h.cst), h.nchunk};
}
// Powers x^e modulo N (N of `tiles`), x of nhalf 16-bit halves; f2 != null: a
// second input 1 + m f2 (m of mhalf halves) closes the product, else the
// result leaves Montgomery form on output; chalf > 0: also what products of
// ciphertexts of chalf halves need.  E2, c2, kb and ka depend on the
// tile count alone: `same` (null: none) names a modulus whose copies to use.
// T = 0 in the result: the engine does not take this modulus.
RnsOffsets add_rns(DevBuf& buf, const Limbs& N, int T, const Limbs& e, int nhalf, const Limbs* f2,
                   int mhalf, const RnsOffsets* same, int chalf = 0) {
  RnsOffsets o;
  if (T == 0) return o;
  const pc2h::RnsBase& R = pc2h::rns_base(T);
  std::vector<uint32_t> E1, c1;
  if (!pc2h::rns_e1(R, N, &E1, &c1)) return o;
  std::vector<uint32_t> prog[5];
  for (int w = pc2k::SCHED_WMIN; w <= pc2k::SCHED_WMAX; ++w) {
    prog[w - pc2k::SCHED_WMIN] = pc2h::rns_program(sliding_schedule(e, w), w, f2 != nullptr);
    if (prog[w - pc2k::SCHED_WMIN].empty()) return o;
  }
  o.E1 = add_aligned(buf, E1);
  if (same && same->T == T) {
    o.E2 = same->E2;
    o.c2 = same->c2;
    o.kb = same->kb;
    o.ka = same->ka;
  } else {
    o.E2 = add_aligned(buf, R.E2);
    o.c2 = add_aligned(buf, R.c2);
    o.kb = add_aligned(buf, R.kb);
    o.ka = add_aligned(buf, R.ka);
  }
  o.x = add_rns_to(buf, pc2h::rns_to(R, N, R.MA, nhalf, false));
  if (f2) o.gm = add_rns_to(buf, pc2h::rns_to(R, N, *f2, mhalf, true));
  if (chalf) {
    o.c = add_rns_to(buf, pc2h::rns_to(R, N, Limbs{1}, chalf, false));
    std::vector<uint32_t> one;
    for (const Limbs& v : {R.MA, pc2h::mul(R.MA, R.MA), Limbs{1}}) {
      const std::vector<uint32_t> w = pc2h::rns_entry(R, N, v);
      one.insert(one.end(), w.begin(), w.end());
    }
    o.one = add_aligned(buf, one);
  }
  const pc2h::RnsFromHost h = pc2h::rns_from(R, N, f2 == nullptr);
  std::vector<uint32_t> F;
  for (int64_t v : h.F) {
    F.push_back((uint32_t)v);
    F.push_back((uint32_t)((uint64_t)v >> 32));
  }
  o.from = {add_aligned(buf, h.C), add_aligned(buf, h.D), add_aligned(buf, h.O),
            add_aligned(buf, h.N28), add_aligned(buf, F), h.S, h.nblk, h.ntop_inv};
  for (int i = 0; i < 5; ++i) o.ops[i] = add_aligned(buf, prog[i]);
  o.T = T;
  return o;
}
pc2k::RnsTo rns_to_const(const uint32_t* base, const RnsOffsets::To& t, const pc2k::RnsMod& M) {
  return {(const uint8_t*)(base + t.E), (const int32_t*)(base + t.cst), M.kb, M.ka, t.nchunk};
}
pc2k::RnsKey rns_const(const uint32_t* base, const RnsOffsets& o, int nw) {
  pc2k::RnsKey k{};
  if (o.T == 0) return k;
  k.T = o.T;
  k.M = {(const uint8_t*)(base + o.E1), (const uint8_t*)(base + o.E2),
         (const int32_t*)(base + o.c2), base + o.kb, base + o.ka};
  k.x = rns_to_const(base, o.x, k.M);
  if (o.gm.nchunk) k.gm = rns_to_const(base, o.gm, k.M);
  if (o.c.nchunk) {
    k.c = rns_to_const(base, o.c, k.M);
    k.one = (const uint8_t*)(base + o.one);
  }
  k.from = {base + o.from.C, base + o.from.D, base + o.from.O, base + o.from.N28,
            (const int64_t*)(base + o.from.F), o.from.S, o.from.nblk, nw, o.from.ntop_inv};
  for (int i = 0; i < 5; ++i) k.ops[i] = base + o.ops[i];
  return k;
}
// Tile count of a modulus of a key of class cls, by the modulus' own length; 0 in
// the classes below 512-bit keys (nbits <= 256) and for a modulus of fewer than 512
// bits, whose products are short on the VALU engine (the output conversion's
// quotient, too, wants four limbs and more).
constexpr int RNS_MIN_CLASS = 4;
int rns_tiles_for(int cls, const Limbs& N) {
  const int bits = pc2h::bitlen(N);
  return cls >= RNS_MIN_CLASS && bits >= 512 ? pc2h::rns_tiles(bits) : 0;
}

RnsOffsets add_rns_public(DevBuf& buf, const Limbs& n, int cls, int L) {
  Limbs n2 = pc2h::mul(n, n);
  pc2h::trim(n2);
  return add_rns(buf, n2, rns_tiles_for(cls, n2), n, 2 * L, &n, 2 * L, nullptr, 4 * L);
}

struct HalfOffsets {
  ModOffsets s2;
  size_t s, e, sinv, H;
  uint32_t s_n0;
  int Ls;
  SchedOffsets esch;
  size_t nRs;
  SchedOffsets nsch;
};

// constants for the prime s (other prime t, n = s t) of the CRT decryption
HalfOffsets add_half(DevBuf& buf, const Limbs& s, const Limbs& t, const Limbs& n, int cls, int Ls,
                     int nl2) {
  const pc2k::ClassGeo g = pc2k::CLASS_GEO[cls];
  HalfOffsets o{};
  Limbs s2 = pc2h::mul(s, s);
  o.s2 = add_modulus(buf, s2, g.pD, g.pK, g.pT, nl2);
  o.s = buf.add(pc2h::resized(s, Ls));
  o.e = buf.add(pc2h::resized(pc2h::sub(pc2h::resized(s, Ls), Limbs{1}), Ls));
  Limbs sinv = pc2h::inv_pow2(s, Ls);
  o.sinv = buf.add(sinv);
  // h_s = L_s(g^(s-1) mod s^2)^-1 mod s with g = n + 1
  pc2h::Mont32 M2(s2);
  Limbs gm = pc2h::mod(pc2h::add(n, Limbs{1}), s2);
  Limbs y = M2.pow(gm, pc2h::sub(pc2h::resized(s, Ls), Limbs{1}));
  Limbs ym1 = pc2h::sub(pc2h::resized(y, (size_t)2 * Ls + 1), Limbs{1});
  Limbs u = pc2h::resized(pc2h::mul(pc2h::resized(ym1, Ls), sinv), Ls);  // exact (y-1)/s
  Limbs hs = pc2h::inv_mod_prime(pc2h::mod(u, s), s);
  Limbs H = pc2h::shl_mod(hs, (uint64_t)32 * Ls, s);
  o.H = buf.add(pc2h::resized(H, Ls));
  o.s_n0 = 0u - pc2h::inv32(s[0]);
  o.Ls = Ls;
  o.esch = add_schedules(buf, pc2h::sub(s, Limbs{1}));
  // key-holder encryption mod s^2: n R mod s^2 and n mod s (s - 1)
  const uint64_t RBs = (uint64_t)g.pD * g.pK * g.pT;
  o.nRs = buf.add(to_chunk(pc2h::shl_mod(n, RBs, s2), g.pD, g.pK, g.pT));
  Limbs order = pc2h::mul(s, pc2h::sub(s, Limbs{1}));
  pc2h::trim(order);
  Limbs ne = pc2h::mod(n, order);
  pc2h::trim(ne);
  if (ne.empty()) ne = order;  // n = 0 mod s (s-1) cannot happen for n = p q, s | n
  o.nsch = add_schedules(buf, ne);
  (void)t;
  return o;
}

pc2k::HalfConst half_const(const uint32_t* base, const HalfOffsets& o) {
  pc2k::HalfConst h{};
  h.s2 = mod_const(base, o.s2);
  h.s = base + o.s;
  h.e = base + o.e;
  h.sinv = base + o.sinv;
  h.H = base + o.H;
  h.s_n0 = o.s_n0;
  h.Ls = o.Ls;
  h.esch = sched_const(base, o.esch);
  h.nRs = base + o.nRs;
  h.nsch = sched_const(base, o.nsch);
  return h;
}

Limbs limbs_from(const uint32_t* p, size_t n) {
  Limbs v(p, p + n);
  pc2h::trim(v);
  return v;
}

int upload(pc2_ctx* ctx, const DevBuf& buf, void** dev) {
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  if (hipMalloc(dev, buf.words.size() * 4) != hipSuccess) return PC2_E_NOMEM;
  if (hipMemcpy(*dev, buf.words.data(), buf.words.size() * 4, hipMemcpyHostToDevice) !=
      hipSuccess) {
    (void)hipFree(*dev);
    *dev = nullptr;
    return PC2_E_DEVICE;
  }
  return PC2_OK;
}

int auto_window(int geo, int op) {
  // window width minimising products for the exponent lengths of each class
  // (sliding windows for the wave-uniform exponents of encryption and
  // decryption)
  const int cls = pc2k::GEO_CLASS[geo];
  if (op == pc2k::OP_SMUL) return 4;
  return cls >= 6 ? 6 : (cls >= 5 ? 5 : (cls >= 3 ? 4 : 3));
}

int window_for(const pc2_ctx* ctx, int geo, int op) {
  if (ctx->window) return ctx->window;
  if (op == pc2k::OP_FUSED_MFMA || op == pc2k::OP_ENC_TEAM) op = pc2k::OP_ENC_MFMA;
  const int t = ctx->tuned[geo][op == pc2k::OP_FUSED ? pc2k::OP_ENC : op];
  // (matrix-core engine, 2048-bit keys: w = 6 measured 1 % faster than 5)
  if (op == pc2k::OP_ENC_MFMA) return t ? t : (geo >= 6 ? 6 : (geo >= 5 ? 5 : 4));
  return t ? t : auto_window(geo, op);
}

// Whether an encryption under a key of class cls that the RNS engine does not
// take (enc_engine) runs on the matrix cores, a wavefront per element, also when
// it fills the device: when asked for, or automatically from 2048-bit keys
// (class 6) on, where that measured faster than the VALU engine.
constexpr int MFMA_AUTO_CLASS = 6;
bool use_mfma(const pc2_ctx* ctx, int cls) {
  return ctx->modmul == PC2_MODMUL_MFMA ||
         (ctx->modmul == PC2_MODMUL_AUTO && cls >= MFMA_AUTO_CLASS);
}

// Geometry of an encryption of `count` elements under the key class cls:
// the alternative tile if PC2_OPT_TILE asks for wide tiles or names its lane
// count, the class's own tile for any other lane count.  Automatic: a launch
// that gives every SIMD at most one wavefront of the (wider) alternative tile
// is latency-bound, and the wider tile finishes it sooner, so it takes that;
// a larger one takes the autotuned tile, else the class's own.  Batches and
// runners pass no count (their geometry is fixed per key when groups are cut).
int enc_geo(const pc2_ctx* ctx, int cls, size_t count = SIZE_MAX) {
  const int alt = pc2k::ALT_GEO[cls];
  if (alt < 0) return cls;
  if (ctx->tile == PC2_TILE_WIDE) return alt;
  if (ctx->tile) return pc2k::CLASS_GEO[alt].nT == ctx->tile ? alt : cls;
  if (count <= (size_t)ctx->cus * 4 * (size_t)pc2k::elems_per_block(alt)) return alt;
  return ctx->tuned_geo[cls] >= 0 ? ctx->tuned_geo[cls] : cls;
}
// the key's constants in geometry geo (its own class or its alternative tile)
const pc2k::PkConst& geo_const(const pc2_pk* pk, int geo) {
  return geo == pk->cls ? pk->c : pk->alt;
}
// the geometry a batched or queued job of operation op runs in
int job_geo(const pc2_ctx* ctx, const pc2_pk* pk, int op) {
  return op == pc2k::OP_ENC ? enc_geo(ctx, pk->cls) : pk->cls;
}

int occupancy(pc2_ctx* ctx, int geo, int op) {
  int& o = ctx->occ[geo][op];
  if (o == 0) {
    int v = 0;
    int threads = 64;
    const void* k = op == pc2k::OP_ENC_TEAM     ? pc2k::kernel_encrypt_team(geo, &threads)
                    : op == pc2k::OP_ENC_MFMA   ? pc2k::kernel_encrypt_mfma(geo)
                    : op == pc2k::OP_FUSED_MFMA ? pc2k::kernel_encrypt_mfma(geo, true)
                                                : pc2k::kernel_for(geo, op);
    if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k, threads, 0) != hipSuccess ||
        v <= 0)
      v = 1;
    o = v;
  }
  return o;
}

// Grid and table slot of a Paillier launch over `count` elements in geometry
// geo (the key class, except for an encryption in an alternative tile) with
// window w; returns the bytes of scratch the launch needs.  The scratch holds
// aux_words of per-call staging first (Launch::aux, at the same place for
// every launch that asks for the same amount), then the tables.
size_t plan_launch(pc2_ctx* ctx, int geo, int op, size_t count, int Ls, int L, int w,
                   pc2k::Launch* l, void* stream, size_t aux_words) {
  const bool mf = op == pc2k::OP_ENC_MFMA || op == pc2k::OP_FUSED_MFMA || op == pc2k::OP_ENC_TEAM;
  const size_t epb = mf ? 1 : (size_t)pc2k::elems_per_block(geo);
  const size_t groups = (count + epb - 1) / epb;
  const size_t cap = (size_t)ctx->cus * occupancy(ctx, geo, op);
  l->grid = (int)std::max<size_t>(1, std::min(groups, cap));
  l->window = w;
  l->err = ctx->err;
  l->stream = stream;
  int tiles = 0;
  size_t words = 0;
  if (mf) {  // one table of 2^w digit arrays per workgroup
    tiles = 1;
    words = (pc2k::mfma_digit_bytes(geo) << w) / 4;
  } else {
    pc2k::slot_shape(geo, op, w, Ls, L, &tiles, &words);
  }
  words = (words + 3) & ~(size_t)3;
  l->slot_words = words;
  const size_t aux = (aux_words + 63) & ~(size_t)63;
  return (aux + (size_t)l->grid * tiles * words) * 4;
}

// A data call's launch in the context's scratch.  Data calls never allocate:
// the key constructors sized the scratch for every call of their key class
// (class_scratch_need), so a launch that does not fit is PC2_E_NOMEM.
int prepare(pc2_ctx* ctx, int geo, int op, size_t count, int Ls, int L, pc2k::Launch* l,
            void* stream, size_t aux_words = 0) {
  const size_t need = plan_launch(ctx, geo, op, count, Ls, L, window_for(ctx, geo, op), l,
                                  stream, aux_words);
  if (need > ctx->scratch_bytes || !ctx->scratch) return PC2_E_NOMEM;
  const size_t aux = (aux_words + 63) & ~(size_t)63;
  l->aux = aux_words ? ctx->scratch : nullptr;
  l->scratch = ctx->scratch + aux;
  return PC2_OK;
}

// ------------------------------------------------------------- RNS launches
int rns_index(int T) {
  for (int i = 0; i < pc2k::RNS_NT; ++i)
    if (pc2k::RNS_T[i] == T) return i;
  return 0;
}
// resident workgroups of k_rns_pow<T, nb>, or of a kernel with a multiplier per
// element (0: not compiled)
int rns_slots(pc2_ctx* ctx, int T, int nb, int gather = -1, bool wide = false) {
  int& o =
      gather < 0 ? ctx->rocc[wide][rns_index(T)][nb] : ctx->gocc[gather][rns_index(T)][nb];
  if (o == 0) {
    const void* k =
        gather < 0 ? pc2k::rns_pow_kernel(T, nb, wide) : pc2k::rns_gather_kernel(T, nb, gather);
    int v = 0;
    if (!k)
      o = -1;
    else if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k, pc2k::rns_pow_threads(T, nb, wide),
                                                          0) != hipSuccess || v <= 0)
      o = 1;
    else
      o = v;
  }
  return o < 0 ? 0 : ctx->cus * o;
}
// The powering window: widest that pays for the exponent's length.
int rns_window(const pc2_ctx* ctx, int T) { return ctx->window ? ctx->window : (T > 5 ? 6 : 5); }

// Column blocks per workgroup for `count` elements of nmod moduli: the least
// time by rounds of resident workgroups.
RnsPlan rns_plan_nb(pc2_ctx* ctx, int T, int nmod, size_t count, int nb, int w, int gather = -1,
                    bool wide = false) {
  RnsPlan p;
  p.T = T;
  p.nb = nb;
  p.wide = wide;
  p.w = w;
  p.ngroups = (count + 32 * nb - 1) / (32 * nb);
  p.group_bytes = pc2k::rns_group_bytes(T, nb);
  p.grid = (int)std::min<size_t>(p.ngroups * nmod, (size_t)rns_slots(ctx, T, nb, gather, wide));
  const size_t entries = gather < 0 ? (size_t)1 << (w - 1) : 16;
  p.table_bytes = (size_t)p.grid * entries * p.group_bytes;
  return p;
}
// Time of a product of w workgroups of nb column blocks per CU, in units of what
// a column block adds.  As two sides (T >= 17, wide): 1.1 + nb, one a CU
// (2048-bit n^2, nb 1 .. 4: 16.9 / 24.7 / 33.5 / 41.3 ms; 2048-bit decryption
// halves, wide, nb 2 / 3 / 4: 5.5 / 7.1 / 8.9 ms).  Else 1.2 + w (0.3 + nb)
// (decryption halves, nb 1 .. 4: 4.1 / 5.9 / 7.5 / 9.2 ms one a CU, nb 2 / 4: 9.4 /
// 15.6 ms two a CU).
double rns_round(int T, int nb, bool wide, size_t w) {
  if (w == 0) return 0.0;
  return T >= 17 || wide ? (double)w * (1.1 + nb) : 1.2 + (double)w * (0.3 + nb);
}

// Microseconds of a unit of RnsPlan::cost per bit of the exponent, by tile count:
// at least, with a workgroup on every compute unit, and how steeply it falls from
// there, as the units then stream fewer copies of the constants (decryptions, ms,
// 16 elements / a full device: 1024 bits 1.24 / 7.8 for 65536, 2048: 3.3 / 32 for
// 65536, 3072: 7.3 / 48.5 for 32768, 4096: 13.1 / 88 for 32768; encryptions, 3072
// bits on 129 / 208 / 256 units: 5.3 / 7.6 / 8.1 us, 4096 bits on 129 / 232 /
// 256: 8.4 / 13.1 / 14).
struct RnsUnit { double least, full, drop; };
constexpr RnsUnit RNS_UNIT[pc2k::RNS_NT] = {{0.8, 0.8, -0.17},  {1.30, 1.6, 0.6},
                                            {1.91, 2.75, 1.6},  {3.05, 4.1, 1.85},
                                            {5.0, 8.1, 5.6},    {8.0, 14.0, 11.3}};
double rns_unit(const pc2_ctx* ctx, const RnsPlan& p, int nmod) {
  const RnsUnit u = RNS_UNIT[rns_index(p.T)];
  const double fill = std::min(1.0, (double)(p.ngroups * nmod) / ctx->cus);
  return std::max(u.least, u.full - (1 - fill) * u.drop);
}

// The plan of the least time.  From T = 26 a workgroup's streamed constants weigh
// so much that two column blocks on half of the units beat one on all (8192
// encryptions of 3072 / 4096 bits: 50.5 / 106 against 56.6 / 121 ms).
RnsPlan rns_plan(pc2_ctx* ctx, int T, int nmod, size_t count, int gather = -1) {
  const int w = rns_window(ctx, T);
  RnsPlan best;
  double least = 0;
  for (int k = 2; k <= 2 * pc2k::RNS_NBMAX + 1; ++k) {
    const int nb = k / 2;
    const bool wide = k & 1;
    if (wide && gather >= 0) continue;
    const int slots = rns_slots(ctx, T, nb, gather, wide);
    if (!slots) continue;
    RnsPlan p = rns_plan_nb(ctx, T, nmod, count, nb, w, gather, wide);
    const size_t items = p.ngroups * nmod, occ = (size_t)slots / ctx->cus;
    const size_t full = items / slots, rest = (items % slots + ctx->cus - 1) / ctx->cus;
    p.cost = (double)full * rns_round(T, nb, wide, occ) + rns_round(T, nb, wide, rest);
    const double time = T >= 26 ? p.cost * rns_unit(ctx, p, nmod) : p.cost;
    if (!best.T || time < least) {
      best = p;
      least = time;
    }
  }
  return best;
}

// scratch of the RNS calls: the tables, then the per-chunk staging (256-byte
// aligned parts)
size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }
size_t rns_encrypt_bytes(const RnsPlan& p) { return p.table_bytes + 2 * p.stage_bytes(); }
size_t rns_decrypt_bytes(const RnsPlan& p, size_t chunk, int nl2) {
  return p.table_bytes + 2 * p.stage_bytes() + align256(chunk * 2 * (size_t)(nl2 + 1) * 4);
}
size_t rns_smul_bytes(const RnsPlan& p, size_t chunk) {
  return p.table_bytes + p.stage_bytes() + align256(chunk * 4);
}
size_t rns_encrypt_sk_bytes(const RnsPlan& p, size_t chunk, int nl2) {
  return p.table_bytes + 4 * p.stage_bytes() + align256(chunk * 2 * (size_t)(nl2 + 1) * 4);
}

// Largest scratch any data call under a key of class cls can need: every
// operation and encryption tile, the widest window an option can select,
// a device-filling grid and the largest per-call staging (DEC_CHUNK
// elements).  L: limbs of n; Ls, nl2: limbs of the larger prime and of its
// square.  Also caches every occupancy the calls will look up, so that no
// data call queries the runtime for it (e.g. under graph capture).
size_t class_scratch_need(pc2_ctx* ctx, int cls, int L, int Ls, int nl2) {
  const size_t big = (size_t)1 << 40;  // enough elements to fill the device
  const size_t ch = pc2k::DEC_CHUNK;
  const int w = pc2k::SCHED_WMAX;
  pc2k::Launch l{};
  size_t need = 0;
  auto take = [&](int geo, int op, size_t aux) {
    need = std::max(need, plan_launch(ctx, geo, op, big, Ls, L, w, &l, nullptr, aux));
  };
  take(cls, pc2k::OP_ENC, 0);
  if (pc2k::ALT_GEO[cls] >= 0) take(pc2k::ALT_GEO[cls], pc2k::OP_ENC, 0);
  take(cls, pc2k::OP_SMUL, 0);
  take(cls, pc2k::OP_ENC_MFMA, 0);
  take(cls, pc2k::OP_ENC_TEAM, 0);
  take(cls, pc2k::OP_DEC, ch * 2 * (size_t)(Ls + 1));
  const size_t acc_words =
      std::max(pc2k::chunk_words(cls), pc2k::mfma_digit_bytes(cls) / 4);  // either engine
  const size_t fused_aux =
      ch * 2 * (size_t)L + ch * 2 * (size_t)(Ls + 1) + 128 + ch * (acc_words + 1);
  take(cls, pc2k::OP_DEC, fused_aux);
  take(cls, pc2k::OP_FUSED, fused_aux);
  take(cls, pc2k::OP_FUSED_MFMA, fused_aux);
  take(cls, pc2k::OP_ENC_CRT, ch * 2 * (size_t)(nl2 + 1));
  (void)occupancy(ctx, cls, pc2k::OP_SUM);
  if (cls >= RNS_MIN_CLASS) {  // the RNS engine, any tile count of the class's moduli
    const pc2k::ClassGeo g = pc2k::CLASS_GEO[cls];
    const int tn = pc2h::rns_tiles(64 * L), tp = pc2h::rns_tiles(g.pD * g.pK * g.pT - 2);
    for (int T : pc2k::RNS_T)
      for (int nb = 1; nb <= pc2k::RNS_NBMAX; ++nb) {
        if (T > tn || !rns_slots(ctx, T, nb)) continue;
        (void)rns_slots(ctx, T, nb, -1, true);
        for (int g = 0; g < pc2k::RNS_NGATHER; ++g) (void)rns_slots(ctx, T, nb, g);
        if (rns_slots(ctx, T, nb, pc2k::RNS_SMUL))
          need = std::max(need,
                          rns_smul_bytes(rns_plan_nb(ctx, T, 1, ch, nb, w, pc2k::RNS_SMUL), ch));
        const RnsPlan p = rns_plan_nb(ctx, T, 2, ch, nb, w);
        need = std::max(need, rns_encrypt_bytes(p) + 2 * align256(ch * 8 * (size_t)L));
        if (T <= tp) {
          need = std::max(need, rns_decrypt_bytes(p, ch, nl2) + align256(ch * 8 * (size_t)L));
          need = std::max(need, rns_decrypt_bytes(p, ch, nl2));
          need = std::max(need, rns_encrypt_sk_bytes(p, ch, nl2));
        }
      }
  }
  return need;
}

// Grow the context's scratch to `need` bytes.  Only the key constructors and
// pc2_ctx_reserve call this (never a data call): it waits for the device,
// since work in flight may still use the old buffer.
int grow_scratch(pc2_ctx* ctx, size_t need) {
  if (need <= ctx->scratch_bytes && ctx->scratch) return PC2_OK;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  if (hipDeviceSynchronize() != hipSuccess) return PC2_E_DEVICE;
  if (ctx->scratch) (void)hipFree(ctx->scratch);
  ctx->scratch = nullptr;
  ctx->scratch_bytes = 0;
  ctx->done_valid = false;
  if (hipMalloc(&ctx->scratch, need) != hipSuccess) return PC2_E_NOMEM;
  ctx->scratch_bytes = need;
  return PC2_OK;
}

// Bounds on a private key's prime sizes in class cls: a prime s must satisfy
// 4 s^2 < R of the class's s^2 digit geometry.
void class_prime_limbs(int cls, int* Ls, int* nl2) {
  const pc2k::ClassGeo g = pc2k::CLASS_GEO[cls];
  const int p2bits = g.pD * g.pK * g.pT - 2;
  *nl2 = (p2bits + 31) / 32;
  *Ls = (p2bits / 2 + 31) / 32;
}

bool capturing(void* stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing((hipStream_t)stream, &st) == hipSuccess &&
         st != hipStreamCaptureStatusNone;
}

// Calls that use the context's scratch run one after another whatever their
// streams: a call on a stream other than the previous call's first makes its
// stream wait for that call's completion event (on the device; the host does
// not block), and records the event after its own launches.  Under graph
// capture neither happens: the caller orders a graph's replays against other
// calls on the context.
int scratch_begin(pc2_ctx* ctx, void* stream) {
  if (!ctx->done_valid || ctx->done_stream == stream || capturing(stream)) return PC2_OK;
  return hipStreamWaitEvent((hipStream_t)stream, ctx->done, 0) == hipSuccess ? PC2_OK
                                                                            : PC2_E_DEVICE;
}
int scratch_end(pc2_ctx* ctx, void* stream, int rc) {
  if (rc || capturing(stream)) return rc;
  if (hipEventRecord(ctx->done, (hipStream_t)stream) != hipSuccess) return PC2_E_DEVICE;
  ctx->done_stream = stream;
  ctx->done_valid = true;
  return PC2_OK;
}

int status_of(hipError_t e) { return e == hipSuccess ? PC2_OK : PC2_E_DEVICE; }

// The Montgomery engine of a public-key encryption of `count` elements.  The
// RNS engine needs a device-filling number of elements; below that an element
// with a wavefront of its own finishes sooner (one launch, ms, per-element /
// RNS: 1024 bits, 2048 elements 1.9 / 3.2, 4096: 3.6 / 3.4; 2048 bits, 2048:
// 6.7 / 13.1, 4096: 13.7 / 13.3; 3072 bits, 7168, which fill the device's wavefronts
// once more: 48.3 / 51.4, 7500: 55.4 / 50.4; 4096 bits, 6900: 98 / 105, 7424: 115 /
// 105; 512 bits, 4096: 1.14 / 1.26, 8192: 2.0 /
// 1.34).  256-bit keys stay on the VALU engine once it fills the device (VALU /
// per-element: 4096: 0.62 / 0.40, 16384: 0.68 / 1.46), and so do keys that the
// RNS engine does not take (512 bits, 16384: 2.71 / 4.05; 1024: 9.6 / 11.6).
enum Engine { ENG_VALU, ENG_ELEM, ENG_RNS };
constexpr size_t RNS_MIN_COUNT[pc2k::NUM_CLASSES] = {0, 0, 0, 0, 4097, 3584, 3840, 7169, 7169};
constexpr size_t ELEM_MAX_COUNT[pc2k::NUM_CLASSES] = {0, 0, 0, 4096, 8192, 12288};
Engine enc_engine(const pc2_ctx* ctx, const pc2_pk* pk, size_t count) {
  if (ctx->modmul == PC2_MODMUL_VALU) return ENG_VALU;
  const bool mfma = use_mfma(ctx, pk->cls);
  if (ctx->tile && !mfma) return ENG_VALU;  // a tile asked for is a tile of the VALU engine
  if (pk->rn.T && count >= RNS_MIN_COUNT[pk->cls]) return ENG_RNS;
  return mfma || count <= ELEM_MAX_COUNT[pk->cls] ? ENG_ELEM : ENG_VALU;
}
// The matrix-core encryption of `count` elements by workgroups of several
// wavefronts per element (mfma_team.hpp): while one round of them holds all
// elements.  A second round takes as long as the first, and then a wavefront
// per element is no slower (ms, team / wavefront, at one full round and past
// it: 1024 bits, 512 elements 1.25 / 1.6, 2048 bits, 256: 2.9 / 5.4 and 257: 5.9
// / 5.4, 3072 bits, 256: 5.5 / 11.3).
bool enc_team(pc2_ctx* ctx, int cls, size_t count) {
  int threads;
  return pc2k::kernel_encrypt_team(cls, &threads) &&
         count <= (size_t)ctx->cus * occupancy(ctx, cls, pc2k::OP_ENC_TEAM);
}
// Decryption and key-holder encryption of `count` elements: on the RNS engine at
// any count from 1024-bit keys.  512-bit keys' squares of 512 bits fill half of
// the smallest bases, which pays only while the VALU engine is latency-bound (ms,
// RNS / VALU: decryption, 4096 elements 0.76 / 0.87, 8192 0.98 / 0.88, 65536 4.0 /
// 1.6; key-holder encryption, 4096 1.38 / 1.64, 8192 1.81 / 1.65).
constexpr size_t HALF_RNS_MAX_512 = 5632;
bool half_rns(const pc2_ctx* ctx, const pc2_sk* sk, size_t count) {
  return ctx->modmul != PC2_MODMUL_VALU && (sk->pk.cls > 4 || count <= HALF_RNS_MAX_512);
}
bool dec_rns(const pc2_ctx* ctx, const pc2_sk* sk, size_t count) {
  return sk->dec[0].T && half_rns(ctx, sk, count);
}

pc2k::RnsJobs one_job(const uint32_t* x, const uint32_t* m, int m_limbs, uint32_t* out,
                      size_t count) {
  pc2k::RnsJobs J{};
  J.one = {x, m, out, 0, (uint32_t)count, 0, m_limbs};
  J.n = 1;
  J.npos = (uint32_t)count;
  return J;
}

// The launches of one key's jobs; base: scratch of rns_encrypt_bytes (...)
int rns_encrypt_run(pc2_ctx* ctx, const pc2_pk* pk, const pc2k::RnsJobs& J, const RnsPlan& p,
                    uint8_t* base, void* stream) {
  const pc2k::RnsKey& K = pk->rn;
  pc2k::RnsPow pw{};
  pw.M[0] = K.M;
  pw.ops[0] = K.ops[p.w - pc2k::SCHED_WMIN];
  pw.in[0] = base + p.table_bytes;
  pw.gm[0] = pw.in[0] + p.stage_bytes();
  pw.table = base;
  pw.nmod = 1;
  pw.ngroups = (int)((J.npos + 32 * p.nb - 1) / (32 * p.nb));
  pw.entries = 1 << (p.w - 1);
  hipError_t e = pc2k::launch_rns_to(K.x, K.T, p.nb, J, false, pk->L, pw.in[0], stream);
  if (e == hipSuccess) e = pc2k::launch_rns_to(K.gm, K.T, p.nb, J, true, 0, pw.gm[0], stream);
  if (e == hipSuccess)
    e = pc2k::launch_rns_pow(K.T, p.nb, p.wide, std::min(p.grid, pw.ngroups), pw, stream);
  if (e == hipSuccess)
    e = pc2k::launch_rns_from(K.from, K.T, p.nb, pw.in[0], J, nullptr, 0, stream);
  if (e == hipSuccess)
    e = pc2k::launch_rns_enc_check(pk->c, J, nullptr, 0, ctx->err, stream);
  return status_of(e);
}

// out[i] = c[i]^k[i], at any count (ms, RNS against VALU: 1024 bits, 1 element
// 0.30 / 1.25, 20000: 0.88 / 1.39; 2048 bits, 1: 0.58 / 2.57, 20000: 2.4 / 4.6;
// 4096 bits, 1: 2.05 / 4.9, 20000: 9.4 / 13.4; 512 bits, 1: 0.18 / 0.41, 65536:
// 0.80 / 0.82)
int rns_scalar_mul(const pc2_pk* pk, const uint32_t* c, const uint64_t* k, uint32_t* out,
                   size_t count, void* stream) {
  pc2_ctx* ctx = pk->ctx;
  const pc2k::RnsKey& K = pk->rn;
  const size_t chunk = std::min(count, pc2k::DEC_CHUNK), L2 = 2 * (size_t)pk->L;
  const RnsPlan p = rns_plan(ctx, K.T, 1, chunk, pc2k::RNS_SMUL);
  if (!p.T || !ctx->scratch || rns_smul_bytes(p, chunk) > ctx->scratch_bytes) return PC2_E_NOMEM;
  pc2k::RnsSmul s{};
  s.M = K.M;
  s.one = K.one;
  s.table = reinterpret_cast<uint8_t*>(ctx->scratch);
  s.in = s.table + p.table_bytes;
  uint32_t* bad = reinterpret_cast<uint32_t*>(s.in + p.stage_bytes());
  int rc = scratch_begin(ctx, stream);
  for (size_t at = 0; at < count && !rc; at += chunk) {
    const size_t n = std::min(chunk, count - at);
    const pc2k::RnsJobs J = one_job(c + at * L2, nullptr, 0, out + at * L2, n);
    s.k = k + at;
    s.count = n;
    s.ngroups = (int)((n + 32 * p.nb - 1) / (32 * p.nb));
    hipError_t e = pc2k::launch_rns_to(K.c, K.T, p.nb, J, false, (int)L2, s.in, stream);
    if (e == hipSuccess)
      e = pc2k::launch_rns_row_check(c + at * L2, pk->c.n2.Nl, (int)L2, bad, n, stream);
    if (e == hipSuccess)
      e = pc2k::launch_rns_gather(K.T, p.nb, pc2k::RNS_SMUL, std::min(p.grid, s.ngroups), &s,
                                  stream);
    if (e == hipSuccess) e = pc2k::launch_rns_from(K.from, K.T, p.nb, s.in, J, nullptr, 0, stream);
    if (e == hipSuccess)
      e = pc2k::launch_rns_row_clear(bad, out + at * L2, (int)L2, n, ctx->err, stream);
    rc = status_of(e);
  }
  return scratch_end(ctx, stream, rc);
}

int rns_decrypt_run(pc2_ctx* ctx, const pc2_sk* sk, const pc2k::RnsJobs& J, const RnsPlan& p,
                    uint8_t* base, void* stream) {
  const int T = p.T, nl2 = sk->c.h[0].s2.nl;
  uint8_t* in = base + p.table_bytes;
  uint32_t* ys = reinterpret_cast<uint32_t*>(in + 2 * p.stage_bytes());
  const size_t stride = nl2 + 1;
  pc2k::RnsPow pw{};
  pw.table = base;
  pw.nmod = 2;
  pw.ngroups = (int)((J.npos + 32 * p.nb - 1) / (32 * p.nb));
  pw.entries = 1 << (p.w - 1);
  hipError_t e = hipSuccess;
  for (int i = 0; i < 2 && e == hipSuccess; ++i) {
    pw.M[i] = sk->dec[i].M;
    pw.ops[i] = sk->dec[i].ops[p.w - pc2k::SCHED_WMIN];
    pw.in[i] = in + i * p.stage_bytes();
    e = pc2k::launch_rns_to(sk->dec[i].x, T, p.nb, J, false, 2 * sk->pk.L, pw.in[i], stream);
  }
  if (e == hipSuccess)
    e = pc2k::launch_rns_pow(T, p.nb, p.wide, std::min(p.grid, 2 * pw.ngroups), pw, stream);
  for (int i = 0; i < 2 && e == hipSuccess; ++i)
    e = pc2k::launch_rns_from(sk->dec[i].from, T, p.nb, pw.in[i], J, ys + i * stride, 2 * stride,
                              stream);
  if (e == hipSuccess)
    e = pc2k::launch_rns_dec_finish(sk->c, J, ys, stride, ctx->err, stream);
  return status_of(e);
}

int rns_encrypt_sk_run(pc2_ctx* ctx, const pc2_sk* sk, const pc2k::RnsJobs& J, const RnsPlan& p,
                       uint8_t* base, void* stream) {
  const int T = p.T, nl2 = sk->c.h[0].s2.nl;
  uint8_t* in = base + p.table_bytes;
  uint32_t* stage = reinterpret_cast<uint32_t*>(in + 4 * p.stage_bytes());
  const size_t stride = nl2 + 1;
  pc2k::RnsPow pw{};
  pw.table = base;
  pw.nmod = 2;
  pw.ngroups = (int)((J.npos + 32 * p.nb - 1) / (32 * p.nb));
  pw.entries = 1 << (p.w - 1);
  hipError_t e = hipSuccess;
  for (int i = 0; i < 2 && e == hipSuccess; ++i) {
    pw.M[i] = sk->enc[i].M;
    pw.ops[i] = sk->enc[i].ops[p.w - pc2k::SCHED_WMIN];
    pw.in[i] = in + 2 * i * p.stage_bytes();
    pw.gm[i] = pw.in[i] + p.stage_bytes();
    e = pc2k::launch_rns_to(sk->enc[i].x, T, p.nb, J, false, sk->pk.L, pw.in[i], stream);
    if (e == hipSuccess)
      e = pc2k::launch_rns_to(sk->enc[i].gm, T, p.nb, J, true, 0, pw.gm[i], stream);
  }
  if (e == hipSuccess)
    e = pc2k::launch_rns_pow(T, p.nb, p.wide, std::min(p.grid, 2 * pw.ngroups), pw, stream);
  for (int i = 0; i < 2 && e == hipSuccess; ++i)
    e = pc2k::launch_rns_from(sk->enc[i].from, T, p.nb, pw.in[i], J, stage + i * stride,
                              2 * stride, stream);
  if (e == hipSuccess)
    e = pc2k::launch_rns_enc_check(sk->pk.c, J, stage + nl2, stride, nullptr, stream);
  if (e == hipSuccess) e = pc2k::launch_rns_garner_crt(sk->c, J, stage, ctx->err, stream);
  return status_of(e);
}

// One-call forms in the context's scratch, in chunks of DEC_CHUNK elements.
int rns_encrypt(const pc2_pk* pk, const uint32_t* m, int m_limbs, const uint32_t* r, uint32_t* c,
                size_t count, void* stream) {
  pc2_ctx* ctx = pk->ctx;
  const size_t chunk = std::min(count, pc2k::DEC_CHUNK), L = pk->L;
  const RnsPlan p = rns_plan(ctx, pk->rn.T, 1, chunk);
  if (!ctx->scratch || rns_encrypt_bytes(p) > ctx->scratch_bytes) return PC2_E_NOMEM;
  int rc = scratch_begin(ctx, stream);
  for (size_t b = 0; b < count && !rc; b += chunk)
    rc = rns_encrypt_run(ctx, pk,
                         one_job(r + b * L, m + b * m_limbs, m_limbs, c + b * 2 * L,
                                 std::min(chunk, count - b)),
                         p, reinterpret_cast<uint8_t*>(ctx->scratch), stream);
  return scratch_end(ctx, stream, rc);
}

int rns_decrypt(const pc2_sk* sk, const uint32_t* c, uint32_t* m, size_t count, void* stream) {
  pc2_ctx* ctx = sk->ctx;
  const size_t chunk = std::min(count, pc2k::DEC_CHUNK), L = sk->pk.L;
  const RnsPlan p = rns_plan(ctx, sk->dec[0].T, 2, chunk);
  if (!ctx->scratch ||
      rns_decrypt_bytes(p, chunk, sk->c.h[0].s2.nl) > ctx->scratch_bytes)
    return PC2_E_NOMEM;
  int rc = scratch_begin(ctx, stream);
  for (size_t b = 0; b < count && !rc; b += chunk)
    rc = rns_decrypt_run(
        ctx, sk, one_job(c + b * 2 * L, nullptr, 0, m + b * L, std::min(chunk, count - b)), p,
        reinterpret_cast<uint8_t*>(ctx->scratch), stream);
  return scratch_end(ctx, stream, rc);
}

int rns_encrypt_sk(const pc2_sk* sk, const uint32_t* m, int m_limbs, const uint32_t* r,
                   uint32_t* c, size_t count, void* stream) {
  pc2_ctx* ctx = sk->ctx;
  const size_t chunk = std::min(count, pc2k::DEC_CHUNK), L = sk->pk.L;
  const RnsPlan p = rns_plan(ctx, sk->enc[0].T, 2, chunk);
  if (!ctx->scratch || rns_encrypt_sk_bytes(p, chunk, sk->c.h[0].s2.nl) > ctx->scratch_bytes)
    return PC2_E_NOMEM;
  int rc = scratch_begin(ctx, stream);
  for (size_t b = 0; b < count && !rc; b += chunk)
    rc = rns_encrypt_sk_run(ctx, sk,
                            one_job(r + b * L, m + b * m_limbs, m_limbs, c + b * 2 * L,
                                    std::min(chunk, count - b)),
                            p, reinterpret_cast<uint8_t*>(ctx->scratch), stream);
  return scratch_end(ctx, stream, rc);
}

// The fused path's first phase: prod = prod_k Enc(m_k, r_k), one encryption and
// one aggregation per addend (a bad input's ciphertext is zero, and so is its
// product, which does not decrypt).  stage: prod and one addend's ciphertexts.
int rns_enc_prod(const pc2_sk* sk, const pc2k::PtrList& ms, const pc2k::PtrList& rs, int K,
                 int m_limbs, uint32_t* prod, uint32_t* tmp, size_t n, const RnsPlan& p,
                 uint8_t* base, void* stream) {
  pc2_ctx* ctx = sk->ctx;
  int rc = PC2_OK;
  for (int k = 0; k < K && !rc; ++k) {
    uint32_t* dst = k ? tmp : prod;
    rc = rns_encrypt_run(ctx, &sk->pk, one_job(rs.p[k], ms.p[k], m_limbs, dst, n), p, base,
                         stream);
    if (!rc && k) {
      const uint32_t* two[2] = {prod, tmp};
      rc = pc2_hom_sum(&sk->pk, two, 2, prod, n, stream);
    }
  }
  return rc;
}


// Two device arrays [a, a + na) and [b, b + nb) overlap without being the
// same array of the same size (the only aliasing the data calls accept).
bool partial_overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  if (x + na <= y || y + nb <= x) return false;
  return !(x == y && na == nb);
}

// A job's output against its inputs under the same rule (L: limbs of n).
bool job_overlaps(const pc2_job& j, int L) {
  const size_t n = j.count;
  if (j.op == PC2_OP_ENCRYPT) {
    const size_t cb = 8 * (size_t)L * n;
    return partial_overlap(j.out, cb, j.in0, 4 * (size_t)j.m_limbs * n) ||
           partial_overlap(j.out, cb, j.in1, 4 * (size_t)L * n);
  }
  if (j.op == PC2_OP_DECRYPT) return partial_overlap(j.out, 4 * (size_t)L * n, j.in0, 8 * (size_t)L * n);
  for (uint32_t k = 0; k < j.K; ++k) {  // input k holds lengths[k] rows (ragged) or count
    const size_t rows = j.lengths ? j.lengths[k] : n;
    if (partial_overlap(j.out, 8 * (size_t)L * n, j.inputs[k], 8 * (size_t)L * rows)) return true;
  }
  return false;
}
}  // namespace

// ================================================================ ABI
extern "C" {

const char* pc2_strerror(int status) {
  switch (status) {
    case PC2_OK: return "ok";
    case PC2_E_INVAL: return "invalid argument";
    case PC2_E_RANGE: return "input value out of range";
    case PC2_E_NOMEM: return "out of memory";
    case PC2_E_DEVICE: return "HIP device error";
    case PC2_E_UNSUPPORTED: return "unsupported size or option";
    case PC2_E_BUSY: return "resource busy";
  }
  return "unknown status";
}

int pc2_ctx_create(int hip_device, pc2_ctx** out) {
  if (!out) return PC2_E_INVAL;
  *out = nullptr;
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess || hip_device < 0 || hip_device >= n)
    return PC2_E_DEVICE;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, hip_device) != hipSuccess) return PC2_E_DEVICE;
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return PC2_E_DEVICE;
  if (hipSetDevice(hip_device) != hipSuccess) return PC2_E_DEVICE;
  // the device address of the allocation-free calls' static scratch
  if (pc2k::static_scratch_setup(hip_device) != 0) return PC2_E_DEVICE;
  pc2_ctx* c = new (std::nothrow) pc2_ctx();
  if (!c) return PC2_E_NOMEM;
  c->device = hip_device;
  c->cus = prop.multiProcessorCount;
  if (hipMalloc(&c->err, sizeof(int)) != hipSuccess) {
    delete c;
    return PC2_E_NOMEM;
  }
  if (hipMemset(c->err, 0, sizeof(int)) != hipSuccess ||
      hipEventCreateWithFlags(&c->done, hipEventDisableTiming) != hipSuccess) {
    (void)hipFree(c->err);
    delete c;
    return PC2_E_DEVICE;
  }
  *out = c;
  return PC2_OK;
}

int pc2_ctx_destroy(pc2_ctx* ctx) {
  if (!ctx) return PC2_E_INVAL;
  (void)hipSetDevice(ctx->device);
  (void)hipDeviceSynchronize();
  if (ctx->scratch) (void)hipFree(ctx->scratch);
  if (ctx->err) (void)hipFree(ctx->err);
  if (ctx->done) (void)hipEventDestroy(ctx->done);
  delete ctx;
  return PC2_OK;
}

int pc2_ctx_take_error(pc2_ctx* ctx) {
  if (!ctx) return PC2_E_INVAL;
  int v = 0;
  if (hipMemcpy(&v, ctx->err, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
    return PC2_E_DEVICE;
  if (v && hipMemset(ctx->err, 0, sizeof(int)) != hipSuccess) return PC2_E_DEVICE;
  return (v & pc2k::ERR_RANGE) ? PC2_E_RANGE : PC2_OK;
}

int pc2_ctx_sync(pc2_ctx* ctx, void* hip_stream) {
  if (!ctx) return PC2_E_INVAL;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  if (hipStreamSynchronize((hipStream_t)hip_stream) != hipSuccess) return PC2_E_DEVICE;
  return pc2_ctx_take_error(ctx);
}

int pc2_ctx_reserve(pc2_ctx* ctx, uint32_t max_nbits) {
  if (!ctx) return PC2_E_INVAL;
  const int cls = pc2k::class_for_bits((int)max_nbits);
  if (max_nbits < 2 || cls < 0) return PC2_E_UNSUPPORTED;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  int Ls = 0, nl2 = 0;
  class_prime_limbs(cls, &Ls, &nl2);
  return grow_scratch(ctx, class_scratch_need(ctx, cls, (int)((max_nbits + 31) / 32), Ls, nl2));
}

int pc2_ctx_set_option(pc2_ctx* ctx, int option, int64_t value) {
  if (!ctx) return PC2_E_INVAL;
  if (option == PC2_OPT_WINDOW) {
    if (value != 0 && (value < 2 || value > 6)) return PC2_E_INVAL;
    ctx->window = (int)value;
    return PC2_OK;
  }
  if (option == PC2_OPT_MODMUL) {
    if (value == PC2_MODMUL_VALU || value == PC2_MODMUL_MFMA || value == PC2_MODMUL_AUTO) {
      ctx->modmul = (int)value;
      return PC2_OK;
    }
    return PC2_E_UNSUPPORTED;
  }
  if (option == PC2_OPT_TILE) {
    if (value != 0 && value != PC2_TILE_WIDE && value != 2 && value != 4 && value != 8)
      return PC2_E_INVAL;
    ctx->tile = (int)value;
    return PC2_OK;
  }
  return PC2_E_INVAL;
}

int pc2_ctx_get_option(pc2_ctx* ctx, int option, int64_t* value) {
  if (!ctx || !value) return PC2_E_INVAL;
  if (option == PC2_OPT_WINDOW) *value = ctx->window;
  else if (option == PC2_OPT_MODMUL) *value = ctx->modmul;
  else if (option == PC2_OPT_TILE) *value = ctx->tile;
  else return PC2_E_INVAL;
  return PC2_OK;
}

// ---------------------------------------------------------------- keys
int pc2_pk_create(pc2_ctx* ctx, uint32_t nbits, const uint32_t* n_limbs, pc2_pk** out) {
  if (!ctx || !n_limbs || !out) return PC2_E_INVAL;
  *out = nullptr;
  const int cls = pc2k::class_for_bits((int)nbits);
  if (nbits < 2 || cls < 0) return PC2_E_UNSUPPORTED;
  const int L = (int)((nbits + 31) / 32);
  Limbs n = limbs_from(n_limbs, L);
  const int nb = pc2h::bitlen(n);
  if (nb > (int)nbits || (n[0] & 1u) == 0 || pc2h::cmp(n, Limbs{15}) < 0) return PC2_E_INVAL;
  DevBuf buf;
  PkOffsets o = add_public(buf, n, cls, L);
  const RnsOffsets rn = add_rns_public(buf, n, cls, L);
  pc2_pk* pk = new (std::nothrow) pc2_pk();
  if (!pk) return PC2_E_NOMEM;
  int rc = upload(ctx, buf, &pk->dev);
  if (rc) {
    delete pk;
    return rc;
  }
  pk->ctx = ctx;
  pk->device = ctx->device;
  pk->nbits = nbits;
  pk->L = L;
  pk->cls = cls;
  pk->c = pk_const((const uint32_t*)pk->dev, o, L, nb);
  if (pc2k::ALT_GEO[cls] >= 0) pk->alt = pk_const_alt((const uint32_t*)pk->dev, o, pk->c);
  pk->rn = rns_const((const uint32_t*)pk->dev, rn, 2 * L);
  rc = pc2_ctx_reserve(ctx, nbits);  // every later data call under this key fits
  if (rc) {
    (void)hipFree(pk->dev);
    delete pk;
    return rc;
  }
  *out = pk;
  return PC2_OK;
}

int pc2_sk_create(pc2_ctx* ctx, uint32_t nbits, const uint32_t* p_limbs, const uint32_t* q_limbs,
                  pc2_sk** out) {
  if (!ctx || !p_limbs || !q_limbs || !out) return PC2_E_INVAL;
  *out = nullptr;
  const int cls = pc2k::class_for_bits((int)nbits);
  if (nbits < 2 || cls < 0) return PC2_E_UNSUPPORTED;
  const int L = (int)((nbits + 31) / 32);
  Limbs p = limbs_from(p_limbs, L), q = limbs_from(q_limbs, L);
  if ((p[0] & 1u) == 0 || (q[0] & 1u) == 0 || pc2h::cmp(p, Limbs{3}) < 0 ||
      pc2h::cmp(q, Limbs{3}) < 0 || pc2h::cmp(p, q) == 0)
    return PC2_E_INVAL;
  if (pc2h::cmp(p, q) < 0) std::swap(p, q);  // p > q: m_q < q < p in the recombination
  Limbs n = pc2h::mul(p, q);
  pc2h::trim(n);
  const int nb = pc2h::bitlen(n);
  if (nb > (int)nbits) return PC2_E_INVAL;
  const pc2k::ClassGeo g = pc2k::CLASS_GEO[cls];
  Limbs p2 = pc2h::mul(p, p);
  // the s^2 moduli must satisfy 4 s^2 < R for their digit geometry
  if (pc2h::bitlen(p2) + 2 > g.pD * g.pK * g.pT) return PC2_E_UNSUPPORTED;
  const int Ls = (int)pc2h::resized(p, p.size()).size();
  if (Ls > pc2k::LS_MAX) return PC2_E_UNSUPPORTED;
  const int nl2 = (pc2h::bitlen(p2) + 31) / 32;
  DevBuf buf;
  PkOffsets po = add_public(buf, n, cls, L);
  const RnsOffsets rn = add_rns_public(buf, n, cls, L);
  HalfOffsets hp = add_half(buf, p, q, n, cls, Ls, nl2);
  HalfOffsets hq = add_half(buf, q, p, n, cls, Ls, nl2);
  // q^-1 2^(32 Ls) mod p
  Limbs qinv = pc2h::inv_mod_prime(pc2h::mod(q, p), p);
  size_t qi = buf.add(pc2h::resized(pc2h::shl_mod(qinv, (uint64_t)32 * Ls, p), Ls));
  // (q^2)^-1 2^(32 nl2) mod p^2: q^-2 mod p^2 by Euler (phi(p^2) = p (p - 1))
  Limbs q2 = pc2h::mul(q, q);
  pc2h::trim(q2);
  pc2h::Mont32 MP2(p2);
  Limbs phi = pc2h::mul(p, pc2h::sub(p, Limbs{1}));
  pc2h::trim(phi);
  Limbs q2inv = MP2.pow(pc2h::mod(q2, p2), pc2h::sub(phi, Limbs{1}));
  size_t p2inv = buf.add(pc2h::inv_pow2(p2, nl2));
  size_t q2i = buf.add(pc2h::resized(pc2h::shl_mod(q2inv, (uint64_t)32 * nl2, p2), nl2));
  // the RNS engine modulo p^2 and q^2, each operation on one tile count for both
  // primes, or neither (a modulus that shares a factor with a channel is refused)
  RnsOffsets rd[2], re[2];
  const int rt = rns_tiles_for(cls, p2), rtq = rns_tiles_for(cls, q2);
  if (rt && rtq && rtq <= rt) {
    const Limbs* sq[2] = {&p2, &q2};
    const Limbs* pr[2] = {&p, &q};
    for (int i = 0; i < 2 && (i == 0 || rd[0].T); ++i) {
      const Limbs sm1 = pc2h::sub(*pr[i], Limbs{1});
      Limbs order = pc2h::mul(*pr[i], sm1);
      rd[i] = add_rns(buf, *sq[i], rt, sm1, 4 * L, nullptr, 0, i ? &rd[0] : nullptr);
      if (rd[i].T)
        re[i] = add_rns(buf, *sq[i], rt, pc2h::mod(n, order), 2 * L, &n, 2 * L, &rd[0]);
    }
    if (!rd[1].T) rd[0].T = 0;
    if (!re[0].T || !re[1].T) re[0].T = re[1].T = 0;
  }
  // the key-holder encryption needs r, m < n < 2 q^2, i.e. p < 2 q
  const bool crt_ok = pc2h::cmp(p, pc2h::add(q, q)) < 0;
  pc2_sk* sk = new (std::nothrow) pc2_sk();
  if (!sk) return PC2_E_NOMEM;
  int rc = upload(ctx, buf, &sk->dev);
  if (rc) {
    delete sk;
    return rc;
  }
  const uint32_t* base = (const uint32_t*)sk->dev;
  sk->ctx = ctx;
  sk->pk.ctx = ctx;
  sk->pk.device = ctx->device;
  sk->pk.nbits = nbits;
  sk->pk.L = L;
  sk->pk.cls = cls;
  sk->pk.dev = nullptr;
  sk->pk.c = pk_const(base, po, L, nb);
  if (pc2k::ALT_GEO[cls] >= 0) sk->pk.alt = pk_const_alt(base, po, sk->pk.c);
  sk->c.pk = sk->pk.c;
  sk->c.h[0] = half_const(base, hp);
  sk->c.h[1] = half_const(base, hq);
  sk->c.QI = base + qi;
  sk->c.Q2I = base + q2i;
  sk->c.P2inv = base + p2inv;
  sk->c.p2_n0 = 0u - pc2h::inv32(p2[0]);
  sk->pk.rn = rns_const(base, rn, 2 * L);
  for (int i = 0; i < 2; ++i) {
    sk->dec[i] = rns_const(base, rd[i], nl2);
    sk->enc[i] = rns_const(base, re[i], nl2);
  }
  sk->crt_ok = crt_ok;
  Limbs pm1 = pc2h::sub(p, Limbs{1}), qm1 = pc2h::sub(q, Limbs{1});
  sk->c.ebits = std::max(pc2h::bitlen(pm1), pc2h::bitlen(qm1));
  rc = pc2_ctx_reserve(ctx, nbits);  // every later data call under this key fits
  if (rc) {
    (void)hipFree(sk->dev);
    delete sk;
    return rc;
  }
  *out = sk;
  return PC2_OK;
}

const pc2_pk* pc2_sk_public(const pc2_sk* sk) { return sk ? &sk->pk : nullptr; }

int pc2_pk_destroy(pc2_pk* pk) {
  if (!pk || !pk->ctx) return PC2_E_INVAL;
  if (!pk->dev) return PC2_E_INVAL;  // the public part of a private key
  (void)hipSetDevice(pk->device);  // the context may already be gone
  (void)hipDeviceSynchronize();
  (void)hipFree(pk->dev);
  delete pk;
  return PC2_OK;
}

int pc2_sk_destroy(pc2_sk* sk) {
  if (!sk || !sk->ctx) return PC2_E_INVAL;
  (void)hipSetDevice(sk->pk.device);  // the context may already be gone
  (void)hipDeviceSynchronize();
  (void)hipFree(sk->dev);
  delete sk;
  return PC2_OK;
}

int pc2_pk_info(const pc2_pk* pk, uint32_t* nbits, uint32_t* limbs) {
  if (!pk) return PC2_E_INVAL;
  if (nbits) *nbits = pk->nbits;
  if (limbs) *limbs = (uint32_t)pk->L;
  return PC2_OK;
}

int pc2_pk_context(const pc2_pk* pk, pc2_ctx** ctx, int* hip_device) {
  if (!pk || !pk->ctx) return PC2_E_INVAL;
  if (ctx) *ctx = pk->ctx;
  if (hip_device) *hip_device = pk->ctx->device;
  return PC2_OK;
}

// ---------------------------------------------------------------- data
int pc2_quantize(pc2_ctx* ctx, const pc2_qparams* q, const double* x, uint64_t* m, size_t count,
                 void* stream) {
  if (!ctx || !q) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!x || !m) return PC2_E_INVAL;
  if (partial_overlap(x, 8 * count, m, 8 * count)) return PC2_E_INVAL;
  if (q->log2_scale < -1074 || q->log2_scale > 1023 || q->offset > q->delta) return PC2_E_INVAL;
  pc2k::Launch l{};
  l.grid = (int)std::min<size_t>((count + 255) / 256, (size_t)ctx->cus * 8);
  l.err = ctx->err;
  l.stream = stream;
  return status_of(pc2k::launch_quantize(l, q->log2_scale, q->offset, q->delta, x, m, count));
}

int pc2_dequantize(pc2_ctx* ctx, const pc2_qparams* q, const uint32_t* m, uint32_t m_limbs,
                   uint64_t weight, double* x, size_t count, void* stream) {
  if (!ctx || !q) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!x || !m || m_limbs < 1 || m_limbs > 4096) return PC2_E_INVAL;
  if (partial_overlap(m, 4 * (size_t)m_limbs * count, x, 8 * count)) return PC2_E_INVAL;
  if (q->log2_scale < -1074 || q->log2_scale > 1023) return PC2_E_INVAL;
  pc2k::Launch l{};
  l.grid = (int)std::min<size_t>((count + 255) / 256, (size_t)ctx->cus * 8);
  l.err = ctx->err;
  l.stream = stream;
  return status_of(pc2k::launch_dequantize(l, q->log2_scale, q->offset, m, (int)m_limbs, weight,
                                           x, count));
}

int pc2_encrypt(const pc2_pk* pk, const uint32_t* m, uint32_t m_limbs, const uint32_t* r,
                uint32_t* c, size_t count, void* stream) {
  if (!pk || !pk->ctx) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!m || !r || !c || m_limbs < 1 || (int)m_limbs > pk->L) return PC2_E_INVAL;
  const size_t cb = 8 * (size_t)pk->L * count;
  if (partial_overlap(c, cb, m, 4 * (size_t)m_limbs * count) ||
      partial_overlap(c, cb, r, 4 * (size_t)pk->L * count))
    return PC2_E_INVAL;
  pc2_ctx* ctx = pk->ctx;
  pc2k::Launch l{};
  const Engine eng = enc_engine(ctx, pk, count);
  if (eng == ENG_RNS) return rns_encrypt(pk, m, (int)m_limbs, r, c, count, stream);
  if (eng == ENG_ELEM) {
    const bool team = enc_team(ctx, pk->cls, count);
    int rc = prepare(ctx, pk->cls, team ? pc2k::OP_ENC_TEAM : pc2k::OP_ENC_MFMA, count, 0, pk->L,
                     &l, stream);
    if (!rc) rc = scratch_begin(ctx, stream);
    if (rc) return rc;
    return scratch_end(ctx, stream, status_of(pc2k::launch_encrypt_mfma(
                                        pk->cls, l, pk->c, m, (int)m_limbs, r, c, count, team)));
  }
  const int geo = enc_geo(ctx, pk->cls, count);
  int rc = prepare(ctx, geo, pc2k::OP_ENC, count, 0, pk->L, &l, stream);
  if (!rc) rc = scratch_begin(ctx, stream);
  if (rc) return rc;
  return scratch_end(ctx, stream, status_of(pc2k::launch_encrypt(
                                      geo, l, geo_const(pk, geo), m, (int)m_limbs, r, c, count)));
}

int pc2_decrypt(const pc2_sk* sk, const uint32_t* c, uint32_t* m, size_t count, void* stream) {
  if (!sk || !sk->ctx) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!c || !m) return PC2_E_INVAL;
  if (partial_overlap(c, 8 * (size_t)sk->pk.L * count, m, 4 * (size_t)sk->pk.L * count))
    return PC2_E_INVAL;
  if (dec_rns(sk->ctx, sk, count)) return rns_decrypt(sk, c, m, count, stream);
  // the two CRT halves of up to DEC_CHUNK elements are staged between the
  // per-prime phase and the recombination
  const int Ls = sk->c.h[0].Ls;
  const size_t chunk = std::min(count, pc2k::DEC_CHUNK);
  pc2k::Launch l{};
  int rc = prepare(sk->ctx, sk->pk.cls, pc2k::OP_DEC, chunk, Ls, sk->pk.L, &l, stream,
                   chunk * 2 * (size_t)(Ls + 1));
  if (!rc) rc = scratch_begin(sk->ctx, stream);
  if (rc) return rc;
  const size_t L2 = 2 * (size_t)sk->pk.L;
  for (size_t b = 0; b < count && !rc; b += chunk) {
    const size_t n = std::min(chunk, count - b);
    rc = status_of(pc2k::launch_decrypt(sk->pk.cls, l, sk->c, c + b * L2, m + b * sk->pk.L, n,
                                        l.aux));
  }
  return scratch_end(sk->ctx, stream, rc);
}

// pc2_decrypt with its staging and tables in the static device scratch
// (static_scratch.hip) instead of the context's: nothing is allocated and no
// event is waited for or recorded.
int pc2_decrypt_static(const pc2_sk* sk, const uint32_t* c, uint32_t* m, size_t count,
                       void* stream) {
  if (!sk || !sk->ctx) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!c || !m) return PC2_E_INVAL;
  if (partial_overlap(c, 8 * (size_t)sk->pk.L * count, m, 4 * (size_t)sk->pk.L * count))
    return PC2_E_INVAL;
  uint32_t* base = pc2k::static_scratch(sk->pk.device);
  if (!base) return PC2_E_DEVICE;
  pc2_ctx* ctx = sk->ctx;
  const int Ls = sk->c.h[0].Ls, L = sk->pk.L, cls = sk->pk.cls;
  const size_t total = PC2_STATIC_SCRATCH_BYTES / 4;
  // staging of one chunk's CRT halves: at most an eighth of the array
  const size_t per = 2 * (size_t)(Ls + 1);
  const size_t chunk = std::min({count, pc2k::DEC_CHUNK, total / 8 / per});
  if (chunk == 0) return PC2_E_NOMEM;
  const size_t aux = (chunk * per + 63) & ~(size_t)63;
  const size_t tab_words = total - aux;
  // the widest window up to pc2_decrypt's whose device-filling grid fits;
  // else the narrowest window on as many workgroups as fit
  pc2k::Launch l{};
  int w = window_for(ctx, cls, pc2k::OP_DEC);
  size_t need = 0;
  for (;; --w) {
    need = plan_launch(ctx, cls, pc2k::OP_DEC, chunk, Ls, L, w, &l, stream, 0) / 4;
    if (need <= tab_words || w == pc2k::SCHED_WMIN) break;
  }
  if (need > tab_words) {
    const size_t per_wg = need / (size_t)l.grid;  // tiles x slot words of one workgroup
    const size_t grid = tab_words / per_wg;
    if (grid == 0) return PC2_E_NOMEM;
    l.grid = (int)grid;
  }
  l.aux = base;
  l.scratch = base + aux;
  const size_t L2 = 2 * (size_t)L;
  int rc = PC2_OK;
  for (size_t b = 0; b < count && !rc; b += chunk) {
    const size_t n = std::min(chunk, count - b);
    rc = status_of(pc2k::launch_decrypt(cls, l, sk->c, c + b * L2, m + b * L, n, l.aux));
  }
  return rc;
}

int pc2_encrypt_sk(const pc2_sk* sk, const uint32_t* m, uint32_t m_limbs, const uint32_t* r,
                   uint32_t* c, size_t count, void* stream) {
  if (!sk || !sk->ctx) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!m || !r || !c || m_limbs < 1 || (int)m_limbs > sk->pk.L) return PC2_E_INVAL;
  {
    const size_t cb = 8 * (size_t)sk->pk.L * count;
    if (partial_overlap(c, cb, m, 4 * (size_t)m_limbs * count) ||
        partial_overlap(c, cb, r, 4 * (size_t)sk->pk.L * count))
      return PC2_E_INVAL;
  }
  if (!sk->crt_ok) return PC2_E_UNSUPPORTED;
  if (sk->enc[0].T && half_rns(sk->ctx, sk, count))
    return rns_encrypt_sk(sk, m, (int)m_limbs, r, c, count, stream);
  // the two halves of up to DEC_CHUNK elements are staged before the recombination
  const int nl2 = sk->c.h[0].s2.nl, L = sk->pk.L, cls = sk->pk.cls;
  const size_t chunk = std::min(count, pc2k::DEC_CHUNK);
  pc2k::Launch l{};
  int rc = prepare(sk->ctx, cls, pc2k::OP_ENC_CRT, chunk, sk->c.h[0].Ls, L, &l, stream,
                   chunk * 2 * (size_t)(nl2 + 1));
  if (!rc) rc = scratch_begin(sk->ctx, stream);
  if (rc) return rc;
  for (size_t b = 0; b < count && !rc; b += chunk) {
    const size_t n = std::min(chunk, count - b);
    rc = status_of(pc2k::launch_encrypt_crt(cls, l, sk->c, m + b * m_limbs, (int)m_limbs,
                                            r + b * (size_t)L, c + b * 2 * (size_t)L, n, l.aux));
  }
  return scratch_end(sk->ctx, stream, rc);
}

int pc2_hom_sum(const pc2_pk* pk, const uint32_t* const* c_k, uint32_t K, uint32_t* out,
                size_t count, void* stream) {
  if (!pk || !pk->ctx) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!c_k || !out || K < 1 || K > (uint32_t)pc2k::RK_MAX) return PC2_E_INVAL;
  pc2k::PtrList lst{};
  const size_t cb = 8 * (size_t)pk->L * count;
  for (uint32_t k = 0; k < K; ++k) {
    if (!c_k[k] || partial_overlap(out, cb, c_k[k], cb)) return PC2_E_INVAL;
    lst.p[k] = c_k[k];
  }
  pc2_ctx* ctx = pk->ctx;
  pc2k::Launch l{};
  const size_t epb = (size_t)pc2k::elems_per_block(pk->cls);
  const size_t groups = (count + epb - 1) / epb;
  l.grid = (int)std::max<size_t>(
      1, std::min(groups, (size_t)ctx->cus * occupancy(ctx, pk->cls, pc2k::OP_SUM)));
  l.err = ctx->err;
  l.stream = stream;
  return status_of(pc2k::launch_hom_sum(pk->cls, l, pk->c, lst, (int)K, out, count));
}

int pc2_hom_add(const pc2_pk* pk, const uint32_t* c1, const uint32_t* c2, uint32_t* out,
                size_t count, void* stream) {
  if (!pk) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!c1 || !c2) return PC2_E_INVAL;
  const uint32_t* lst[2] = {c1, c2};
  return pc2_hom_sum(pk, lst, 2, out, count, stream);
}

int pc2_hom_scalar_mul(const pc2_pk* pk, const uint32_t* c, const uint64_t* k, uint32_t* out,
                       size_t count, void* stream) {
  if (!pk || !pk->ctx) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!c || !k || !out) return PC2_E_INVAL;
  {
    const size_t cb = 8 * (size_t)pk->L * count;
    if (partial_overlap(out, cb, c, cb) || partial_overlap(out, cb, k, 8 * count))
      return PC2_E_INVAL;
  }
  if (pk->rn.T && pk->ctx->modmul != PC2_MODMUL_VALU)
    return rns_scalar_mul(pk, c, k, out, count, stream);
  pc2k::Launch l{};
  int rc = prepare(pk->ctx, pk->cls, pc2k::OP_SMUL, count, 0, pk->L, &l, stream);
  if (!rc) rc = scratch_begin(pk->ctx, stream);
  if (rc) return rc;
  return scratch_end(pk->ctx, stream, status_of(pc2k::launch_scalar_mul(
                                          pk->cls, l, pk->c, c, (const uint32_t*)k, out, count)));
}

int pc2_enc_sum_dec(const pc2_sk* sk, const uint32_t* const* m_k, const uint32_t* const* r_k,
                    uint32_t K, uint32_t m_limbs, uint32_t* m_out, size_t count, void* stream) {
  if (!sk || !sk->ctx) return PC2_E_INVAL;
  if (count == 0) return PC2_OK;
  if (!m_k || !r_k || !m_out || K < 1 || K > (uint32_t)pc2k::RK_MAX || m_limbs < 1 ||
      (int)m_limbs > sk->pk.L)
    return PC2_E_INVAL;
  pc2k::PtrList ms{}, rs{};
  for (uint32_t k = 0; k < K; ++k) {
    if (!m_k[k] || !r_k[k]) return PC2_E_INVAL;
    if (partial_overlap(m_out, 4 * (size_t)sk->pk.L * count, m_k[k],
                        4 * (size_t)m_limbs * count) ||
        partial_overlap(m_out, 4 * (size_t)sk->pk.L * count, r_k[k],
                        4 * (size_t)sk->pk.L * count))
      return PC2_E_INVAL;
    ms.p[k] = m_k[k];
    rs.p[k] = r_k[k];
  }
  pc2_ctx* ctx = sk->ctx;
  const int Ls = sk->c.h[0].Ls, L = sk->pk.L, cls = sk->pk.cls;
  const size_t chunk = std::min(count, pc2k::DEC_CHUNK);
  const Engine eng = enc_engine(ctx, &sk->pk, chunk);
  if (eng == ENG_RNS && dec_rns(ctx, sk, chunk)) {
    const size_t cb = align256(chunk * 8 * (size_t)L);
    const RnsPlan pe = rns_plan(ctx, sk->pk.rn.T, 1, chunk);
    const RnsPlan pd = rns_plan(ctx, sk->dec[0].T, 2, chunk);
    if (!ctx->scratch || 2 * cb + rns_encrypt_bytes(pe) > ctx->scratch_bytes ||
        cb + rns_decrypt_bytes(pd, chunk, sk->c.h[0].s2.nl) > ctx->scratch_bytes)
      return PC2_E_NOMEM;
    uint32_t* prod = ctx->scratch;
    uint8_t* rest = reinterpret_cast<uint8_t*>(ctx->scratch) + cb;
    int rc = scratch_begin(ctx, stream);
    for (size_t b = 0; b < count && !rc; b += chunk) {
      const size_t n = std::min(chunk, count - b);
      pc2k::PtrList mb{}, rb{};
      for (uint32_t k = 0; k < K; ++k) {
        mb.p[k] = ms.p[k] + b * m_limbs;
        rb.p[k] = rs.p[k] + b * (size_t)L;
      }
      rc = rns_enc_prod(sk, mb, rb, (int)K, (int)m_limbs, prod,
                        reinterpret_cast<uint32_t*>(rest), n, pe, rest + cb, stream);
      if (!rc)
        rc = rns_decrypt_run(ctx, sk, one_job(prod, nullptr, 0, m_out + b * L, n), pd, rest,
                             stream);
    }
    return scratch_end(ctx, stream, rc);
  }
  // per chunk: the products (2L limbs per element), the CRT halves, the
  // running products (chunked, 16-byte aligned) and the input checks
  const bool mf = eng == ENG_ELEM || (eng == ENG_RNS && use_mfma(ctx, cls));
  const size_t prod_words = (chunk * 2 * (size_t)L + 63) & ~(size_t)63;
  const size_t half_words = (chunk * 2 * (size_t)(Ls + 1) + 63) & ~(size_t)63;
  const size_t acc_words =
      chunk * (mf ? pc2k::mfma_digit_bytes(cls) / 4 : pc2k::chunk_words(cls));
  const size_t aux = prod_words + half_words + acc_words + chunk;
  pc2k::Launch le{}, ld{};
  int rc = prepare(ctx, cls, pc2k::OP_DEC, chunk, Ls, L, &ld, stream, aux);
  if (!rc)
    rc = prepare(ctx, cls, mf ? pc2k::OP_FUSED_MFMA : pc2k::OP_FUSED, chunk, Ls, L, &le, stream,
                 aux);
  if (!rc) rc = scratch_begin(ctx, stream);
  if (rc) return rc;
  uint32_t* prod = le.aux;
  uint32_t* halves = le.aux + prod_words;
  uint32_t* acc = halves + half_words;
  uint32_t* okw = acc + acc_words;
  for (size_t b = 0; b < count && !rc; b += chunk) {
    const size_t n = std::min(chunk, count - b);
    pc2k::PtrList mb{}, rb{};
    for (uint32_t k = 0; k < K; ++k) {
      mb.p[k] = ms.p[k] + b * m_limbs;
      rb.p[k] = rs.p[k] + b * (size_t)L;
    }
    rc = status_of(mf ? pc2k::launch_enc_prod_mfma(cls, le, sk->pk.c, mb, rb, (int)K,
                                                   (int)m_limbs, prod, n,
                                                   reinterpret_cast<uint8_t*>(acc), okw)
                      : pc2k::launch_enc_prod(cls, le, sk->pk.c, mb, rb, (int)K, (int)m_limbs,
                                              prod, n, acc, okw));
    if (!rc)
      rc = status_of(pc2k::launch_decrypt(cls, ld, sk->c, prod, m_out + b * L, n, halves));
  }
  return scratch_end(ctx, stream, rc);
}

// ---------------------------------------------------------------- batches
namespace {
// Positions of a part's jobs: each from the next multiple of 32.
uint32_t round32(uint32_t v) { return (v + 31) & ~31u; }

// A part holds at most RNS_PART positions, and a key's jobs are cut into as many
// parts as they need, which share one scratch: a launch's staging (2.2 KB a
// position at 2048 bits) stays bounded whatever its jobs' lengths.
constexpr uint32_t RNS_PART = (uint32_t)pc2k::DEC_CHUNK;

// The jobs of one key in a launch.
struct KeyJobs {
  const pc2_pk* pk = nullptr;
  const pc2_sk* sk = nullptr;
  std::vector<size_t> jobs;
  size_t total = 0;
  bool takes = false;  // the RNS engine takes them (enc_engine, dec_rns)
  bool only = false;   // ... and the persistent kernels have none for the key's class
  bool rns = false;
};
int key_ebits(const KeyJobs& k) { return k.sk ? k.sk->c.ebits : (int)k.pk->nbits; }

// Estimates in microseconds per bit of the exponents for the choice between the
// engines where a launch holds several keys (rns_choose).  On residues every key
// is a launch sequence of its own, however few its elements (rns_unit).
double rns_time(const pc2_ctx* ctx, const RnsPlan& p, int nmod, int ebits) {
  return p.cost * rns_unit(ctx, p, nmod) * ebits;
}
// The persistent kernels run all keys of a launch together: no sooner than one
// element's chain of products, and than the device does the products of all, on
// the VALU in rounds of as many elements as it holds (`round`).  Measured, ms, few
// elements / a device-filling number of them: VALU decryption 1024 bits 4.7 / 5.7
// for 32768 and 9.7 for 65536, 2048: 16.4 / 17.5 for 16384 and 58.5 for 65536,
// 3072: 31 / 100.8 for 32768, 4096: 72 / 232.7 for 32768; VALU encryption 1024: 17 /
// 30.3 for 65536; per-element encryption 1024: 1.5 / 0.0007 an element, 2048: 5.2 /
// 0.0028, 3072: 9.5 / 0.0066, 4096: 19.4 / 0.0135.
struct PersistentUnit { double chain, each, round; };
constexpr PersistentUnit VALU_DEC[4] = {{9.2, 0.00027, 32768}, {16.0, 0.00086, 16384},
                                        {20.2, 0.0020, 8192}, {35.2, 0.0034, 8192}};
constexpr PersistentUnit VALU_ENC_1024 = {16.6, 0.00045, 32768};
constexpr PersistentUnit ELEM_ENC[4] = {{1.46, 0.00069, 1}, {2.56, 0.00135, 1},
                                        {3.10, 0.00216, 1}, {4.74, 0.00329, 1}};
PersistentUnit persistent_unit(const pc2_ctx* ctx, int op, int cls) {
  // (smaller keys stay in the persistent kernels whatever is chosen for the others)
  if (cls < 5) return {0, 0, 1};
  if (op == pc2k::OP_DEC) return VALU_DEC[cls - 5];
  return use_mfma(ctx, cls) ? ELEM_ENC[cls - 5] : VALU_ENC_1024;
}

// Which keys of a launch run on residues: the one key of a launch of its own
// whenever the engine takes it, else those of the most elements, as many as
// make the launch's estimated time the least (decryption batches, 2048 bits, 16
// elements a key, 4 / 8 / 16 keys: 13.4 / 26.9 / 53.7 ms as sequences, 16.5 in the
// persistent kernel; encryptions of 3840 elements, 4 keys: 53.8 against 45.7).
void rns_choose(pc2_ctx* ctx, int op, std::vector<KeyJobs>& keys) {
  size_t open = 0;
  for (KeyJobs& k : keys) {
    k.rns = k.only;
    open += !k.only;
  }
  if (open <= 1) {
    for (KeyJobs& k : keys) k.rns = k.takes;
    return;
  }
  const int nmod = op == pc2k::OP_DEC ? 2 : 1;
  struct Load { double chain = 0, each = 0, round = 1; size_t keys = 0; } load[pc2k::NUM_CLASSES];
  auto load_of = [&](const KeyJobs& k) -> Load& { return load[k.sk ? k.sk->pk.cls : k.pk->cls]; };
  std::vector<size_t> order;
  for (size_t i = 0; i < keys.size(); ++i) {
    const KeyJobs& k = keys[i];
    if (k.only) continue;
    const int cls = k.sk ? k.sk->pk.cls : k.pk->cls;
    const PersistentUnit u = persistent_unit(ctx, op, cls);
    load_of(k).chain = std::max(load_of(k).chain, u.chain * key_ebits(k));
    load_of(k).each += u.each * key_ebits(k) * (double)k.total;
    load_of(k).round = std::max(load_of(k).round, u.each * key_ebits(k) * u.round);
    ++load_of(k).keys;
    if (k.takes) order.push_back(i);
  }
  // the VALU classes in one launch (two fill each other's last round), each class
  // on the matrix cores in its own
  auto persistent = [&] {
    double chain = 0, each = 0, round = 0, elem = 0;
    int classes = 0;
    for (int c = 0; c < pc2k::NUM_CLASSES; ++c) {
      if (!load[c].keys) continue;
      if (op == pc2k::OP_ENC && use_mfma(ctx, c)) {
        elem += std::max(load[c].chain, load[c].each);
      } else {
        chain = std::max(chain, load[c].chain);
        each += load[c].each;
        round = load[c].round;
        ++classes;
      }
    }
    if (classes == 1) each = std::ceil(each / round - 1e-9) * round;
    return std::max(chain, each) + elem;
  };
  std::stable_sort(order.begin(), order.end(),
                   [&](size_t a, size_t b) { return keys[a].total > keys[b].total; });
  double best = persistent(), rns = 0;
  size_t take = 0;
  for (size_t m = 0; m < order.size(); ++m) {
    const KeyJobs& k = keys[order[m]];
    const int T = op == pc2k::OP_DEC ? k.sk->dec[0].T : k.pk->rn.T;
    const PersistentUnit u = persistent_unit(ctx, op, k.sk ? k.sk->pk.cls : k.pk->cls);
    rns += rns_time(ctx, rns_plan(ctx, T, nmod, k.total), nmod, key_ebits(k));
    load_of(k).each -= u.each * key_ebits(k) * (double)k.total;
    --load_of(k).keys;
    const double time = rns + persistent();
    if (time < best) {
      best = time;
      take = m + 1;
    }
  }
  for (size_t m = 0; m < take; ++m) keys[order[m]].rns = true;
}

// The jobs that the RNS engine takes, by key: count[i] elements from element
// first[i] of job i.  in_rns[i] tells which; hjobs receives their descriptors
// (part after part, jobs.many holding an index until rns_parts_place).
std::vector<RnsPart> rns_parts(pc2_ctx* ctx, int op, const pc2_job* jobs, const size_t* first,
                               const size_t* count, size_t njobs, std::vector<bool>* in_rns,
                               std::vector<pc2k::RnsJob>* hjobs) {
  std::vector<RnsPart> parts;
  in_rns->assign(njobs, false);
  if (op != pc2k::OP_ENC && op != pc2k::OP_DEC) return parts;
  const bool dec = op == pc2k::OP_DEC;
  std::vector<KeyJobs> keys;  // by first appearance
  std::unordered_map<const void*, size_t> at;
  for (size_t i = 0; i < njobs; ++i) {
    if (count[i] == 0) continue;
    const void* key = dec ? (const void*)jobs[i].sk : (const void*)jobs[i].pk;
    const auto ins = at.emplace(key, keys.size());
    if (ins.second) {
      keys.emplace_back();
      keys.back().pk = dec ? nullptr : jobs[i].pk;
      keys.back().sk = dec ? jobs[i].sk : nullptr;
    }
    KeyJobs& k = keys[ins.first->second];
    k.jobs.push_back(i);
    k.total += count[i];
  }
  for (KeyJobs& k : keys) {
    k.takes = dec ? dec_rns(ctx, k.sk, k.total) : enc_engine(ctx, k.pk, k.total) == ENG_RNS;
    k.only = k.takes &&
             pc2k::batch_group_elems(op, job_geo(ctx, dec ? &k.sk->pk : k.pk, op)) == 0;
  }
  rns_choose(ctx, op, keys);
  for (const KeyJobs& k : keys) {
    if (!k.rns) continue;
    RnsPart p;
    size_t from = 0;
    uint32_t pos = 0;
    auto start = [&] {
      p = RnsPart();
      p.pk = k.pk;
      p.sk = k.sk;
      from = hjobs->size();
      pos = 0;
    };
    auto close = [&] {
      p.jobs.n = (int)(hjobs->size() - from);
      p.jobs.many = reinterpret_cast<const pc2k::RnsJob*>(from * sizeof(pc2k::RnsJob));
      p.jobs.npos = pos;
      p.plan = rns_plan(ctx, dec ? k.sk->dec[0].T : k.pk->rn.T, dec ? 2 : 1, pos);
      parts.push_back(p);
    };
    start();
    for (size_t i : k.jobs) {
      const pc2_job& j = jobs[i];
      (*in_rns)[i] = true;
      for (size_t done = 0; done < count[i];) {
        if (round32(pos) >= RNS_PART) {
          close();
          start();
        }
        pos = round32(pos);
        const size_t n = std::min<size_t>(count[i] - done, RNS_PART - pos);
        hjobs->push_back({dec ? j.in0 : j.in1, dec ? nullptr : j.in0, j.out, first[i] + done,
                          (uint32_t)n, pos, (int)j.m_limbs});
        pos += (uint32_t)n;
        done += n;
      }
    }
    close();
  }
  return parts;
}
// Two parts that together have no more workgroups than there are compute units
// run side by side, each on units of its own, with the column blocks per
// workgroup that make the later of the two earliest: a part of few groups would
// leave most of the device idle.  (A product's time goes with T, the products
// with T.  6100 elements of a 2048-bit key and 8000 of a 1024-bit key, ms: one
// after the other 15.7 + 4.5, beside each other with the plans of either
// alone 18.6, with the second in 63 workgroups 15.9.)
void rns_parts_pair(pc2_ctx* ctx, std::vector<RnsPart>& parts, int nmod) {
  if (parts.size() != 2) return;
  RnsPlan best[2];
  double best_time = 0, serial = 0;
  for (const RnsPart& p : parts) serial += p.plan.cost * p.plan.T * p.plan.T;
  for (int n0 = 1; n0 <= pc2k::RNS_NBMAX; ++n0)
    for (int n1 = 1; n1 <= pc2k::RNS_NBMAX; ++n1) {
      const int nb[2] = {n0, n1};
      RnsPlan p[2];
      double time = 0;
      size_t groups = 0;
      for (int i = 0; i < 2; ++i) {
        const int T = parts[i].plan.T;
        if (!rns_slots(ctx, T, nb[i])) break;
        const bool wide = rns_slots(ctx, T, nb[i], -1, true) > 0;
        p[i] = rns_plan_nb(ctx, T, nmod, parts[i].jobs.npos, nb[i], parts[i].plan.w, -1, wide);
        groups += p[i].ngroups * nmod;
        time = std::max(time, rns_round(T, nb[i], wide, 1) * T * T);
      }
      if (!p[1].T || groups > (size_t)ctx->cus) continue;
      if (best_time == 0 || time < best_time) {
        best_time = time;
        best[0] = p[0];
        best[1] = p[1];
      }
    }
  if (best_time == 0 || best_time > 0.95 * serial) return;
  for (int i = 0; i < 2; ++i) parts[i].plan = best[i];
  parts[1].side = true;
}
void rns_parts_place(std::vector<RnsPart>& parts, const void* dev) {
  for (RnsPart& p : parts)
    p.jobs.many = reinterpret_cast<const pc2k::RnsJob*>((const char*)dev +
                                                        (size_t)p.jobs.many);
}
// A class whose (only) encryption jobs outside the RNS engine would run on the
// VALU engine, but are few enough for an element a wavefront (enc_engine's
// rule); -1: none.
int few_elements_class(const pc2_ctx* ctx, int op, const pc2_job* jobs, const size_t* count,
                       size_t njobs, const std::vector<bool>& in_rns) {
  if (op != pc2k::OP_ENC || ctx->modmul != PC2_MODMUL_AUTO || ctx->tile) return -1;
  int cls = -1;
  size_t total = 0;
  for (size_t i = 0; i < njobs; ++i) {
    if (count[i] == 0 || in_rns[i] || use_mfma(ctx, jobs[i].pk->cls)) continue;
    if (cls >= 0 && cls != jobs[i].pk->cls) return -1;
    cls = jobs[i].pk->cls;
    total += count[i];
  }
  return cls >= 0 && total <= ELEM_MAX_COUNT[cls] ? cls : -1;
}
size_t rns_part_bytes(const RnsPart& p, int op) {
  return op == pc2k::OP_DEC
             ? rns_decrypt_bytes(p.plan, p.jobs.npos, p.sk->c.h[0].s2.nl)
             : rns_encrypt_bytes(p.plan);
}
int rns_part_run(pc2_ctx* ctx, const RnsPart& p, int op, uint8_t* scratch, void* stream) {
  return op == pc2k::OP_DEC ? rns_decrypt_run(ctx, p.sk, p.jobs, p.plan, scratch, stream)
                            : rns_encrypt_run(ctx, p.pk, p.jobs, p.plan, scratch, stream);
}
}  // namespace

// Work-queue counters at the end of a batch's or runner's descriptor
// allocation: the VALU launch's, then one per matrix-core class, each on
// its own 128-byte line.
constexpr int QUEUE_STRIDE = 32;                 // ints between two counters
constexpr size_t QUEUE_BYTES = 3 * QUEUE_STRIDE * sizeof(int);
// resident workgroups per CU of a 64-lane kernel (1 if the runtime cannot tell)
int occupancy_of(const void* k) {
  int occ = 0;
  if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, 64, 0) != hipSuccess ||
      occ <= 0)
    occ = 1;
  return occ;
}

static void batch_rns_free(pc2_batch* b) {
  if (b->rscratch) (void)hipFree(b->rscratch);
  if (b->rscratch2) (void)hipFree(b->rscratch2);
  if (b->forked) (void)hipEventDestroy(b->forked);
  if (b->joined) (void)hipEventDestroy(b->joined);
  if (b->side) (void)hipStreamDestroy(b->side);
  b->rscratch = b->rscratch2 = nullptr;
  b->forked = b->joined = nullptr;
  b->side = nullptr;
}
static void batch_free(pc2_batch* b) {
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->dev) (void)hipFree(b->dev);
  if (b->scratch) (void)hipFree(b->scratch);
  if (b->mscratch) (void)hipFree(b->mscratch);
  if (b->stage) (void)hipFree(b->stage);
  batch_rns_free(b);
  delete b;
}

// What a batch's parts on the RNS engine run in; false if the device has no
// memory for it (the jobs then stay on the persistent kernels).
static bool batch_rns_alloc(pc2_batch* b, pc2_ctx* ctx, int op) {
  rns_parts_pair(ctx, b->rparts, op == pc2k::OP_DEC ? 2 : 1);
  size_t bytes[2] = {0, 0};
  for (const RnsPart& p : b->rparts)
    bytes[p.side] = std::max(bytes[p.side], rns_part_bytes(p, op));
  if (hipSetDevice(ctx->device) == hipSuccess &&
      hipMalloc(&b->rscratch, bytes[0]) == hipSuccess &&
      (!bytes[1] ||
       (hipMalloc(&b->rscratch2, bytes[1]) == hipSuccess &&
        hipStreamCreateWithFlags(&b->side, hipStreamNonBlocking) == hipSuccess &&
        hipEventCreateWithFlags(&b->forked, hipEventDisableTiming) == hipSuccess &&
        hipEventCreateWithFlags(&b->joined, hipEventDisableTiming) == hipSuccess)))
    return true;
  (void)hipGetLastError();
  batch_rns_free(b);
  return false;
}

int pc2_batch_create(pc2_ctx* ctx, const pc2_job* jobs, size_t njobs, pc2_batch** out) {
  if (!ctx || !jobs || !out || njobs == 0) return PC2_E_INVAL;
  *out = nullptr;
  const int op_abi = jobs[0].op;
  int op;
  if (op_abi == PC2_OP_ENCRYPT) op = pc2k::OP_ENC;
  else if (op_abi == PC2_OP_DECRYPT) op = pc2k::OP_DEC;
  else if (op_abi == PC2_OP_HOM_SUM) op = pc2k::OP_SUM;
  else return PC2_E_INVAL;
  // validate and collect classes: the VALU kernel's pair, and the (up to
  // two) classes whose encryptions run on the matrix cores (use_mfma)
  int ca = -1, cb = -1, mca = -1, mcb = -1, Ls = 0;
  for (size_t i = 0; i < njobs; ++i) {
    const pc2_job& j = jobs[i];
    if (j.op != op_abi) return PC2_E_INVAL;
    if (j.count == 0) continue;
    const pc2_pk* pk = (op == pc2k::OP_DEC) ? (j.sk ? &j.sk->pk : nullptr) : j.pk;
    if (!pk || pk->ctx != ctx || !j.out) return PC2_E_INVAL;
    if (op == pc2k::OP_ENC &&
        (!j.in0 || !j.in1 || j.m_limbs < 1 || (int)j.m_limbs > pk->L))
      return PC2_E_INVAL;
    if (op == pc2k::OP_DEC && !j.in0) return PC2_E_INVAL;
    if (op == pc2k::OP_SUM) {
      if (!j.inputs || j.K < 1 || j.K > (uint32_t)pc2k::RK_MAX) return PC2_E_INVAL;
      for (uint32_t k = 0; k < j.K; ++k)
        if (!j.inputs[k] || (j.lengths && j.lengths[k] > j.count)) return PC2_E_INVAL;
    }
    if (job_overlaps(j, pk->L)) return PC2_E_INVAL;
    if (op == pc2k::OP_DEC) Ls = std::max(Ls, j.sk->c.h[0].Ls);
    if (op == pc2k::OP_ENC && use_mfma(ctx, pk->cls)) {
      if (mca < 0 || mca == pk->cls) mca = pk->cls;
      else if (mcb < 0 || mcb == pk->cls) mcb = pk->cls;
      else return PC2_E_UNSUPPORTED;
      continue;
    }
    const int g = job_geo(ctx, pk, op);
    if (ca < 0 || ca == g) ca = g;
    else if (cb < 0 || cb == g) cb = g;
    else return PC2_E_UNSUPPORTED;
  }
  if (ca < 0 && mca < 0) return PC2_E_INVAL;  // every job empty
  if (mca >= 0 && mcb > mca) std::swap(mca, mcb);  // the more expensive class first
  int pair = -1, pa = -1, pb = -1;
  if (ca >= 0) {
    if (cb < 0) cb = ca;
    pair = pc2k::batch_pair(ca, cb);
    if (pair < 0) return PC2_E_UNSUPPORTED;
    pa = pc2k::batch_pair_geo(pair, 0);
    pb = pc2k::batch_pair_geo(pair, 1);
  }
  pc2_batch* b = new (std::nothrow) pc2_batch();
  if (!b) return PC2_E_NOMEM;
  std::vector<size_t> zero(njobs, 0), counts(njobs);
  for (size_t i = 0; i < njobs; ++i) counts[i] = jobs[i].count;
  std::vector<bool> in_rns;
  std::vector<pc2k::RnsJob> rjobs;
  b->rparts = rns_parts(ctx, op, jobs, zero.data(), counts.data(), njobs, &in_rns, &rjobs);
  bool lost = false;
  if (!b->rparts.empty() && !batch_rns_alloc(b, ctx, op)) {
    b->rparts.clear();
    rjobs.clear();
    in_rns.assign(njobs, false);
    lost = true;
  }
  for (size_t i = 0; i < njobs; ++i) {  // a class that no persistent kernel has
    if (jobs[i].count == 0 || in_rns[i]) continue;
    const pc2_pk* pk = (op == pc2k::OP_DEC) ? &jobs[i].sk->pk : jobs[i].pk;
    if (pc2k::batch_group_elems(op, job_geo(ctx, pk, op)) > 0) continue;
    batch_free(b);
    return lost ? PC2_E_NOMEM : PC2_E_UNSUPPORTED;
  }
  const int few = few_elements_class(ctx, op, jobs, counts.data(), njobs, in_rns);
  if (few >= 0 && mcb < 0) {
    (mca < 0 ? mca : mcb) = few;
    if (mcb > mca) std::swap(mca, mcb);
    pair = -1;
  }
  b->ctx = ctx;
  b->op = op;
  b->pair = pair;
  if (pair >= 0) {
    b->w_a = window_for(ctx, pa, op);
    b->w_b = window_for(ctx, pb, op);
  }
  b->mp[0].cls = mca;
  b->mp[1].cls = mcb;
  for (auto& m : b->mp)
    if (m.cls >= 0) m.w = window_for(ctx, m.cls, pc2k::OP_ENC_MFMA);
  // descriptors and items (most expensive class first)
  std::vector<pc2k::BatchJob> dj;
  std::vector<pc2k::BatchItem> items;
  std::vector<size_t> ptrbuf;  // per hom_sum job: K pointers then K lengths
  std::vector<size_t> ptr_off;
  std::vector<bool> mjob;      // runs on the matrix cores
  for (size_t i = 0; i < njobs; ++i) {
    const pc2_job& j = jobs[i];
    if (j.count == 0 || in_rns[i]) continue;
    pc2k::BatchJob d{};
    const pc2_pk* pk = (op == pc2k::OP_DEC) ? &j.sk->pk : j.pk;
    const bool mf = op == pc2k::OP_ENC && (pk->cls == mca || pk->cls == mcb);
    d.geo = mf ? pk->cls : job_geo(ctx, pk, op);
    d.group = pc2k::batch_group_elems(op, job_geo(ctx, pk, op));
    d.op = op;
    d.m_limbs = (int)j.m_limbs;
    d.K = (int)j.K;
    d.pk = mf ? pk->c : geo_const(pk, d.geo);
    mjob.push_back(mf);
    if (op == pc2k::OP_DEC) d.sk = j.sk->c;
    d.in0 = j.in0;
    d.in1 = j.in1;
    d.out = j.out;
    d.count = j.count;
    size_t off = ptrbuf.size();
    if (op == pc2k::OP_SUM) {
      for (uint32_t k = 0; k < j.K; ++k) ptrbuf.push_back((size_t)j.inputs[k]);
      for (uint32_t k = 0; k < j.K; ++k) ptrbuf.push_back(j.lengths ? j.lengths[k] : j.count);
    }
    ptr_off.push_back(off);
    dj.push_back(d);
  }
  for (int pass = 0; pair >= 0 && pass < 2; ++pass) {
    const int first_geo = pc2k::GEO_CLASS[pa] >= pc2k::GEO_CLASS[pb] ? pa : pb;
    const int want = pass == 0 ? first_geo : (first_geo == pa ? pb : pa);
    if (pass == 1 && pa == pb) break;
    for (size_t ji = 0; ji < dj.size(); ++ji) {
      if (mjob[ji] || dj[ji].geo != want) continue;
      const size_t epw = (size_t)pc2k::batch_group_elems(op, dj[ji].geo);
      const size_t groups = (dj[ji].count + epw - 1) / epw;
      for (size_t g = 0; g < groups; ++g) {
        items.push_back(pc2k::BatchItem{(int)ji, 0, g});
        if (op == pc2k::OP_DEC) items.push_back(pc2k::BatchItem{(int)ji, 1, g});
      }
    }
  }
  b->nitems = (int)items.size();
  std::vector<size_t> mfirst(2, 0);
  for (int part = 0; part < 2; ++part) {  // matrix-core items after the others, per class
    mfirst[part] = items.size();
    for (size_t ji = 0; ji < dj.size(); ++ji) {
      if (!mjob[ji] || b->mp[part].cls < 0 || dj[ji].geo != b->mp[part].cls) continue;
      b->mp[part].sub = std::max(b->mp[part].sub, dj[ji].group);
      const size_t groups = (dj[ji].count + dj[ji].group - 1) / dj[ji].group;
      for (size_t g = 0; g < groups; ++g) items.push_back(pc2k::BatchItem{(int)ji, 0, g});
    }
    b->mp[part].nitems = (int)(items.size() - mfirst[part]);
  }
  // decryption: staging for the two CRT halves of every element
  std::vector<size_t> stage_off(dj.size(), 0);
  size_t stage_words = 0;
  if (op == pc2k::OP_DEC) {
    for (size_t ji = 0; ji < dj.size(); ++ji) {
      const size_t epw = (size_t)pc2k::batch_group_elems(op, dj[ji].geo);
      stage_off[ji] = stage_words;
      stage_words += (dj[ji].count + epw - 1) / epw * epw * 2 * (size_t)(dj[ji].sk.h[0].Ls + 1);
    }
  }
  // one device allocation: jobs | items | pointer/length arrays | queue
  const size_t jobs_b = (dj.size() * sizeof(pc2k::BatchJob) + 255) & ~(size_t)255;
  const size_t items_b = (items.size() * sizeof(pc2k::BatchItem) + 255) & ~(size_t)255;
  const size_t ptr_b = (ptrbuf.size() * sizeof(size_t) + 255) & ~(size_t)255;
  const size_t rjobs_b = (rjobs.size() * sizeof(pc2k::RnsJob) + 255) & ~(size_t)255;
  const size_t total = jobs_b + items_b + ptr_b + QUEUE_BYTES + rjobs_b;
  int rc = PC2_OK;
  if (hipSetDevice(ctx->device) != hipSuccess) rc = PC2_E_DEVICE;
  if (!rc && hipMalloc(&b->dev, total) != hipSuccess) rc = PC2_E_NOMEM;
  if (!rc && stage_words && hipMalloc(&b->stage, stage_words * 4) != hipSuccess)
    rc = PC2_E_NOMEM;
  if (!rc && stage_words)
    for (size_t ji = 0; ji < dj.size(); ++ji) {
      dj[ji].stage = b->stage + stage_off[ji];
      dj[ji].stage_g0 = 0;
    }
  if (!rc) {
    char* base = (char*)b->dev;
    b->jobs = (pc2k::BatchJob*)base;
    b->items = (pc2k::BatchItem*)(base + jobs_b);
    size_t* dptr = (size_t*)(base + jobs_b + items_b);
    b->queue = (int*)(base + jobs_b + items_b + ptr_b);
    for (int part = 0; part < 2; ++part) {
      b->mp[part].items = b->items + mfirst[part];
      b->mp[part].queue = b->queue + QUEUE_STRIDE * (part + 1);
    }
    for (size_t ji = 0; ji < dj.size(); ++ji)
      if (op == pc2k::OP_SUM) {
        dj[ji].inputs = (const uint32_t* const*)(dptr + ptr_off[ji]);
        dj[ji].lengths = dptr + ptr_off[ji] + dj[ji].K;
      }
    void* rdev = base + jobs_b + items_b + ptr_b + QUEUE_BYTES;
    rns_parts_place(b->rparts, rdev);
    if ((!dj.empty() && hipMemcpy(b->jobs, dj.data(), dj.size() * sizeof(pc2k::BatchJob),
                                  hipMemcpyHostToDevice) != hipSuccess) ||
        (!items.empty() && hipMemcpy(b->items, items.data(),
                                     items.size() * sizeof(pc2k::BatchItem),
                                     hipMemcpyHostToDevice) != hipSuccess) ||
        (!rjobs.empty() && hipMemcpy(rdev, rjobs.data(), rjobs.size() * sizeof(pc2k::RnsJob),
                                     hipMemcpyHostToDevice) != hipSuccess) ||
        (!ptrbuf.empty() && hipMemcpy(dptr, ptrbuf.data(), ptrbuf.size() * sizeof(size_t),
                                      hipMemcpyHostToDevice) != hipSuccess))
      rc = PC2_E_DEVICE;
  }
  // grids and the batch's own scratch
  size_t mbytes = 0;
  for (auto& m : b->mp) {
    if (rc || !m.nitems) continue;
    m.grid = std::max<int>(
        1, (int)std::min<size_t>((size_t)ctx->cus * occupancy_of(pc2k::batch_mfma_kernel(m.cls)),
                                 (size_t)m.nitems * m.sub));
    mbytes = std::max(mbytes, (size_t)m.grid * (pc2k::mfma_digit_bytes(m.cls) << m.w));
  }
  if (!rc && mbytes && hipMalloc(&b->mscratch, mbytes) != hipSuccess) rc = PC2_E_NOMEM;
  if (!rc && b->nitems) {
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, pc2k::batch_kernel(op, pair), 64, 0) !=
            hipSuccess ||
        occ <= 0)
      occ = 1;
    b->grid = std::max(1, std::min(ctx->cus * occ, b->nitems));
    int ta = 0, tb = 0;
    size_t wa = 0, wb = 0;
    pc2k::batch_slot_shape(op, pa, b->w_a, Ls, &ta, &wa);
    pc2k::batch_slot_shape(op, pb, b->w_b, Ls, &tb, &wb);
    const int tiles = std::max(ta, tb);
    b->slot_words = (std::max(wa, wb) + 3) & ~(size_t)3;
    const size_t bytes = (size_t)b->grid * tiles * b->slot_words * 4;
    if (bytes && hipMalloc(&b->scratch, bytes) != hipSuccess) rc = PC2_E_NOMEM;
  }
  if (rc) {
    batch_free(b);
    return rc;
  }
  *out = b;
  return PC2_OK;
}

int pc2_batch_run(pc2_batch* b, void* hip_stream) {
  if (!b || !b->ctx) return PC2_E_INVAL;
  if (hipSetDevice(b->ctx->device) != hipSuccess) return PC2_E_DEVICE;
  auto launch = [&](void* st) {
    hipError_t e = hipSuccess;
    if (b->side) {
      e = hipEventRecord(b->forked, (hipStream_t)st);
      if (e == hipSuccess) e = hipStreamWaitEvent(b->side, b->forked, 0);
    }
    if (e == hipSuccess && b->nitems)
      e = pc2k::launch_batch(b->op, b->pair, b->grid, b->jobs, b->items, b->nitems, b->queue,
                             b->scratch, b->slot_words, b->w_a, b->w_b, b->ctx->err, st);
    for (const auto& m : b->mp)
      if (e == hipSuccess && m.nitems)
        e = pc2k::launch_batch_mfma(m.cls, m.grid, b->jobs, m.items, m.nitems, m.sub, m.queue,
                                    b->mscratch, m.w, b->ctx->err, st);
    for (const RnsPart& p : b->rparts)
      if (e == hipSuccess && rns_part_run(b->ctx, p, b->op, p.side ? b->rscratch2 : b->rscratch,
                                          p.side ? (void*)b->side : st) != PC2_OK)
        e = hipErrorLaunchFailure;
    if (b->side) {  // joined whatever happened, as a capture ends with no open branch
      const hipError_t j = hipEventRecord(b->joined, b->side);
      const hipError_t w = hipStreamWaitEvent((hipStream_t)st, b->joined, 0);
      if (e == hipSuccess) e = j != hipSuccess ? j : w;
    }
    return e;
  };
  if (!hip_stream) return status_of(launch(nullptr));
  if (!b->exec || b->graph_stream != hip_stream) {
    if (b->exec) {
      (void)hipGraphExecDestroy(b->exec);
      b->exec = nullptr;
    }
    hipStream_t st = (hipStream_t)hip_stream;
    if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess)
      return PC2_E_DEVICE;
    hipError_t le = launch(hip_stream);
    hipGraph_t g = nullptr;
    hipError_t ee = hipStreamEndCapture(st, &g);
    if (le != hipSuccess || ee != hipSuccess || !g) {
      if (g) (void)hipGraphDestroy(g);
      return PC2_E_DEVICE;
    }
    hipError_t ie = hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ie != hipSuccess) {
      b->exec = nullptr;
      return PC2_E_DEVICE;
    }
    b->graph_stream = hip_stream;
  }
  return status_of(hipGraphLaunch(b->exec, (hipStream_t)hip_stream));
}

int pc2_batch_destroy(pc2_batch* b) {
  if (!b || !b->ctx) return PC2_E_INVAL;
  (void)hipSetDevice(b->ctx->device);
  (void)hipDeviceSynchronize();
  batch_free(b);
  return PC2_OK;
}

// -------------------------------------------------------------- autotune
// Times encryption in each tile the key's class has (lanes per ciphertext)
// with windows 4..6, and decryption with windows 4..6, on a few
// device-filling waves of elements of the VALU engine; keeps the fastest choices in
// the context, where that engine's calls read them.
int pc2_autotune(const pc2_sk* sk, void* hip_stream, int* w_enc, int* w_dec, int* tile_enc) {
  if (!sk || !sk->ctx) return PC2_E_INVAL;
  pc2_ctx* ctx = sk->ctx;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  const int cls = sk->pk.cls, L = sk->pk.L;
  int geos[2] = {cls, pc2k::ALT_GEO[cls]};
  const int ngeo = geos[1] >= 0 ? 2 : 1;
  // the same element count for every candidate: four waves of the widest
  size_t count = 0;
  for (int g = 0; g < ngeo; ++g)
    count = std::max(count, (size_t)ctx->cus * occupancy(ctx, geos[g], pc2k::OP_ENC) *
                                (size_t)pc2k::elems_per_block(geos[g]));
  count *= 4;
  // the work of the exponentiations does not depend on the data: m = 0,
  // r = 1 is valid under every key
  std::vector<uint32_t> hm(count, 0), hr(count * L, 0);
  for (size_t i = 0; i < count; ++i) hr[i * L] = 1;
  uint32_t *m = nullptr, *r = nullptr, *c = nullptr, *d = nullptr;
  int rc = PC2_OK;
  if (hipMalloc(&m, count * 4) != hipSuccess || hipMalloc(&r, count * L * 4) != hipSuccess ||
      hipMalloc(&c, count * 2 * L * 4) != hipSuccess || hipMalloc(&d, count * L * 4) != hipSuccess)
    rc = PC2_E_NOMEM;
  if (!rc && (hipMemcpy(m, hm.data(), count * 4, hipMemcpyHostToDevice) != hipSuccess ||
              hipMemcpy(r, hr.data(), count * L * 4, hipMemcpyHostToDevice) != hipSuccess))
    rc = PC2_E_DEVICE;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (!rc && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
    rc = PC2_E_DEVICE;
  const int saved_window = ctx->window, saved_tile = ctx->tile, saved_modmul = ctx->modmul;
  ctx->modmul = PC2_MODMUL_VALU;
  int best_w[2] = {0, 0}, best_geo = cls;
  float best_ms[2] = {1e30f, 1e30f};
  // trials: (encryption, geometry) for each tile, then decryption
  for (int trial = 0; trial <= ngeo && !rc; ++trial) {
    const bool dec = trial == ngeo;
    if (!dec) ctx->tile = pc2k::CLASS_GEO[geos[trial]].nT;
    for (int w = 4; w <= 6 && !rc; ++w) {
      ctx->window = w;
      for (int rep = 0; rep < 2 && !rc; ++rep) {  // rep 0 warms up (and sizes scratch)
        if (hipEventRecord(e0, (hipStream_t)hip_stream) != hipSuccess) rc = PC2_E_DEVICE;
        int st = dec ? pc2_decrypt(sk, c, d, count, hip_stream)
                     : pc2_encrypt(&sk->pk, m, 1, r, c, count, hip_stream);
        if (st) rc = st;
        if (!rc && (hipEventRecord(e1, (hipStream_t)hip_stream) != hipSuccess ||
                    hipEventSynchronize(e1) != hipSuccess))
          rc = PC2_E_DEVICE;
        float ms = 0;
        if (!rc && rep == 1 && hipEventElapsedTime(&ms, e0, e1) == hipSuccess &&
            ms < best_ms[dec]) {
          best_ms[dec] = ms;
          best_w[dec] = w;
          if (!dec) best_geo = geos[trial];
        }
      }
    }
  }
  ctx->window = saved_window;
  ctx->tile = saved_tile;
  ctx->modmul = saved_modmul;
  if (!rc) {
    ctx->tuned_geo[cls] = best_geo;
    ctx->tuned[best_geo][pc2k::OP_ENC] = best_w[0];
    ctx->tuned[cls][pc2k::OP_DEC] = best_w[1];
    if (w_enc) *w_enc = best_w[0];
    if (w_dec) *w_dec = best_w[1];
    if (tile_enc) *tile_enc = pc2k::CLASS_GEO[best_geo].nT;
    rc = pc2_ctx_take_error(ctx);
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (m) (void)hipFree(m);
  if (r) (void)hipFree(r);
  if (c) (void)hipFree(c);
  if (d) (void)hipFree(d);
  return rc;
}

// ---------------------------------------------------------------- runners
namespace {
// elements of the largest group of a key up to class cls
size_t runner_group_max(int op, int cls) {
  size_t elems = 0;
  for (int g = 0; g < pc2k::NUM_GEOS; ++g)
    if (pc2k::GEO_CLASS[g] >= RNS_MIN_CLASS && pc2k::GEO_CLASS[g] <= cls)
      elems = std::max(elems, (size_t)std::max(0, pc2k::batch_group_elems(op, g)));
  return elems;
}
int op_from_abi(int op_abi) {
  if (op_abi == PC2_OP_ENCRYPT) return pc2k::OP_ENC;
  if (op_abi == PC2_OP_DECRYPT) return pc2k::OP_DEC;
  if (op_abi == PC2_OP_HOM_SUM) return pc2k::OP_SUM;
  return -1;
}
}  // namespace

int pc2_runner_create(pc2_ctx* ctx, int op_abi, uint32_t max_nbits, size_t max_jobs,
                      size_t max_groups, pc2_runner** out) {
  if (!ctx || !out || max_jobs == 0 || max_groups == 0) return PC2_E_INVAL;
  *out = nullptr;
  const int op = op_from_abi(op_abi);
  const int cls = pc2k::class_for_bits((int)max_nbits);
  if (op < 0) return PC2_E_INVAL;
  if (cls < 0) return PC2_E_UNSUPPORTED;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  pc2_runner* r = new (std::nothrow) pc2_runner();
  if (!r) return PC2_E_NOMEM;
  r->ctx = ctx;
  r->op = op;
  r->max_cls = cls;
  r->max_jobs = max_jobs;
  r->max_groups = max_groups;
  r->max_ptrs = op == pc2k::OP_SUM ? 2 * (size_t)pc2k::RK_MAX * max_jobs : 0;
  r->jobs_b = (max_jobs * sizeof(pc2k::BatchJob) + 255) & ~(size_t)255;
  // a decryption group is two items (one per prime)
  const size_t max_items = (op == pc2k::OP_DEC ? 2 : 1) * max_groups;
  r->items_b = (max_items * sizeof(pc2k::BatchItem) + 255) & ~(size_t)255;
  r->ptr_b = (r->max_ptrs * sizeof(size_t) + 255) & ~(size_t)255;
  // the RNS engine's jobs, of which each part's end may cut one in two
  const size_t max_pos = max_groups * runner_group_max(op, cls) + 32 * max_jobs;
  if (op != pc2k::OP_SUM && cls >= RNS_MIN_CLASS)
    r->rjobs_b =
        ((max_jobs + 2 * (max_pos / RNS_PART) + 1) * sizeof(pc2k::RnsJob) + 255) & ~(size_t)255;
  const size_t total = r->jobs_b + r->items_b + r->ptr_b + QUEUE_BYTES + r->rjobs_b;
  int rc = PC2_OK;
  if (hipMalloc(&r->dev, total) != hipSuccess || hipHostMalloc(&r->host, total) != hipSuccess ||
      hipEventCreateWithFlags(&r->copied, hipEventDisableTiming) != hipSuccess)
    rc = PC2_E_NOMEM;
  // scratch for the widest pair this runner may launch
  if (!rc) {
    int tiles = 0;
    size_t words = 0;
    int occ_max = 1;
    const int L = (int)((max_nbits + 31) / 32);
    const int Ls = std::min(L / 2 + 2, pc2k::LS_MAX);
    r->ls = Ls;
    for (int g = 0; g < pc2k::NUM_GEOS; ++g) {
      if (pc2k::GEO_CLASS[g] > cls) continue;
      const int pair = pc2k::batch_pair(g, g);
      if (pair < 0 || !pc2k::batch_kernel(op, pair)) continue;
      const int w = std::max(window_for(ctx, g, op), 6);
      int t = 0;
      size_t wd = 0;
      pc2k::batch_slot_shape(op, g, w, Ls, &t, &wd);
      tiles = std::max(tiles, t);
      words = std::max(words, wd);
    }
    for (int pair = 0; pair < pc2k::batch_npairs(); ++pair) {
      const void* k = pc2k::batch_kernel(op, pair);
      if (!k) continue;
      int occ = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, 64, 0) == hipSuccess)
        occ_max = std::max(occ_max, occ);
    }
    r->grid_cap = ctx->cus * occ_max;
    r->slot_words = (words + 3) & ~(size_t)3;
    const size_t bytes = (size_t)r->grid_cap * tiles * r->slot_words * 4;
    if (bytes && hipMalloc(&r->scratch, bytes) != hipSuccess) rc = PC2_E_NOMEM;
    // encryption jobs of a class on the matrix cores (the engine option may
    // change after creation, so every class up to the largest is covered)
    for (int c = 0; !rc && op == pc2k::OP_ENC && c <= cls; ++c) {
      r->mocc[c] = occupancy_of(pc2k::batch_mfma_kernel(c));
      r->mscratch_bytes =
          std::max(r->mscratch_bytes, (size_t)ctx->cus * r->mocc[c] *
                                          (pc2k::mfma_digit_bytes(c) << pc2k::SCHED_WMAX));
    }
    if (!rc && r->mscratch_bytes && hipMalloc(&r->mscratch, r->mscratch_bytes) != hipSuccess)
      rc = PC2_E_NOMEM;
    // the RNS engine: a part's positions under any key up to max_nbits (without
    // memory for it, launches stay on the persistent kernels)
    if (!rc && r->rjobs_b) {
      const size_t npos = std::min<size_t>(max_pos, RNS_PART);
      const pc2k::ClassGeo cg = pc2k::CLASS_GEO[cls];
      const int p2bits = cg.pD * cg.pK * cg.pT - 2;
      const int tmax = pc2h::rns_tiles(op == pc2k::OP_DEC ? p2bits : 64 * L);
      for (int T : pc2k::RNS_T)
        for (int nb = 1; nb <= pc2k::RNS_NBMAX; ++nb) {
          if (T > tmax || !rns_slots(ctx, T, nb)) continue;
          const RnsPlan p =
              rns_plan_nb(ctx, T, op == pc2k::OP_DEC ? 2 : 1, npos, nb, pc2k::SCHED_WMAX);
          r->rscratch_bytes = std::max(
              r->rscratch_bytes, op == pc2k::OP_DEC
                                     ? rns_decrypt_bytes(p, npos, (p2bits + 31) / 32)
                                     : rns_encrypt_bytes(p));
        }
      if (r->rscratch_bytes && hipMalloc(&r->rscratch, r->rscratch_bytes) != hipSuccess) {
        (void)hipGetLastError();
        r->rscratch = nullptr;
      }
    }
    if (!rc && op == pc2k::OP_DEC) {  // CRT halves of up to max_groups groups
      size_t per = 0;
      for (int g = 0; g < pc2k::NUM_GEOS; ++g)
        if (pc2k::GEO_CLASS[g] <= cls && pc2k::batch_group_elems(op, g) > 0)
          per = std::max(per, (size_t)pc2k::batch_group_elems(op, g) * 2 * (Ls + 1));
      if (hipMalloc(&r->stage, max_groups * per * 4) != hipSuccess) rc = PC2_E_NOMEM;
    }
  }
  if (rc) {
    if (r->dev) (void)hipFree(r->dev);
    if (r->host) (void)hipHostFree(r->host);
    if (r->scratch) (void)hipFree(r->scratch);
    if (r->mscratch) (void)hipFree(r->mscratch);
    if (r->rscratch) (void)hipFree(r->rscratch);
    if (r->stage) (void)hipFree(r->stage);
    if (r->copied) (void)hipEventDestroy(r->copied);
    delete r;
    return rc;
  }
  *out = r;
  return PC2_OK;
}

int pc2_runner_group_size(const pc2_pk* pk, int op_abi, uint32_t* elems) {
  if (!pk || !pk->ctx || !elems || op_from_abi(op_abi) < 0) return PC2_E_INVAL;
  const int op = op_from_abi(op_abi);
  *elems = (uint32_t)pc2k::batch_group_elems(op, job_geo(pk->ctx, pk, op));
  return PC2_OK;
}

static int runner_launch(pc2_runner* r, const pc2_job* jobs, const size_t* first,
                         const size_t* ngroups, size_t njobs, void* hip_stream) {
  if (!r || !r->ctx || !jobs || !first || !ngroups || njobs == 0) return PC2_E_INVAL;
  if (njobs > r->max_jobs) return PC2_E_BUSY;
  pc2_ctx* ctx = r->ctx;
  const int op = r->op;
  int ca = -1, cb = -1, mca = -1, mcb = -1;
  size_t nitems = 0, nptrs = 0;
  for (size_t i = 0; i < njobs; ++i) {
    const pc2_job& j = jobs[i];
    if (op_from_abi(j.op) != op) return PC2_E_INVAL;
    const pc2_pk* pk = (op == pc2k::OP_DEC) ? (j.sk ? &j.sk->pk : nullptr) : j.pk;
    if (!pk || pk->ctx != ctx || !j.out || pk->cls > r->max_cls) return PC2_E_INVAL;
    const int g = job_geo(ctx, pk, op);
    const size_t epw = (size_t)pc2k::batch_group_elems(op, g);
    if (epw == 0) return PC2_E_UNSUPPORTED;  // no element groups under keys of this class
    if (first[i] + ngroups[i] > (j.count + epw - 1) / epw) return PC2_E_INVAL;
    if (op == pc2k::OP_ENC && (!j.in0 || !j.in1 || j.m_limbs < 1 || (int)j.m_limbs > pk->L))
      return PC2_E_INVAL;
    if (op == pc2k::OP_DEC && (!j.in0 || j.sk->c.h[0].Ls > r->ls)) return PC2_E_INVAL;
    if (op == pc2k::OP_SUM) {
      if (!j.inputs || j.K < 1 || j.K > (uint32_t)pc2k::RK_MAX) return PC2_E_INVAL;
      for (uint32_t k = 0; k < j.K; ++k)
        if (!j.inputs[k] || (j.lengths && j.lengths[k] > j.count)) return PC2_E_INVAL;
      nptrs += 2 * (size_t)j.K;
    }
    if (job_overlaps(j, pk->L)) return PC2_E_INVAL;
    nitems += ngroups[i];
    if (ngroups[i] == 0) continue;
    if (op == pc2k::OP_ENC && use_mfma(ctx, pk->cls)) {
      if (mca < 0 || mca == pk->cls) mca = pk->cls;
      else if (mcb < 0 || mcb == pk->cls) mcb = pk->cls;
      else return PC2_E_UNSUPPORTED;
      continue;
    }
    if (ca < 0 || ca == g) ca = g;
    else if (cb < 0 || cb == g) cb = g;
    else return PC2_E_UNSUPPORTED;
  }
  if (nitems == 0) return PC2_OK;
  if (nitems > r->max_groups || nptrs > r->max_ptrs) return PC2_E_BUSY;
  for (int c : {mca, mcb})  // (the scratch covers every class up to max_cls)
    if (c >= 0 && (!r->mscratch || (pc2k::mfma_digit_bytes(c)
                                    << window_for(ctx, c, pc2k::OP_ENC_MFMA)) > r->mscratch_bytes))
      return PC2_E_NOMEM;
  int pair = -1;
  if (ca >= 0) {
    if (cb < 0) cb = ca;
    pair = pc2k::batch_pair(ca, cb);
    if (pair < 0) return PC2_E_UNSUPPORTED;
  }
  // the jobs that the RNS engine takes (whatever fits the launcher's scratch;
  // the others stay on the persistent kernels)
  std::vector<size_t> relem(njobs), rcount(njobs);
  for (size_t i = 0; i < njobs; ++i) {
    const pc2_pk* pk = (op == pc2k::OP_DEC) ? &jobs[i].sk->pk : jobs[i].pk;
    const size_t epw = (size_t)pc2k::batch_group_elems(op, job_geo(ctx, pk, op));
    relem[i] = first[i] * epw;
    rcount[i] = std::min(ngroups[i] * epw, jobs[i].count - std::min(jobs[i].count, relem[i]));
  }
  std::vector<bool> in_rns;
  std::vector<pc2k::RnsJob> rjobs;
  std::vector<RnsPart> parts =
      rns_parts(ctx, op, jobs, relem.data(), rcount.data(), njobs, &in_rns, &rjobs);
  for (const RnsPart& p : parts)
    if (!r->rscratch || rns_part_bytes(p, op) > r->rscratch_bytes ||
        rjobs.size() * sizeof(pc2k::RnsJob) > r->rjobs_b) {
      parts.clear();
      rjobs.clear();
      in_rns.assign(njobs, false);
      break;
    }
  const int few = few_elements_class(ctx, op, jobs, rcount.data(), njobs, in_rns);
  if (few >= 0 && mcb < 0 && r->mscratch) {
    (mca < 0 ? mca : mcb) = few;
    pair = -1;
  }
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  // the previous launch's copies must have read the staging buffers
  if (r->pending && hipEventSynchronize(r->copied) != hipSuccess) return PC2_E_DEVICE;
  char* hb = (char*)r->host;
  char* db = (char*)r->dev;
  auto* hj = (pc2k::BatchJob*)hb;
  auto* hi = (pc2k::BatchItem*)(hb + r->jobs_b);
  auto* hp = (size_t*)(hb + r->jobs_b + r->items_b);
  auto* dp = (size_t*)(db + r->jobs_b + r->items_b);
  size_t pofs = 0, it = 0, sofs = 0;
  const int pa = pair >= 0 ? pc2k::batch_pair_geo(pair, 0) : -1;
  const int pb = pair >= 0 ? pc2k::batch_pair_geo(pair, 1) : -1;
  for (size_t i = 0; i < njobs; ++i) {
    const pc2_job& j = jobs[i];
    const pc2_pk* pk = (op == pc2k::OP_DEC) ? &j.sk->pk : j.pk;
    const bool mf = op == pc2k::OP_ENC && (pk->cls == mca || pk->cls == mcb);
    pc2k::BatchJob d{};
    d.geo = mf ? pk->cls : job_geo(ctx, pk, op);
    d.group = pc2k::batch_group_elems(op, job_geo(ctx, pk, op));
    d.op = op;
    d.m_limbs = (int)j.m_limbs;
    d.K = (int)j.K;
    d.pk = mf ? pk->c : geo_const(pk, d.geo);
    if (op == pc2k::OP_DEC) d.sk = j.sk->c;
    d.in0 = j.in0;
    d.in1 = j.in1;
    d.out = j.out;
    d.count = j.count;
    if (op == pc2k::OP_DEC) {  // this launch's groups of job i, back to back
      const size_t epw = (size_t)pc2k::batch_group_elems(op, d.geo);
      d.stage = r->stage + sofs;
      d.stage_g0 = first[i];
      sofs += ngroups[i] * epw * 2 * (size_t)(d.sk.h[0].Ls + 1);
    }
    if (op == pc2k::OP_SUM) {
      for (uint32_t k = 0; k < j.K; ++k) hp[pofs + k] = (size_t)j.inputs[k];
      for (uint32_t k = 0; k < j.K; ++k) hp[pofs + j.K + k] = j.lengths ? j.lengths[k] : j.count;
      d.inputs = (const uint32_t* const*)(dp + pofs);
      d.lengths = dp + pofs + j.K;
      pofs += 2 * (size_t)j.K;
    }
    hj[i] = d;
  }
  // most expensive class first; the matrix-core items after the others
  auto on_mfma = [&](size_t i) {
    const pc2_pk* pk = (op == pc2k::OP_DEC) ? &jobs[i].sk->pk : jobs[i].pk;
    return op == pc2k::OP_ENC && (pk->cls == mca || pk->cls == mcb);
  };
  for (int pass = 0; pair >= 0 && pass < 2; ++pass) {
    const int first_geo = pc2k::GEO_CLASS[pa] >= pc2k::GEO_CLASS[pb] ? pa : pb;
    const int want = pass == 0 ? first_geo : (first_geo == pa ? pb : pa);
    if (pass == 1 && pa == pb) break;
    for (size_t i = 0; i < njobs; ++i) {
      if (in_rns[i] || on_mfma(i) || hj[i].geo != want) continue;
      for (size_t g = 0; g < ngroups[i]; ++g) {
        hi[it++] = pc2k::BatchItem{(int)i, 0, first[i] + g};
        if (op == pc2k::OP_DEC) hi[it++] = pc2k::BatchItem{(int)i, 1, first[i] + g};
      }
    }
  }
  const size_t it_valu = it;
  const int mcls[2] = {std::max(mca, mcb), std::min(mca, mcb)};  // the more expensive first
  size_t mfirst[3] = {it, it, it};
  int msub[2] = {1, 1};
  for (int part = 0; part < 2; ++part) {
    mfirst[part] = it;
    for (size_t i = 0; mcls[part] >= 0 && i < njobs; ++i)
      if (!in_rns[i] && on_mfma(i) && hj[i].geo == mcls[part]) {
        msub[part] = std::max(msub[part], hj[i].group);
        for (size_t g = 0; g < ngroups[i]; ++g)
          hi[it++] = pc2k::BatchItem{(int)i, 0, first[i] + g};
      }
    mfirst[part + 1] = it;
  }
  const size_t rofs = r->jobs_b + r->items_b + r->ptr_b + QUEUE_BYTES;
  std::copy(rjobs.begin(), rjobs.end(), (pc2k::RnsJob*)(hb + rofs));
  rns_parts_place(parts, db + rofs);
  hipStream_t st = (hipStream_t)hip_stream;
  if (hipMemcpyAsync(db, hb, njobs * sizeof(pc2k::BatchJob), hipMemcpyHostToDevice, st) !=
          hipSuccess ||
      (it && hipMemcpyAsync(db + r->jobs_b, hb + r->jobs_b, it * sizeof(pc2k::BatchItem),
                            hipMemcpyHostToDevice, st) != hipSuccess) ||
      (!rjobs.empty() && hipMemcpyAsync(db + rofs, hb + rofs,
                                        rjobs.size() * sizeof(pc2k::RnsJob),
                                        hipMemcpyHostToDevice, st) != hipSuccess) ||
      (pofs && hipMemcpyAsync(dp, hp, pofs * sizeof(size_t), hipMemcpyHostToDevice, st) !=
                   hipSuccess) ||
      hipEventRecord(r->copied, st) != hipSuccess)
    return PC2_E_DEVICE;
  r->pending = true;
  int* queue = (int*)(db + r->jobs_b + r->items_b + r->ptr_b);
  const auto* ditems = (const pc2k::BatchItem*)(db + r->jobs_b);
  hipError_t e = hipSuccess;
  if (it_valu) {
    const int grid = (int)std::max<size_t>(1, std::min<size_t>(r->grid_cap, it_valu));
    const int w_a = window_for(ctx, pa, op), w_b = window_for(ctx, pb, op);
    e = pc2k::launch_batch(op, pair, grid, (const pc2k::BatchJob*)db, ditems, (int)it_valu,
                           queue, r->scratch, r->slot_words, w_a, w_b, ctx->err, st);
  }
  for (int part = 0; part < 2 && e == hipSuccess; ++part) {
    const size_t n = mfirst[part + 1] - mfirst[part];
    if (!n) continue;
    const int c = mcls[part];
    const int w = window_for(ctx, c, pc2k::OP_ENC_MFMA);
    const size_t per = pc2k::mfma_digit_bytes(c) << w;
    const size_t cap = (size_t)ctx->cus * std::max(1, r->mocc[c]);
    const int grid = (int)std::max<size_t>(
        1, std::min<size_t>({cap, n * msub[part], r->mscratch_bytes / per}));
    e = pc2k::launch_batch_mfma(c, grid, (const pc2k::BatchJob*)db, ditems + mfirst[part],
                                (int)n, msub[part], queue + QUEUE_STRIDE * (part + 1),
                                r->mscratch, w,
                                ctx->err, st);
  }
  int rc = status_of(e);
  for (const RnsPart& p : parts)
    if (!rc) rc = rns_part_run(ctx, p, op, r->rscratch, hip_stream);
  return rc;
}

int pc2_runner_launch(pc2_runner* r, const pc2_job* jobs, const size_t* first,
                      const size_t* ngroups, size_t njobs, void* hip_stream) {
  try {  // (its job lists by key are host memory; nothing is enqueued before them)
    return runner_launch(r, jobs, first, ngroups, njobs, hip_stream);
  } catch (const std::bad_alloc&) {
    return PC2_E_NOMEM;
  }
}

int pc2_runner_destroy(pc2_runner* r) {
  if (!r || !r->ctx) return PC2_E_INVAL;
  (void)hipSetDevice(r->ctx->device);
  (void)hipDeviceSynchronize();
  if (r->dev) (void)hipFree(r->dev);
  if (r->host) (void)hipHostFree(r->host);
  if (r->scratch) (void)hipFree(r->scratch);
  if (r->mscratch) (void)hipFree(r->mscratch);
  if (r->rscratch) (void)hipFree(r->rscratch);
  if (r->stage) (void)hipFree(r->stage);
  if (r->copied) (void)hipEventDestroy(r->copied);
  delete r;
  return PC2_OK;
}

// ------------------------------------------------------ ciphertext mat-vec
namespace {
size_t matvec_table_bytes(int cls, size_t cols, int ebits, int w) {
  const size_t nw = (size_t)((ebits + w - 1) / w);
  return cols * nw * (((size_t)1 << w) - 1) * pc2k::matvec_entry_words(cls) * 4;
}
int resident_groups(pc2_ctx* ctx, const void* k) {
  int occ = 0;
  if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, 64, 0) != hipSuccess || occ <= 0)
    occ = 1;
  return ctx->cus * occ;
}
// Column chunks of a mat-vec of `rows` rows: the count (up to the aggregation
// limit and max_chunks) whose whole wavefront groups fill the resident
// capacity best; fewer on a near tie.
void pick_chunks(const pc2_matvec* mv, size_t rows, size_t max_chunks, size_t* nch,
                 size_t* chunk_cols) {
  const size_t epw = (size_t)pc2k::elems_per_block(mv->pk->cls);
  const size_t gpc = (rows + epw - 1) / epw;
  const size_t cap = (size_t)mv->cap_apply;
  *nch = 1;
  *chunk_cols = mv->cols;
  double best = -1;
  const size_t top = std::min(std::min(mv->cols, (size_t)pc2k::RK_MAX), std::max<size_t>(1, max_chunks));
  for (size_t c = 1; c <= top; ++c) {
    const size_t cc = (mv->cols + c - 1) / c;
    if ((mv->cols + cc - 1) / cc != c) continue;  // the same split as a smaller count
    const size_t groups = gpc * c;
    const double eff = (double)groups / (double)(((groups + cap - 1) / cap) * cap);
    if (eff > best + 0.02) {
      best = eff;
      *nch = c;
      *chunk_cols = cc;
    }
  }
}
}  // namespace

namespace {
// Column blocks per row group (nb) and column chunks of `rows` rows on the RNS
// engine, their running values at most `blocks` blocks of 32: the least time
// by rounds of resident workgroups (a product measured 1.45 + nb, as its
// multipliers come from HBM, and 1.1 times that with constants in blocks; else see
// rns_round), plus the products that join the chunks.
struct RnsMvShape {
  int nb = 0;
  size_t groups = 0, nch = 0, chunk_cols = 0;
  double cost = 0;
};
int rns_mv_kind(const pc2k::RnsDigits& dg) {
  return dg.nblk > 1 ? pc2k::RNS_MVBLK : pc2k::RNS_MV;
}
RnsMvShape rns_mv_shape(pc2_ctx* ctx, int T, size_t cols, const pc2k::RnsDigits& dg, size_t rows,
                        size_t blocks) {
  RnsMvShape best;
  // products per column, and (constants in blocks) squarings and the last product
  const int per = dg.n * dg.nblk, fix = dg.nblk > 1 ? dg.bits() * (dg.nblk - 1) + 1 : 0;
  auto unit = [&](int nb) { return (1.45 + nb) * (dg.nblk > 1 ? 1.1 : 1.0); };
  for (int nb = 1; nb <= pc2k::RNS_NBMAX; ++nb) {
    const size_t slots = (size_t)rns_slots(ctx, T, nb, rns_mv_kind(dg));
    const size_t G = (rows + 32 * nb - 1) / (32 * nb);
    if (!slots || (G * nb > blocks && best.nb)) continue;
    for (size_t c = 1; c <= std::min(cols, (size_t)256) && (c == 1 || G * nb * c <= blocks); ++c) {
      const size_t cc = (cols + c - 1) / c;
      if ((cols + cc - 1) / cc != c) continue;  // the same split as a smaller count
      const double t = ((double)((G * c + slots - 1) / slots) * (double)(cc * per + fix) +
                        (c > 1 ? (double)c : 0.0)) * unit(nb);
      if (!best.nb || t < best.cost) best = {nb, G, c, cc, t};
    }
  }
  return best;
}

// The RNS engine for a plan: the blocks and digits of the least time among those
// whose tables fit the plan's table bytes; false if there is none or the device has
// no memory for it.  Its entries are 1.7 times the VALU engine's.  Plans for many
// rows, whose windows are wide, hold all digits of a constant; for few rows the
// window is narrow, and blocks that share a small table do with a fraction of its
// bytes.  It is the faster one from a single row up (load / apply in ms, RNS against
// VALU, ebits 50: 1024 bits, 64 rows x 16 columns 0.16 / 0.16 against 1.02 / 2.1; 2048
// bits, 256 x 256: 0.40 / 1.2 against 2.2 / 4.8, 1 x 1000: 0.16 / 1.8 against 3.1 / 9.4;
// 4096 bits, 64 x 16: 1.1 / 1.07 against 4.1 / 1.44).  Constants of one bit, whose
// tables hold one VALU entry, stay on the VALU.
bool rns_matvec_create(pc2_matvec* mv, size_t rows_hint) {
  pc2_ctx* ctx = mv->ctx;
  const int T = mv->pk->rn.T;
  if (!T || ctx->modmul == PC2_MODMUL_VALU) return false;
  const size_t slots = (size_t)rns_slots(ctx, T, 1, pc2k::RNS_MV);
  const size_t tslots = (size_t)rns_slots(ctx, T, 1, pc2k::RNS_MVTAB);
  if (!slots || !tslots) return false;
  const size_t Gc = (mv->cols + 31) / 32, most = 2 * slots;
  // (no hint: rows enough that the tables' cost is small, as for the window)
  const size_t rows = std::min(rows_hint ? rows_hint : (size_t)8192, most * 32);
  double best = 0;
  for (int nblk = 1; nblk <= mv->ebits; ++nblk) {
    const int bits = (mv->ebits + nblk - 1) / nblk;
    for (int nw = (bits + 11) / 12; nw <= bits; ++nw) {
      const pc2k::RnsDigits dg = pc2k::RnsDigits::of(mv->ebits, nw, nblk);
      if (mv->cols * (dg.entries() * (size_t)64 * T) > mv->table_bytes ||
          bits * (nblk - 1) + dg.shift(nw - 1) > 63)  // (the kernel shifts by it)
        continue;
      const double cost = rns_mv_shape(ctx, T, mv->cols, dg, rows, most).cost +
                          2.45 * (double)((Gc * nw + tslots - 1) / tslots) *
                              (double)(((size_t)1 << dg.width(0)) + (size_t)dg.shift(nw - 1));
      if (mv->rdg.n == 0 || cost < best) {
        best = cost;
        mv->rdg = dg;
      }
    }
  }
  if (mv->rdg.n == 0) return false;
  mv->rblocks = std::max(most, Gc + std::min(tslots, Gc * mv->rdg.n));
  const size_t stage = mv->rblocks * pc2k::rns_group_bytes(T, 1);
  mv->rstage_bytes = stage + mv->rblocks * 32 * 4;
  if (hipMalloc(&mv->tab, mv->table_bytes) != hipSuccess ||
      hipMalloc(&mv->rstage, mv->rstage_bytes) != hipSuccess ||
      hipEventCreateWithFlags(&mv->done, hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    if (mv->tab) (void)hipFree(mv->tab);
    if (mv->rstage) (void)hipFree(mv->rstage);
    mv->tab = nullptr;
    mv->rstage = nullptr;
    mv->rdg = {};
    return false;
  }
  mv->rbad = reinterpret_cast<uint32_t*>(mv->rstage + stage);
  return true;
}
// the plan's staging is used by one call after another, whatever their streams
// (as the context's scratch: scratch_begin, scratch_end)
int stage_begin(pc2_matvec* mv, void* stream) {
  if (!mv->done_valid || mv->done_stream == stream || capturing(stream)) return PC2_OK;
  return hipStreamWaitEvent((hipStream_t)stream, mv->done, 0) == hipSuccess ? PC2_OK
                                                                           : PC2_E_DEVICE;
}
int stage_end(pc2_matvec* mv, void* stream, int rc) {
  if (rc || capturing(stream)) return rc;
  if (hipEventRecord(mv->done, (hipStream_t)stream) != hipSuccess) return PC2_E_DEVICE;
  mv->done_stream = stream;
  mv->done_valid = true;
  return PC2_OK;
}

int rns_matvec_load(pc2_matvec* mv, const uint32_t* c, void* stream) {
  pc2_ctx* ctx = mv->ctx;
  const pc2k::RnsKey& K = mv->pk->rn;
  const int L2 = 2 * mv->pk->L;
  const size_t gb = pc2k::rns_group_bytes(K.T, 1), slots = (size_t)rns_slots(ctx, K.T, 1, pc2k::RNS_MVTAB);
  const size_t Gc = (mv->cols + 31) / 32;
  int rc = stage_begin(mv, stream);
  if (rc) return rc;
  pc2k::RnsMvTab t{};
  t.M = K.M;
  t.one = K.one;
  t.in = mv->rstage;
  t.table = mv->rstage + Gc * gb;
  t.tab = reinterpret_cast<uint8_t*>(mv->tab);
  t.c = c;
  t.n2 = mv->pk->c.n2.Nl;
  t.L2 = L2;
  t.dg = mv->rdg;
  t.ngroups = (int)Gc;
  t.cols = mv->cols;
  t.err = ctx->err;
  hipError_t e = pc2k::launch_rns_to(K.c, K.T, 1, one_job(c, nullptr, 0, nullptr, mv->cols), false,
                                     L2, mv->rstage, stream);
  if (e == hipSuccess)
    e = pc2k::launch_rns_gather(K.T, 1, pc2k::RNS_MVTAB,
                                (int)std::min<size_t>(slots, Gc * mv->rdg.n), &t, stream);
  return stage_end(mv, stream, status_of(e));
}

int rns_matvec_apply(pc2_matvec* mv, const uint64_t* B, const uint32_t* alpha, uint32_t* out,
                     size_t rows, void* stream) {
  pc2_ctx* ctx = mv->ctx;
  const pc2k::RnsKey& K = mv->pk->rn;
  const size_t L2 = 2 * (size_t)mv->pk->L;
  int rc = stage_begin(mv, stream);
  for (size_t at = 0; at < rows && !rc; at += mv->rblocks * 32) {
    const size_t n = std::min(rows - at, mv->rblocks * 32);
    const RnsMvShape S = rns_mv_shape(ctx, K.T, mv->cols, mv->rdg, n, mv->rblocks);
    const uint32_t* a = alpha ? alpha + at * L2 : nullptr;
    const pc2k::RnsJobs J = one_job(a, nullptr, 0, out + at * L2, n);
    pc2k::RnsMv m{};
    m.M = K.M;
    m.one = K.one;
    m.in = mv->rstage;
    m.tab = reinterpret_cast<const uint8_t*>(mv->tab);
    m.B = B + at * mv->cols;
    m.bad = mv->rbad;
    m.rows = n;
    m.cols = mv->cols;
    m.chunk_cols = S.chunk_cols;
    m.alpha = alpha != nullptr;
    m.ebits = mv->ebits;
    m.dg = mv->rdg;
    m.nch = (int)S.nch;
    m.ngroups = (int)S.groups;
    hipError_t e = pc2k::launch_rns_row_check(a, mv->pk->c.n2.Nl, (int)L2, mv->rbad, n, stream);
    if (e == hipSuccess && a)
      e = pc2k::launch_rns_to(K.c, K.T, S.nb, J, false, (int)L2, mv->rstage, stream);
    auto gather = [&](int which, size_t items) {
      const size_t slots = (size_t)rns_slots(ctx, K.T, S.nb, which);
      return pc2k::launch_rns_gather(K.T, S.nb, which, (int)std::min(slots, items), &m, stream);
    };
    if (e == hipSuccess) e = gather(rns_mv_kind(mv->rdg), S.groups * S.nch);
    if (e == hipSuccess && S.nch > 1) e = gather(pc2k::RNS_CHAIN, S.groups);
    if (e == hipSuccess)
      e = pc2k::launch_rns_from(K.from, K.T, S.nb, mv->rstage, J, nullptr, 0, stream);
    if (e == hipSuccess)
      e = pc2k::launch_rns_row_clear(mv->rbad, out + at * L2, (int)L2, n, ctx->err, stream);
    rc = status_of(e);
  }
  return stage_end(mv, stream, rc);
}
}  // namespace

int pc2_matvec_create(const pc2_pk* pk, size_t cols, uint32_t ebits, uint32_t window,
                      size_t rows_hint, pc2_matvec** out) {
  if (!pk || !pk->ctx || !out || cols == 0 || ebits < 1 || ebits > 64 || window > 12)
    return PC2_E_INVAL;
  *out = nullptr;
  pc2_ctx* ctx = pk->ctx;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  int w = (int)window;
  if (w == 0) {
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) return PC2_E_DEVICE;
    double best = 0;
    for (int c = 1; c <= 12; ++c) {
      if (matvec_table_bytes(pk->cls, cols, (int)ebits, c) > free_b / 4) break;
      const double nwc = (double)((ebits + c - 1) / c);
      // products per column: rows x windows (rows), windows x table entries (tables)
      const double cost = rows_hint ? nwc * ((double)rows_hint + (double)((1 << c) - 1))
                                    : (c <= 8 ? 1.0 / c : 1e300);
      if (w == 0 || cost < best) {
        w = c;
        best = cost;
      }
    }
    if (w == 0) return PC2_E_NOMEM;
  }
  pc2_matvec* mv = new (std::nothrow) pc2_matvec();
  if (!mv) return PC2_E_NOMEM;
  mv->ctx = ctx;
  mv->pk = pk;
  mv->w = w;
  mv->nw = ((int)ebits + w - 1) / w;
  mv->ebits = (int)ebits;
  mv->cols = cols;
  mv->table_bytes = matvec_table_bytes(pk->cls, cols, (int)ebits, w);
  if (rns_matvec_create(mv, rows_hint)) {
    *out = mv;
    return PC2_OK;
  }
  if (hipMalloc(&mv->tab, mv->table_bytes) != hipSuccess) {
    delete mv;
    return PC2_E_NOMEM;
  }
  mv->cap_table = resident_groups(ctx, pc2k::kernel_matvec(pk->cls, 0));
  mv->cap_apply = resident_groups(ctx, pc2k::kernel_matvec(pk->cls, 1));
  // staging for the partial products of rows_hint rows split over column
  // chunks (pc2_matvec_apply allocates nothing)
  if (rows_hint) {
    size_t nch = 1, cc = 0;
    pick_chunks(mv, rows_hint, (size_t)pc2k::RK_MAX, &nch, &cc);
    if (nch > 1) {
      mv->parts_bytes = nch * rows_hint * 8 * (size_t)pk->L;
      if (hipMalloc(&mv->parts, mv->parts_bytes) != hipSuccess) {
        (void)hipFree(mv->tab);
        delete mv;
        return PC2_E_NOMEM;
      }
    }
  }
  (void)occupancy(ctx, pk->cls, pc2k::OP_SUM);
  *out = mv;
  return PC2_OK;
}

int pc2_matvec_info(const pc2_matvec* mv, uint32_t* window, size_t* table_bytes) {
  if (!mv) return PC2_E_INVAL;
  if (window) *window = (uint32_t)mv->w;
  if (table_bytes) *table_bytes = mv->table_bytes;
  return PC2_OK;
}

int pc2_matvec_engine(const pc2_matvec* mv, int* residues, uint32_t* digits, uint32_t* blocks,
                      size_t* staging_bytes) {
  if (!mv) return PC2_E_INVAL;
  if (blocks) *blocks = (uint32_t)(mv->rdg.n ? mv->rdg.nblk : 1);
  if (residues) *residues = mv->rdg.n > 0;
  if (digits) *digits = (uint32_t)(mv->rdg.n ? mv->rdg.n : mv->nw);
  if (staging_bytes) *staging_bytes = mv->rdg.n ? mv->rstage_bytes : mv->parts_bytes;
  return PC2_OK;
}

int pc2_matvec_load(pc2_matvec* mv, const uint32_t* c, void* hip_stream) {
  if (!mv || !mv->ctx || !c) return PC2_E_INVAL;
  if (hipSetDevice(mv->ctx->device) != hipSuccess) return PC2_E_DEVICE;
  if (mv->rdg.n) {
    const int rc = rns_matvec_load(mv, c, hip_stream);
    if (!rc) mv->loaded = true;
    return rc;
  }
  const int cls = mv->pk->cls;
  const size_t epw = (size_t)pc2k::elems_per_block(cls);
  const size_t groups = (mv->cols + epw - 1) / epw * (size_t)mv->nw;
  const int grid = (int)std::max<size_t>(1, std::min<size_t>(groups, (size_t)mv->cap_table));
  int rc = status_of(pc2k::launch_mv_table(cls, grid, mv->pk->c, c, mv->cols, mv->nw, mv->w,
                                           mv->tab, mv->ctx->err, hip_stream));
  if (!rc) mv->loaded = true;
  return rc;
}

int pc2_matvec_apply(pc2_matvec* mv, const uint64_t* B, const uint32_t* alpha, uint32_t* out,
                     size_t rows, void* hip_stream) {
  if (!mv || !mv->ctx) return PC2_E_INVAL;
  if (rows == 0) return PC2_OK;
  if (!B || !out || !mv->loaded) return PC2_E_INVAL;
  pc2_ctx* ctx = mv->ctx;
  const pc2_pk* pk = mv->pk;
  const int cls = pk->cls;
  const size_t L2 = 2 * (size_t)pk->L, row_bytes = L2 * 4;
  if (alpha && alpha != out) {  // exact aliasing is allowed, partial overlap is not
    const char *a0 = (const char*)alpha, *o0 = (const char*)out;
    if (a0 < o0 + rows * row_bytes && o0 < a0 + rows * row_bytes) return PC2_E_INVAL;
  }
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  if (mv->rdg.n) return rns_matvec_apply(mv, B, alpha, out, rows, hip_stream);
  // column chunks, as many as the plan's staging holds for this many rows
  const size_t epw = (size_t)pc2k::elems_per_block(cls);
  const size_t gpc = (rows + epw - 1) / epw;
  const size_t cap = (size_t)mv->cap_apply;
  size_t nch = 1, chunk_cols = mv->cols;
  pick_chunks(mv, rows, mv->parts_bytes / (rows * row_bytes), &nch, &chunk_cols);
  const size_t groups = gpc * nch;
  const int grid = (int)std::max<size_t>(1, std::min(groups, cap));
  if (nch == 1)
    return status_of(pc2k::launch_mv_apply(cls, grid, pk->c, B, rows, mv->cols, mv->ebits,
                                           mv->nw, mv->w, mv->tab, alpha, 1, chunk_cols, out,
                                           0, ctx->err, hip_stream));
  int rc = status_of(pc2k::launch_mv_apply(cls, grid, pk->c, B, rows, mv->cols, mv->ebits,
                                           mv->nw, mv->w, mv->tab, alpha, nch, chunk_cols,
                                           mv->parts, rows * L2, ctx->err, hip_stream));
  if (rc) return rc;
  pc2k::PtrList lst{};
  for (size_t k = 0; k < nch; ++k) lst.p[k] = mv->parts + k * rows * L2;
  pc2k::Launch l{};
  l.grid = (int)std::max<size_t>(
      1, std::min(gpc, (size_t)ctx->cus * occupancy(ctx, cls, pc2k::OP_SUM)));
  l.err = ctx->err;
  l.stream = hip_stream;
  return status_of(pc2k::launch_hom_sum(cls, l, pk->c, lst, (int)nch, out, rows));
}

int pc2_matvec_destroy(pc2_matvec* mv) {
  if (!mv || !mv->ctx) return PC2_E_INVAL;
  (void)hipSetDevice(mv->ctx->device);
  (void)hipDeviceSynchronize();
  if (mv->tab) (void)hipFree(mv->tab);
  if (mv->parts) (void)hipFree(mv->parts);
  if (mv->rstage) (void)hipFree(mv->rstage);
  if (mv->done) (void)hipEventDestroy(mv->done);
  delete mv;
  return PC2_OK;
}

// ------------------------------------------------- column-split ADMM
namespace {
void* carve(char*& at, size_t bytes) {  // 256-byte aligned sub-buffers of one allocation
  void* p = at;
  at += (bytes + 255) & ~(size_t)255;
  return p;
}
int ceil_log2(size_t v) {
  int b = 0;
  while (((size_t)1 << b) < v) ++b;
  return b;
}
}  // namespace

namespace {
// Plaintexts of the node step stay below 2^(2k + 9 + log2 Nk): they must fit
// 127 bits (the inverse quantization's integers) and the key.
bool colsplit_scale_ok(const pc2_sk* sk, int Nk, int k) {
  const int pbits = 2 * k + 9 + ceil_log2((size_t)Nk);
  return k >= 1 && pbits <= 126 && pbits < (int)sk->pk.c.nbits && sk->pk.L >= 4;
}

// Quantization of every node at scale 2^k: G_k = Gamma_2(rho B_k), its row
// sums, Enc(Gamma_1(alpha_k)) (randomness rows kk Nk .. (kk + 1) Nk - 1 of the
// pool) and the nodes' mat-vec plans over (k + 4)-bit constants.  Earlier
// plans are destroyed first (after the stream's work that reads them).
int colsplit_quantize(pc2_colsplit* cs, int k, void* stream) {
  const pc2_sk* sk = cs->sk;
  const size_t nk = (size_t)cs->Nk, L2 = 2 * (size_t)sk->pk.L;
  if (!cs->mv.empty()) {
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return PC2_E_DEVICE;
    for (pc2_matvec* mv : cs->mv) pc2_matvec_destroy(mv);
    cs->mv.clear();
  }
  int rc = PC2_OK;
  for (int kk = 0; kk < cs->K && !rc; ++kk) {
    const size_t o1 = kk * nk, o2 = kk * nk * nk;
    rc = status_of(pc2k::cs_quantize_node(cs->rhoB + o2, cs->alpha + o1, cs->Nk, k, cs->G + o2,
                                          cs->R + o1, cs->g1 + o1 * 4, cs->ctx->err, stream));
    if (!rc)
      rc = pc2_encrypt(&sk->pk, cs->g1 + o1 * 4, 4, cs->r_pool + o1 * sk->pk.L,
                       cs->ahat + o1 * L2, nk, stream);
    pc2_matvec* mv = nullptr;
    if (!rc) rc = pc2_matvec_create(&sk->pk, nk, (uint32_t)(k + 4), 0, nk, &mv);
    if (!rc) cs->mv.push_back(mv);
  }
  if (!rc) cs->k = k;
  return rc;
}
}  // namespace

int pc2_colsplit_create(const pc2_sk* sk, const double* A, const double* y, uint32_t M,
                        uint32_t N, uint32_t K, double rho, uint32_t log2_scale,
                        const uint32_t* r_pool, size_t r_count, void* hip_stream,
                        pc2_colsplit** out) {
  if (!sk || !sk->ctx || !A || !y || !r_pool || !out || M == 0 || N == 0 || K == 0 ||
      N % K != 0 || !(rho > 0) || log2_scale < 1)
    return PC2_E_INVAL;
  *out = nullptr;
  const int Nk = (int)(N / K), k = (int)log2_scale, L = sk->pk.L;
  if (!colsplit_scale_ok(sk, Nk, k)) return PC2_E_UNSUPPORTED;
  if (r_count < 3 * (size_t)N) return PC2_E_INVAL;
  pc2_ctx* ctx = sk->ctx;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  pc2_colsplit* cs = new (std::nothrow) pc2_colsplit();
  if (!cs) return PC2_E_NOMEM;
  cs->ctx = ctx;
  cs->sk = sk;
  cs->M = (int)M;
  cs->N = (int)N;
  cs->K = (int)K;
  cs->Nk = Nk;
  cs->k = k;
  cs->rho = rho;
  cs->r_pool = r_pool;
  cs->r_count = r_count;
  const size_t nk = (size_t)Nk, L2 = 2 * (size_t)L, n = N;
  const size_t bytes = 256 * 16 + K * nk * 8 * 2 + K * nk * nk * 16 + K * nk * L2 * 4 +
                       n * 8 * 2 + K * 8 + n * L2 * 4 * 4 + n * L * 4 + K * nk * 16;
  void* tmp = nullptr;
  int rc = PC2_OK;
  if (hipMalloc(&cs->dev, bytes) != hipSuccess) rc = PC2_E_NOMEM;
  // setup workspace: T (Nk x 2Nk), rp (2Nk), f (Nk), aty (Nk)
  const size_t tbytes = 256 * 8 + nk * 2 * nk * 8 + nk * 4 * 8;
  if (!rc && hipMalloc(&tmp, tbytes) != hipSuccess) rc = PC2_E_NOMEM;
  if (!rc) {
    char* at = (char*)cs->dev;
    cs->alpha = (double*)carve(at, (K * nk) * sizeof(double));
    cs->rhoB = (double*)carve(at, (K * nk * nk) * sizeof(double));
    cs->G = (uint64_t*)carve(at, (K * nk * nk) * sizeof(uint64_t));
    cs->R = (uint64_t*)carve(at, (K * nk) * sizeof(uint64_t));
    cs->ahat = (uint32_t*)carve(at, (K * nk * L2) * sizeof(uint32_t));
    cs->w = (uint64_t*)carve(at, (2 * n) * sizeof(uint64_t));
    cs->S = (uint64_t*)carve(at, (size_t)K * sizeof(uint64_t));
    cs->cw = (uint32_t*)carve(at, (2 * n * L2) * sizeof(uint32_t));
    cs->c = (uint32_t*)carve(at, (n * L2) * sizeof(uint32_t));
    cs->xhat = (uint32_t*)carve(at, (n * L2) * sizeof(uint32_t));
    cs->P = (uint32_t*)carve(at, (n * L) * sizeof(uint32_t));
    cs->g1 = (uint32_t*)carve(at, (K * nk * 4) * sizeof(uint32_t));
    char* wt = (char*)tmp;
    double* T = (double*)carve(wt, (nk * 2 * nk) * sizeof(double));
    double* rp = (double*)carve(wt, (2 * nk) * sizeof(double));
    double* f = (double*)carve(wt, (nk) * sizeof(double));
    double* aty = (double*)carve(wt, (nk) * sizeof(double));
    for (int kk = 0; kk < (int)K && !rc; ++kk) {
      const size_t o1 = kk * nk, o2 = kk * nk * nk;
      rc = status_of(pc2k::cs_setup_node(A, y, (int)M, (int)N, kk * Nk, Nk, rho, T, rp, f, aty,
                                         cs->alpha + o1, cs->rhoB + o2, hip_stream));
    }
    if (!rc) rc = colsplit_quantize(cs, k, hip_stream);
    // the workspace is released once the setup has run
    if (!rc && hipStreamSynchronize((hipStream_t)hip_stream) != hipSuccess) rc = PC2_E_DEVICE;
  }
  if (tmp) (void)hipFree(tmp);
  if (rc) {
    (void)hipDeviceSynchronize();
    for (pc2_matvec* mv : cs->mv) pc2_matvec_destroy(mv);
    if (cs->dev) (void)hipFree(cs->dev);
    delete cs;
    return rc;
  }
  *out = cs;
  return PC2_OK;
}

int pc2_colsplit_set_scale(pc2_colsplit* cs, uint32_t log2_scale, void* hip_stream) {
  if (!cs || !cs->ctx) return PC2_E_INVAL;
  if (!colsplit_scale_ok(cs->sk, cs->Nk, (int)log2_scale)) return PC2_E_UNSUPPORTED;
  if (hipSetDevice(cs->ctx->device) != hipSuccess) return PC2_E_DEVICE;
  int rc = colsplit_quantize(cs, (int)log2_scale, hip_stream);
  if (!rc && hipStreamSynchronize((hipStream_t)hip_stream) != hipSuccess) rc = PC2_E_DEVICE;
  return rc;
}

int pc2_colsplit_iterate(pc2_colsplit* cs, double lambda, int quantized, double* x, double* z,
                         double* v, void* hip_stream) {
  if (!cs || !cs->ctx || !x || !z || !v || !(lambda >= 0)) return PC2_E_INVAL;
  pc2_ctx* ctx = cs->ctx;
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  const pc2_sk* sk = cs->sk;
  const pc2_pk* pk = &sk->pk;
  const int Nk = cs->Nk, L = pk->L, k = cs->k;
  const size_t nk = (size_t)Nk, L2 = 2 * (size_t)L, n = (size_t)cs->N;
  int rc = PC2_OK;
  if (quantized) {
    if (cs->mv.size() != (size_t)cs->K) return PC2_E_INVAL;  // a failed change of scale
    // master: Gamma_2(z) and Gamma_2(-v) of every node, encrypted in one launch
    // with the next 2N rows of the randomness pool (after the rows of alpha)
    const size_t span = cs->r_count - 3 * n + 1;
    const size_t base = n + (cs->iter * 2 * n) % span;
    rc = status_of(pc2k::cs_quant_zv(z, v, cs->N, cs->K, k, cs->w, cs->w + n, cs->S, ctx->err,
                                     hip_stream));
    if (!rc) rc = pc2_encrypt(pk, (const uint32_t*)cs->w, 2, cs->r_pool + base * L, cs->cw,
                              2 * n, hip_stream);
    // node k: alpha_k (+) G_k (x) (z_k (+) -v_k)  (eq. (itq2))
    if (!rc) rc = pc2_hom_add(pk, cs->cw, cs->cw + n * L2, cs->c, n, hip_stream);
    for (int kk = 0; kk < cs->K && !rc; ++kk) {
      const size_t k0 = kk * nk;
      rc = pc2_matvec_load(cs->mv[kk], cs->c + k0 * L2, hip_stream);
      if (!rc) rc = pc2_matvec_apply(cs->mv[kk], cs->G + kk * nk * nk, cs->ahat + k0 * L2,
                                     cs->xhat + k0 * L2, nk, hip_stream);
    }
    // master: decrypt every node's result and invert the quantization
    if (!rc) rc = pc2_decrypt(sk, cs->xhat, cs->P, n, hip_stream);
    if (!rc) rc = status_of(pc2k::cs_dequant(cs->P, L, cs->N, cs->K, cs->R, cs->S, k, x,
                                             ctx->err, hip_stream));
  } else {
    for (int kk = 0; kk < cs->K && !rc; ++kk) {
      const size_t k0 = kk * nk;
      rc = status_of(pc2k::cs_plain_node(cs->rhoB + kk * nk * nk, Nk, z + k0, v + k0,
                                         cs->alpha + k0, x + k0, hip_stream));
    }
  }
  if (!rc) rc = status_of(pc2k::cs_update(x, z, v, cs->N, lambda / cs->rho, hip_stream));
  if (!rc) ++cs->iter;
  return rc;
}

int pc2_colsplit_destroy(pc2_colsplit* cs) {
  if (!cs || !cs->ctx) return PC2_E_INVAL;
  (void)hipSetDevice(cs->ctx->device);
  (void)hipDeviceSynchronize();
  for (pc2_matvec* mv : cs->mv) pc2_matvec_destroy(mv);
  if (cs->dev) (void)hipFree(cs->dev);
  delete cs;
  return PC2_OK;
}

// ------------------------------------------------------------------ ADMM
int pc2_admm_create(pc2_ctx* ctx, const double* A, const double* y, uint32_t M, uint32_t N,
                    uint32_t K, double rho, void* hip_stream, pc2_admm** out) {
  if (!ctx || !A || !y || !out || M == 0 || N == 0 || K == 0 || M % K != 0 || !(rho > 0.0))
    return PC2_E_INVAL;
  *out = nullptr;
  const size_t B = M / K;
  if (B > 4096) return PC2_E_UNSUPPORTED;  // the per-node solve keeps B doubles in LDS
  if (hipSetDevice(ctx->device) != hipSuccess) return PC2_E_DEVICE;
  pc2_admm* a = new (std::nothrow) pc2_admm();
  if (!a) return PC2_E_NOMEM;
  const size_t words = K * B * B + 2 * (size_t)K * N + 2 * (size_t)K * B;
  if (hipMalloc(&a->buf, words * sizeof(double)) != hipSuccess) {
    delete a;
    return PC2_E_NOMEM;
  }
  a->ctx = ctx;
  a->A = A;
  a->N = (int)N;
  a->B = (int)B;
  a->K = (int)K;
  a->rho = rho;
  a->W = a->buf;
  a->aty = a->W + K * B * B;
  a->w = a->aty + (size_t)K * N;
  a->t = a->w + (size_t)K * N;
  a->s = a->t + (size_t)K * B;
  if (pc2k::admm_setup(A, y, (int)N, (int)B, (int)K, rho, a->W, a->aty, hip_stream) !=
      hipSuccess) {
    (void)hipFree(a->buf);
    delete a;
    return PC2_E_DEVICE;
  }
  *out = a;
  return PC2_OK;
}

int pc2_admm_local(pc2_admm* a, const double* z, const double* u, double* x, double* xu,
                   void* hip_stream) {
  if (!a || !z || !u || !x || !xu) return PC2_E_INVAL;
  if (hipSetDevice(a->ctx->device) != hipSuccess) return PC2_E_DEVICE;
  return status_of(pc2k::admm_local(a->A, a->W, a->aty, z, u, a->N, a->B, a->K, a->rho, a->w,
                                    a->t, a->s, x, xu, hip_stream));
}

int pc2_admm_consensus(pc2_admm* a, const double* sum, const double* x, double lambda, double* z,
                       double* u, void* hip_stream) {
  if (!a || !sum || !x || !z || !u || !(lambda >= 0.0)) return PC2_E_INVAL;
  if (hipSetDevice(a->ctx->device) != hipSuccess) return PC2_E_DEVICE;
  const double kappa = lambda / (a->rho * a->K);
  return status_of(pc2k::admm_consensus(sum, x, a->N, a->K, kappa, z, u, hip_stream));
}

int pc2_admm_destroy(pc2_admm* a) {
  if (!a || !a->ctx) return PC2_E_INVAL;
  (void)hipSetDevice(a->ctx->device);
  (void)hipDeviceSynchronize();
  if (a->buf) (void)hipFree(a->buf);
  delete a;
  return PC2_OK;
}

}  // extern "C"
