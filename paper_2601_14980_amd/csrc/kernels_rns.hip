// Powering kernels of the RNS engine (rns_mont.hpp) and its conversions.
//
//   k_rns_to      integers (32-bit limbs) -> residues of both bases, times a
//                 constant (a matrix product of the input's bytes)
//   k_rns_pow     runs a program of Montgomery products over groups of 32 NB
//                 elements, one group at a time per workgroup: the table of
//                 odd powers, sliding windows, the closing product
//   k_rns_smul    powers with a 64-bit exponent per element
//   k_rns_mvtab, k_rns_mv, k_rns_mvblk, k_rns_chain  fixed-base tables, rows (with
//                 constants whole, or in blocks) and the join of column chunks of
//                 the ciphertext matrix-vector product
//   k_rns_from    residues of base B -> the canonical integer mod N (sums on the
//                 vector ALUs: 0.1 ms, its carries one wavefront's serial chain)
//   k_rns_dec_finish, k_rns_garner_crt  the ends of decryption and of key-holder
//                 encryption
#include <hip/hip_runtime.h>

#include "bn_scalar.hpp"
#include "paillier_ops.hpp"
#include "rns_launch.hpp"
#include "rns_mont.hpp"
#include "wave_bn.hpp"

using namespace pc2r;
using pc2k::RnsFrom;
using pc2k::RnsMv;
using pc2k::RnsMvTab;
using pc2k::RnsPow;
using pc2k::RnsSmul;
using pc2k::RnsTo;

namespace {

// A program over the workgroup's groups: table of odd powers, sliding windows
// and the closing product.
template <class G, int SIDE>
__device__ __forceinline__ void pow_run(const RnsPow& P, RWork<G>& ws, int wave, int lane) {
  constexpr size_t GB = 2 * (size_t)G::PART * 16;  // bytes of one group's residues
  using OP = Operands<G>;
  Stepper<G, SIDE, OP> st(wave, lane);
  const int nitems = P.ngroups * P.nmod;
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const int mod = P.nmod == 2 ? (it & 1) : 0;
    const int g = P.nmod == 2 ? it >> 1 : it;
    const RConst<G> M(P.M[mod]);
    const uint32_t* ops = P.ops[mod];
    uint8_t* in = P.in[mod] + (size_t)g * GB;
    uint8_t* gm = P.gm[mod] ? P.gm[mod] + (size_t)g * GB : in;
    uint8_t* slot = P.table + ((size_t)blockIdx.x * P.entries - 1) * GB;
    auto entry = [&](uint32_t e) {
      uint8_t* p = slot + (size_t)e * GB;
      if (e == pc2k::RNS_GM) p = gm;
      if (e == 0 || e >= pc2k::RNS_OUT) p = in;
      return Buf(p, (uint32_t)GB);
    };
    auto is_mul = [](uint32_t op) { return op >> 16 == pc2k::RNS_MUL && (op & 0xFF) != pc2k::RNS_SQ; };
    auto stores = [](uint32_t op) { return ((op >> 8) & 0xFF) != pc2k::RNS_NODST; };
    uint32_t op = ops[0];
    for (int k = 1;; ++k) {
      const uint32_t next = ops[k];
      if (op >> 16 == pc2k::RNS_LOAD) {
        const Buf e = entry(op & 0xFF), y = entry(next & 0xFF);
        const bool mul = is_mul(next);
        st.load(
            M, ws,
            [&](int t, int b, bool, v4u& x) {
              const uint32_t at = (t * G::NB + b) * 1024;
              x = e.load(lane * 16, G::PART * 16 + at);
              return e.load(lane * 16, at);
            },
            [&](int t, int b, bool, const v4u& x) {
              return mul ? y.load(lane * 16, G::PART * 16 + (t * G::NB + b) * 1024) : x;
            });
      } else {
        OP o{is_mul(op), stores(op), entry(op & 0xFF), entry((op >> 8) & 0xFF)};
        OP n{is_mul(next), stores(op), entry(next & 0xFF), entry((op >> 8) & 0xFF)};
        const bool last = next >> 16 == pc2k::RNS_END;
        st.product(M, ws, o, n, last);
        if (last) break;
      }
      op = next;
    }
  }
}

template <class G>
__global__ __launch_bounds__(G::W * 64, 2) void k_rns_pow(RnsPow P) {
  __shared__ __align__(16) RWork<G> ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_constants<G>(P.M[0], ws);
  PC2R_SIDES(G, wave, (pow_run<G, SIDE>(P, ws, wave, lane)));
}

// c^k with a 64-bit k per element (fixed windows of 4 bits): in holds c, the
// result replaces its residues in base B.
template <class G, int SIDE>
__device__ __forceinline__ void smul_run(const RnsSmul& P, RWork<G>& ws, int wave, int lane) {
  constexpr size_t GB = 2 * (size_t)G::PART * 16;
  using OP = Gather<G, true>;
  Stepper<G, SIDE, OP> st(wave, lane);
  const RConst<G> M(P.M);
  const int n = lane & 31, h = lane >> 5;
  uint8_t* slot = P.table + (size_t)blockIdx.x * 16 * GB;  // entry d: c^d MA
  const Buf tab(slot, (uint32_t)(16 * GB));
  const Buf one(P.one, G::T * 64), r2(P.one + G::T * 64, G::T * 64),
      unit(P.one + 2 * G::T * 64, G::T * 64);
  for (int g = blockIdx.x; g < P.ngroups; g += gridDim.x) {
    const Buf in(P.in + (size_t)g * GB, (uint32_t)GB);
    uint64_t e[G::NB], eu = 0;
#pragma unroll
    for (int b = 0; b < G::NB; ++b) {
      const size_t i = ((size_t)g * G::NB + b) * 32 + n;
      e[b] = P.k[i < P.count ? i : P.count - 1];
      if (b == st.bu) eu = e[b];
    }
    auto entry = [&](OP& o, uint32_t d, uint32_t du, int b) {
      o.off[b] = d * (uint32_t)GB + lane * 16 + b * 1024;
      if (b == st.bu) o.offu = du * (uint32_t)GB + lane * 16 + b * 1024;
    };
    auto group = [&](OP& o) {
      o.y = tab;
      o.ts = G::NB * 1024;
      o.ps = G::PART * 16;
    };
    // entry 0: one
    st.each([&](int t, int b, bool) {
      const uint32_t at = (t * G::NB + b) * 1024;
      tab.store(one.load(h * 16, t * 32), lane * 16, at);
      tab.store(one.load(h * 16, (G::T + t) * 32), lane * 16, G::PART * 16 + at);
    });
    // entry 1: c MA^2 / MA, then products by it
    st.load(
        M, ws,
        [&](int t, int b, bool, v4u& x) {
          const uint32_t at = (t * G::NB + b) * 1024;
          x = in.load(lane * 16, G::PART * 16 + at);
          return in.load(lane * 16, at);
        },
        [&](int t, int, bool, const v4u&) { return r2.load(h * 16, (G::T + t) * 32); });
    OP o, nx;
    o.single(r2, lane);
    group(nx);
#pragma unroll
    for (int b = 0; b < G::NB; ++b) entry(nx, 1, 1, b);
    o.store = nx.store = true;
#pragma unroll 1
    for (int d = 1; d < 16; ++d) {
      o.mul = d != 2;  // (the square)
      nx.mul = d >= 2;
      o.dst = nx.dst = Buf(slot + (size_t)d * GB, (uint32_t)GB);
      st.product(M, ws, o, nx, false);
      if (d == 2) {
        group(o);
#pragma unroll
        for (int b = 0; b < G::NB; ++b) o.off[b] = nx.off[b];
        o.offu = nx.offu;
      }
    }
    // the top digit's entry, four squarings and a product per digit, and the
    // product by 1 that leaves Montgomery form
    st.load(
        M, ws,
        [&](int t, int b, bool u, v4u& x) {
          const uint32_t d = (uint32_t)((u ? eu : e[b]) >> 60);
          const uint32_t off = d * (uint32_t)GB + lane * 16, at = (t * G::NB + b) * 1024;
          x = tab.load(off, G::PART * 16 + at);
          return tab.load(off, at);
        },
        [&](int, int, bool, const v4u& x) { return x; });
    group(o);
    o.store = nx.store = o.mul = false;
    o.dst = nx.dst = in;
    int sh = 56, s = 0;  // s: squarings done for the digit at sh
#pragma unroll 1
    for (;;) {
      const bool last = sh < 0;
      nx.mul = s == 3 || (s == 4 && sh == 0);
      if (s == 3) {
        group(nx);
#pragma unroll
        for (int b = 0; b < G::NB; ++b)
          entry(nx, (uint32_t)(e[b] >> sh) & 15u, (uint32_t)(eu >> sh) & 15u, b);
      } else if (nx.mul) {
        nx.single(unit, lane);
      }
      o.store = last;
      st.product(M, ws, o, nx, last);
      if (last) break;
      o.mul = nx.mul;
      o.y = nx.y;
      o.ts = nx.ts;
      o.ps = nx.ps;
      o.offu = nx.offu;
#pragma unroll
      for (int b = 0; b < G::NB; ++b) o.off[b] = nx.off[b];
      if (++s == 5) {
        s = 0;
        sh -= 4;
      }
    }
  }
}

template <class G>
__global__ __launch_bounds__(G::W * 64, 2) void k_rns_smul(RnsSmul P) {
  __shared__ __align__(16) RWork<G> ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_constants<G>(P.M, ws);
  PC2R_SIDES(G, wave, (smul_run<G, SIDE>(P, ws, wave, lane)));
}

// Fixed-base tables of the ciphertext matrix-vector product: item (digit t,
// column group) takes the columns' c_j to c_j^(2^shift(t)) and writes its powers
// d < 2^width(t) in Montgomery form, each element's entry on its own (2 T x 32
// bytes: base B, base A).  A column with c_j >= n^2 gets zeros (entry 0, the
// Montgomery one, apart).
template <class G, int SIDE>
__device__ __forceinline__ void mvtab_run(const RnsMvTab& P, RWork<G>& ws, int wave, int lane) {
  constexpr size_t GB = 2 * (size_t)G::PART * 16;
  constexpr size_t EB = (size_t)G::T * 64;
  using OP = Scatter<G>;
  Stepper<G, SIDE, OP> st(wave, lane);
  const RConst<G> M(P.M);
  const int n = lane & 31, h = lane >> 5;
  const Buf base(P.table + (size_t)blockIdx.x * GB, (uint32_t)GB);
  const Buf one(P.one, G::T * 64), r2(P.one + G::T * 64, G::T * 64);
  const pc2k::RnsDigits D = P.dg;
  const size_t col = D.entries() * EB;
  for (int it = blockIdx.x; it < P.ngroups * D.n; it += gridDim.x) {
    const int win = D.n - 1 - it / P.ngroups, g = it % P.ngroups;  // the longest first
    const int per = 1 << D.width(win);
    const Buf in(P.in + (size_t)g * GB, (uint32_t)GB);
    uint8_t *ent[G::NB], *entu = nullptr;  // the entry before the digit's first
    bool ok[G::NB], oku = false;
    auto where = [&](int b, bool& good) -> uint8_t* {
      const size_t j = ((size_t)g * G::NB + b) * 32 + n;
      good = j < P.cols && pc2d::sc_cmp(P.c + j * P.L2, P.L2, P.n2, P.L2) < 0;
      return j < P.cols ? P.tab + j * col + D.before(win) * EB + h * 16 : nullptr;
    };
#pragma unroll
    for (int b = 0; b < G::NB; ++b) ent[b] = where(b, ok[b]);
    entu = where(st.bu, oku);
    if (win == 0 && wave == 0 && h == 0)
#pragma unroll
      for (int b = 0; b < G::NB; ++b)
        if (ent[b] && !ok[b]) atomicOr(P.err, pc2k::ERR_RANGE);
    st.each([&](int t, int b, bool u) {
      uint8_t* p = u ? entu : ent[b];
      if (!p || win != 0) return;
      *reinterpret_cast<v4u*>(p + t * 32) = one.load(h * 16, t * 32);
      *reinterpret_cast<v4u*>(p + (G::T + t) * 32) = one.load(h * 16, (G::T + t) * 32);
    });
    st.load(
        M, ws,
        [&](int t, int b, bool, v4u& x) {
          const uint32_t at = (t * G::NB + b) * 1024;
          x = in.load(lane * 16, G::PART * 16 + at);
          return in.load(lane * 16, at);
        },
        [&](int t, int, bool, const v4u&) { return r2.load(h * 16, (G::T + t) * 32); });
    // products: c MA, the squarings (the last result is entry 1), then by the base
    const int nsq = D.shift(win);
    OP o{}, nx{};
    o.dst = nx.dst = nx.y = base;
#pragma unroll 1
    for (int s = 0; s < nsq + per - 1; ++s) {
      const int d = s - nsq + 1;  // the entry that product s makes (d >= 1)
      o.mul = s == 0 || d > 2;    // (entry 2 squares the base)
      nx.mul = d >= 2;
      o.y = s == 0 ? r2 : base;
      o.store = nx.store = d >= 1;
      o.group = nx.group = d == 1;
      const size_t at = d >= 1 ? (size_t)d * EB : 0;
#pragma unroll
      for (int b = 0; b < G::NB; ++b) {
        o.p[b] = nx.p[b] = ent[b] ? ent[b] + at : nullptr;
        o.ok[b] = nx.ok[b] = ok[b];
      }
      o.pu = nx.pu = entu ? entu + at : nullptr;
      o.oku = nx.oku = oku;
      o.single = s == 0;
      nx.single = false;
      st.product(M, ws, o, nx, false);
    }
    st.flush(M, ws);
  }
}

template <class G>
__global__ __launch_bounds__(G::W * 64, 2) void k_rns_mvtab(RnsMvTab P) {
  __shared__ __align__(16) RWork<G> ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_constants<G>(P.M, ws);
  PC2R_SIDES(G, wave, (mvtab_run<G, SIDE>(P, ws, wave, lane)));
}

// Rows of the ciphertext matrix-vector product: item (column chunk, row group)
// multiplies its rows' start values (the first chunk's in place if there is an
// alpha, else 1; the other chunks' the Montgomery one) by one table entry per
// digit of each of the chunk's constants.  A digit that is zero in the
// whole group is skipped (every wavefront of a workgroup sees the same digits).
template <class G, int SIDE>
__device__ __forceinline__ void mv_run(const RnsMv& P, RWork<G>& ws, int wave, int lane) {
  constexpr size_t GB = 2 * (size_t)G::PART * 16;
  constexpr size_t EB = (size_t)G::T * 64;
  using OP = Gather<G, (G::MT <= 2)>;
  Stepper<G, SIDE, OP> st(wave, lane);
  const RConst<G> M(P.M);
  const int n = lane & 31, h = lane >> 5;
  const pc2k::RnsDigits D = P.dg;
  const uint32_t col = D.entries() * (uint32_t)EB;
  for (int it = blockIdx.x; it < P.ngroups * P.nch; it += gridDim.x) {
    const int ch = it / P.ngroups, g = it % P.ngroups;
    const Buf in(P.in + (size_t)it * GB, (uint32_t)GB);
    const bool own = ch == 0 && P.alpha;
    const Buf from(own ? P.in + (size_t)it * GB : P.one + (ch == 0 ? 2 * EB : 0),
                   own ? (uint32_t)GB : (uint32_t)EB);
    auto start = [&](int t, int b, int part) {
      return own ? from.load(lane * 16, part * G::PART * 16 + (t * G::NB + b) * 1024)
                 : from.load(h * 16, (part * G::T + t) * 32);
    };
    const size_t j0 = (size_t)ch * P.chunk_cols;
    const size_t j1 = j0 + P.chunk_cols < P.cols ? j0 + P.chunk_cols : P.cols;
    const uint64_t* row[G::NB];
    bool bad[G::NB];
    uint64_t e[G::NB], en[G::NB];  // the constants of column j, and of j + 1 in flight
#pragma unroll
    for (int b = 0; b < G::NB; ++b) {
      const size_t i = ((size_t)g * G::NB + b) * 32 + n;
      row[b] = P.B + (i < P.rows ? i : P.rows - 1) * P.cols;
      bad[b] = false;
      e[b] = 0;
      en[b] = row[b][j0];
    }
    size_t j = j0 - 1;
    int win = D.n - 1;
    // the next digit with work into o; false at the end
    auto advance = [&](OP& o) -> bool {
      for (;;) {
        if (++win == D.n) {
          if (++j == j1) return false;
          win = 0;
#pragma unroll
          for (int b = 0; b < G::NB; ++b) {
            e[b] = en[b];
            if (P.ebits < 64 && (e[b] >> P.ebits) != 0) bad[b] = true;
            if (j + 1 < j1) en[b] = row[b][j + 1];
          }
        }
        const uint32_t mask = (1u << D.width(win)) - 1, before = D.before(win);
        const int shift = D.shift(win);
        uint32_t any = 0;
#pragma unroll
        for (int b = 0; b < G::NB; ++b) {
          const uint32_t d = (uint32_t)(e[b] >> shift) & mask;
          any |= d;
          o.off[b] = (d ? before + d : 0u) * (uint32_t)EB + h * 16;
          if (b == st.bu) o.offu = o.off[b];
        }
        if (__ballot(any != 0) == 0) continue;
        o.y = Buf(P.tab + j * (size_t)col, col);
        return true;
      }
    };
    OP o, nx;
    o.ts = nx.ts = 32;
    o.ps = nx.ps = G::T * 32;
    o.dst = nx.dst = in;
    o.store = nx.store = false;
    bool more = advance(nx);
    if (more) {
      st.load(
          M, ws,
          [&](int t, int b, bool, v4u& x) {
            x = start(t, b, 1);
            return start(t, b, 0);
          },
          [&](int t, int b, bool u, const v4u&) {
            return nx.y.load(u ? nx.offu : nx.off[b], (G::T + t) * 32);
          });
    } else if (!own) {  // every digit zero: the start value stands
      st.each([&](int t, int b, bool) {
        const uint32_t at = (t * G::NB + b) * 1024;
        in.store(start(t, b, 0), lane * 16, at);
        in.store(start(t, b, 1), lane * 16, G::PART * 16 + at);
      });
    }
    o.mul = true;
#pragma unroll 1
    while (more) {
      o.y = nx.y;
      o.offu = nx.offu;
#pragma unroll
      for (int b = 0; b < G::NB; ++b) o.off[b] = nx.off[b];
      nx.mul = more = advance(nx);
      o.store = nx.store = !more;
      st.product(M, ws, o, nx, false);
    }
    st.flush(M, ws);
    if (wave == 0 && h == 0)
#pragma unroll
      for (int b = 0; b < G::NB; ++b) {
        const size_t i = ((size_t)g * G::NB + b) * 32 + n;
        if (bad[b] && i < P.rows) P.bad[i] = 1;
      }
  }
}

template <class G>
__global__ __launch_bounds__(G::W * 64, 2) void k_rns_mv(RnsMv P) {
  __shared__ __align__(16) RWork<G> ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_constants<G>(P.M, ws);
  PC2R_SIDES(G, wave, (mv_run<G, SIDE>(P, ws, wave, lane)));
}

// The same rows where the constants are taken in blocks of bits that share the
// tables (RnsDigits), for plans made for few rows, whose tables have to be small:
// item (column chunk, row group) starts from the Montgomery one, multiplies by the
// entries of a block's digits over all its columns, squares the value once per bit
// of a block and goes on with the next lower block.  The first chunk's value leaves
// Montgomery form by a last product, with its alpha or 1.  One column block: with
// two, the rows of a call are not few.  What bounds it is the chain of one item: a
// chunk's products and, in every chunk, the squarings (50 of 50-bit constants less a
// block's).  1000 columns made for one row, 2048 bits, tables / row: 0.16 / 1.8 ms
// in 17 of the 32 KB a column; with all digits (8 of 6 to 7 bits, 1.1 MB a column)
// 0.86 / 2.0; the same bytes on the VALU 3.1 / 9.4.
template <class G, int SIDE>
__device__ __forceinline__ void mvblk_run(const RnsMv& P, RWork<G>& ws, int wave, int lane) {
  static_assert(G::NB == 1, "one column block");
  constexpr size_t GB = 2 * (size_t)G::PART * 16;
  constexpr size_t EB = (size_t)G::T * 64;
  using OP = Gather<G, (G::MT <= 2)>;
  Stepper<G, SIDE, OP> st(wave, lane);
  const RConst<G> M(P.M);
  const int n = lane & 31, h = lane >> 5;
  const pc2k::RnsDigits D = P.dg;
  const uint32_t col = D.entries() * (uint32_t)EB;
  for (int it = blockIdx.x; it < P.ngroups * P.nch; it += gridDim.x) {
    const int ch = it / P.ngroups, g = it % P.ngroups;
    const Buf in(P.in + (size_t)it * GB, (uint32_t)GB), one(P.one, (uint32_t)EB);
    const size_t j0 = (size_t)ch * P.chunk_cols;
    const size_t j1 = j0 + P.chunk_cols < P.cols ? j0 + P.chunk_cols : P.cols;
    const size_t i = (size_t)g * 32 + n;
    const uint64_t* row = P.B + (i < P.rows ? i : P.rows - 1) * P.cols;
    bool bad = false, begun = false;
    uint64_t e = 0, en = row[j0];  // the constants of column j, and of j + 1 in flight
    size_t j = j0 - 1;
    int win = D.n - 1, blk = D.nblk - 1, squarings = 0;
    bool close = ch == 0;
    auto column = [&] {
      e = en;
      if (P.ebits < 64 && (e >> P.ebits) != 0) bad = true;
      if (j + 1 < j1) en = row[j + 1];
    };
    // the next product's multiplier into o; false at the end
    auto advance = [&](OP& o) -> bool {
      for (;;) {
        if (squarings) {
          --squarings;
          o.mul = false;
          return true;
        }
        if (++win == D.n) {
          win = 0;
          if (++j == j1) {
            j = j1 - 1;
            win = D.n - 1;
            if (blk > 0) {
              --blk;
              if (begun) squarings = D.bits();
              j = j0;
              win = -1;
              en = row[j0];
              column();
              continue;
            }
            o.mul = close && begun;
            if (!o.mul) return false;
            close = false;
            if (P.alpha) {
              o.y = in;
              o.ts = 1024;
              o.ps = G::PART * 16;
              o.offu = o.off[0] = lane * 16;
            } else {
              o.single(Buf(P.one + 2 * EB, (uint32_t)EB), lane);
            }
            return true;
          }
          column();
        }
        const uint32_t d =
            (uint32_t)(e >> (blk * D.bits() + D.shift(win))) & ((1u << D.width(win)) - 1);
        if (__ballot(d != 0) == 0) continue;
        o.y = Buf(P.tab + j * (size_t)col, col);
        o.offu = o.off[0] = (d ? D.before(win) + d : 0u) * (uint32_t)EB + h * 16;
        o.ts = 32;
        o.ps = G::T * 32;
        o.mul = begun = true;
        return true;
      }
    };
    OP o, nx;
    o.dst = nx.dst = in;
    o.store = nx.store = false;
    bool more = advance(nx);
    if (more) {
      st.load(
          M, ws,
          [&](int t, int, bool, v4u& x) {
            x = one.load(h * 16, (G::T + t) * 32);
            return one.load(h * 16, t * 32);
          },
          [&](int t, int, bool, const v4u&) {
            return nx.y.load(nx.off[0], (G::T + t) * 32);
          });
    } else if (!(ch == 0 && P.alpha)) {  // every digit zero: 1, or the Montgomery one
      const Buf s(P.one + (ch == 0 ? 2 * EB : 0), (uint32_t)EB);
      st.each([&](int t, int b, bool) {
        const uint32_t at = (t * G::NB + b) * 1024;
        in.store(s.load(h * 16, t * 32), lane * 16, at);
        in.store(s.load(h * 16, (G::T + t) * 32), lane * 16, G::PART * 16 + at);
      });
    }
#pragma unroll 1
    while (more) {
      o.mul = nx.mul;
      o.y = nx.y;
      o.ts = nx.ts;
      o.ps = nx.ps;
      o.offu = nx.offu;
      o.off[0] = nx.off[0];
      more = advance(nx);
      o.store = nx.store = !more;
      st.product(M, ws, o, nx, false);
    }
    st.flush(M, ws);
    if (wave == 0 && h == 0 && bad && i < P.rows) P.bad[i] = 1;
  }
}

template <class G>
__global__ __launch_bounds__(G::W * 64, 2) void k_rns_mvblk(RnsMv P) {
  __shared__ __align__(16) RWork<G> ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_constants<G>(P.M, ws);
  PC2R_SIDES(G, wave, (mvblk_run<G, SIDE>(P, ws, wave, lane)));
}

// The chunks' values of each row group multiplied together (base B of the
// result in the first chunk's place).
template <class G, int SIDE>
__device__ __forceinline__ void chain_run(const RnsMv& P, RWork<G>& ws, int wave, int lane) {
  constexpr size_t GB = 2 * (size_t)G::PART * 16;
  using OP = Operands<G>;
  Stepper<G, SIDE, OP> st(wave, lane);
  const RConst<G> M(P.M);
  for (int g = blockIdx.x; g < P.ngroups; g += gridDim.x) {
    auto value = [&](int ch) {
      return Buf(P.in + ((size_t)ch * P.ngroups + g) * GB, (uint32_t)GB);
    };
    const Buf v0 = value(0), v1 = value(1);
    st.load(
        M, ws,
        [&](int t, int b, bool, v4u& x) {
          const uint32_t at = (t * G::NB + b) * 1024;
          x = v0.load(lane * 16, G::PART * 16 + at);
          return v0.load(lane * 16, at);
        },
        [&](int t, int b, bool, const v4u&) {
          return v1.load(lane * 16, G::PART * 16 + (t * G::NB + b) * 1024);
        });
#pragma unroll 1
    for (int ch = 1; ch < P.nch; ++ch) {
      const bool last = ch + 1 == P.nch;
      OP o{true, last, value(ch), v0}, nx{!last, false, value(last ? ch : ch + 1), v0};
      st.product(M, ws, o, nx, last);
    }
  }
}

template <class G>
__global__ __launch_bounds__(G::W * 64, 2) void k_rns_chain(RnsMv P) {
  __shared__ __align__(16) RWork<G> ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_constants<G>(P.M, ws);
  PC2R_SIDES(G, wave, (chain_run<G, SIDE>(P, ws, wave, lane)));
}

// bad[i] = alpha_i >= n^2 (one lane per row; alpha null: 0)
__global__ __launch_bounds__(64) void k_rns_row_check(const uint32_t* __restrict__ alpha,
                                                      const uint32_t* __restrict__ n2, int L2,
                                                      uint32_t* __restrict__ bad, size_t rows) {
  const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x;
  if (i < rows) bad[i] = alpha ? pc2d::sc_cmp(alpha + i * L2, L2, n2, L2) >= 0 : 0;
}
// rows with bad[i] are zeroed and ERR_RANGE latched
__global__ __launch_bounds__(64) void k_rns_row_clear(const uint32_t* __restrict__ bad,
                                                      uint32_t* __restrict__ out, int L2,
                                                      size_t rows, int* err) {
  const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x;
  if (i >= rows || !bad[i]) return;
  for (int k = 0; k < L2; ++k) out[i * L2 + k] = 0u;
  atomicOr(err, pc2k::ERR_RANGE);
}

// the job and element at a position; false if there is none
__device__ __forceinline__ bool find_job(const pc2k::RnsJobs& J, uint32_t pos, pc2k::RnsJob& j,
                                         size_t& e) {
  if (J.many == nullptr) {
    j = J.one;
  } else {
    int lo = 0, hi = J.n - 1;  // the last job with pos0 <= pos (job 0 starts at 0)
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (J.many[mid].pos0 <= pos)
        lo = mid;
      else
        hi = mid - 1;
    }
    j = J.many[lo];
  }
  e = j.first + (pos - j.pos0);
  return pos - j.pos0 < j.count;
}

// Residues of both bases for 64 positions: the block's input bytes (less 128)
// go to LDS as the matrix product's column operand, and its wavefronts share
// the 2 T row tiles.  After 512 bytes a channel's sum is reduced, as 512 * 128 *
// 24500 is what 32 bits hold.  As sums on the vector ALUs this took 250 us for
// 10007 ciphertexts of 2048-bit keys and 2 x 700 us for the halves of 65536
// decryptions, now 37 and 2 x 46.
__global__ __launch_bounds__(512) void k_rns_to(RnsTo C, pc2k::RnsJobs J, bool plain, int limbs,
                                                int T, int nb, uint8_t* __restrict__ out) {
  extern __shared__ __align__(16) uint32_t lds[];
  v4u* sb = reinterpret_cast<v4u*>(lds);  // [chunk][2 column blocks][64]
  __shared__ int top;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t per = nb * 32, total = (J.npos + per - 1) / per * per;
  int kc;
  {
    const int p = threadIdx.x >> 3;
    const uint32_t pos = blockIdx.x * 64 + p;
    pc2k::RnsJob j{};
    size_t e = 0;
    const bool live = pos < J.npos && find_job(J, pos, j, e);
    if (plain) limbs = j.m_limbs;
    const int words = live ? limbs : 0;
    if (threadIdx.x == 0) top = 1;
    __syncthreads();
    if ((threadIdx.x & 7) == 0) atomicMax(&top, words);
    __syncthreads();
    kc = (top + 7) / 8;
    if (kc > C.nchunk) kc = C.nchunk;
    const uint32_t* xe = (plain ? j.m : j.x) + e * (size_t)limbs;
    for (int q = threadIdx.x & 7; q < 2 * kc; q += 8) {
      v4u v = {0u, 0u, 0u, 0u};
      if (4 * q + 3 < words) {
        __builtin_memcpy(&v, xe + 4 * q, 16);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * q + i < words) v[i] = xe[4 * q + i];
      }
      sb[((q >> 1) * 2 + (p >> 5)) * 64 + (q & 1) * 32 + (p & 31)] = v ^ 0x80808080u;
    }
  }
  kc = __builtin_amdgcn_readfirstlane(kc);
  __syncthreads();
  const v4i* s = reinterpret_cast<const v4i*>(sb) + lane;
  const int h = lane >> 5, n = lane & 31;
  for (int tt = wave; tt < 2 * T; tt += 8) {
    const bool part = tt >= T;
    const int t = part ? tt - T : tt;
    const v4i* E = reinterpret_cast<const v4i*>(C.E) + (size_t)tt * C.nchunk * 64 + lane;
    const uint32_t* k = (part ? C.ka : C.kb) + (t * 2 + h) * 24;
    const int32_t* cst = C.cst + ((size_t)kc * 2 * T + tt) * 16 + h * 8;
    v16i acc[2];
    uint32_t inv[8], negm[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      inv[u] = k[u];
      negm[u] = k[8 + u];
      acc[0][2 * u] = acc[1][2 * u] = cst[u];
      acc[0][2 * u + 1] = acc[1][2 * u + 1] = 0;
    }
    for (int c0 = 0; c0 < kc; c0 += 16) {
      const int c1 = c0 + 16 < kc ? c0 + 16 : kc;
#pragma unroll 4
      for (int c = c0; c < c1; ++c) {
        const v4i a = E[c * 64];
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, s[(c * 2 + b) * 64], acc[b], 0, 0, 0);
      }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int w = (acc[b][2 * u + 1] << 8) + acc[b][2 * u];
          acc[b][2 * u] = (int)(int16_t)reduce(w, inv[u], negm[u]);
          acc[b][2 * u + 1] = 0;
        }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t pos = blockIdx.x * 64 + b * 32;
      if (pos >= total) break;
      v4u o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = pack16((uint32_t)acc[b][4 * i], (uint32_t)acc[b][4 * i + 2]);
      const uint32_t grp = pos / per, blk = pos % per / 32;
      uint8_t* g = out + grp * pc2k::rns_group_bytes(T, nb);
      reinterpret_cast<v4u*>(g)[((size_t)tt * nb + blk) * 64 + h * 32 + n] = o;
    }
  }
}

// The value of base-B residues mod N, canonical.  A block handles 64
// elements, one per lane of every wavefront: the wavefronts form the columns
// sum_j w_j C_j[l] + beta D[l] + O[l] of eight limbs each (constants by
// scalar loads) and resolve the carries inside their block of limbs; the
// first wavefront then joins the blocks, subtracts the quotient by N, and
// all write the words.
__global__ __launch_bounds__(512) void k_rns_from(RnsFrom C, const uint8_t* __restrict__ in,
                                                  pc2k::RnsJobs J, int T, int nb,
                                                  uint32_t* __restrict__ stage, size_t stride) {
  extern __shared__ __align__(16) uint32_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = C.nblk;
  uint32_t* limb = lds;                                              // [8 nblk][64]
  int64_t* cy = reinterpret_cast<int64_t*>(lds + (size_t)nblk * 512);  // [nblk][64]
  const uint32_t pos0 = blockIdx.x * 64 + lane;
  const uint32_t pos = pos0 < J.npos ? pos0 : J.npos - 1;
  const uint32_t per = nb * 32;
  const uint32_t grp = pos / per, b = pos % per / 32, n = pos & 31;
  const v4u* g = reinterpret_cast<const v4u*>(in + grp * pc2k::rns_group_bytes(T, nb)) + b * 64 + n;
  // beta = round(sum_j w_j g_j / b_j)
  int64_t s = 0;
  for (int ts = 0; ts < 2 * T; ++ts) {
    const v4u v = g[(size_t)(ts >> 1) * nb * 64 + (ts & 1) * 32];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      s += (int64_t)(int16_t)(v[i >> 1] >> (16 * (i & 1))) * C.F[ts * 8 + i];
  }
  const int32_t beta = (int32_t)((s + ((int64_t)1 << 35)) >> 36);
  for (int k = wave; k < nblk; k += 8) {
    int64_t col[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) col[c] = (int64_t)beta * C.D[k * 8 + c] + C.O[k * 8 + c];
    const uint32_t* Ck = C.C + (size_t)k * 16 * T * 8;
    for (int ts = 0; ts < 2 * T; ++ts) {
      const v4u v = g[(size_t)(ts >> 1) * nb * 64 + (ts & 1) * 32];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int32_t w = (int16_t)(v[i >> 1] >> (16 * (i & 1)));
#pragma unroll
        for (int c = 0; c < 8; ++c)
          col[c] += (int64_t)w * (int32_t)Ck[(ts * 8 + i) * 8 + c];
      }
    }
    int64_t carry = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int64_t v = col[c] + carry;
      limb[(k * 8 + c) * 64 + lane] = (uint32_t)v & 0xFFFFFFFu;
      carry = v >> 28;
    }
    cy[k * 64 + lane] = carry;
  }
  __syncthreads();
  if (wave == 0) {
    // join the blocks: y in [0, 2^27 N)
    const int S = C.S;
    int64_t carry = 0;
    for (int k = 0; k < nblk; ++k) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int64_t v = (int64_t)limb[(k * 8 + c) * 64 + lane] + carry;
        limb[(k * 8 + c) * 64 + lane] = (uint32_t)v & 0xFFFFFFFu;
        carry = v >> 28;
      }
      carry += cy[k * 64 + lane];
    }
    // quotient from the top limbs, exact or one too small
    double top = 0.0;
    for (int i = S - 1; i >= S - 4 && i >= 0; --i)
      top = top * 268435456.0 + (double)limb[i * 64 + lane];
    double qd = top * C.ntop_inv - 0.001;
    const int64_t q = qd > 0.0 ? (int64_t)qd : 0;
    carry = 0;
    for (int i = 0; i < S; ++i) {
      const int64_t v = (int64_t)limb[i * 64 + lane] - q * (int64_t)C.N28[i] + carry;
      limb[i * 64 + lane] = (uint32_t)v & 0xFFFFFFFu;
      carry = v >> 28;
    }
    int c = 0;  // y >= N ?
    for (int i = S - 1; i >= 0 && c == 0; --i) {
      const uint32_t v = limb[i * 64 + lane];
      if (v != C.N28[i]) c = v > C.N28[i] ? 1 : -1;
    }
    if (c >= 0) {
      carry = 0;
      for (int i = 0; i < S; ++i) {
        const int64_t v = (int64_t)limb[i * 64 + lane] - (int64_t)C.N28[i] + carry;
        limb[i * 64 + lane] = (uint32_t)v & 0xFFFFFFFu;
        carry = v >> 28;
      }
    }
  }
  __syncthreads();
  // 32-bit words, coalesced over the words of an element
  for (int e = wave; e < 64; e += 8) {
    const uint32_t p = blockIdx.x * 64 + e;
    if (p >= J.npos) break;
    pc2k::RnsJob job;
    size_t el;
    if (!find_job(J, p, job, el)) continue;
    uint32_t* out = stage ? stage + p * stride : job.out + el * C.nw;
    for (int j = lane; j < C.nw; j += 64) out[j] = pc2k::rns_word28(limb + e, 8 * nblk, 64, j);
  }
}

// Input checks of an encryption, one lane per position: the element's
// ciphertext is zeroed if m >= n, r = 0 or r >= n, and ERR_RANGE latched;
// with okw the result of the check goes there instead (both halves' words).
__global__ __launch_bounds__(64) void k_rns_enc_check(pc2k::PkConst pk, pc2k::RnsJobs J,
                                                      uint32_t* __restrict__ okw, size_t stride,
                                                      int* err) {
  const uint32_t pos = blockIdx.x * 64 + threadIdx.x;
  pc2k::RnsJob j;
  size_t e;
  if (pos >= J.npos || !find_job(J, pos, j, e)) return;
  const int L = pk.L;
  const uint32_t* re = j.x + e * L;
  bool ok = pc2d::sc_cmp(j.m + e * j.m_limbs, j.m_limbs, pk.n, L) < 0 &&
            pc2d::sc_cmp(re, L, pk.n, L) < 0;
  int i = L - 1;
  while (i >= 0 && re[i] == 0) --i;
  ok = ok && i >= 0;
  if (okw) {
    okw[2 * (size_t)pos * stride] = ok;
    okw[(2 * (size_t)pos + 1) * stride] = ok;
  } else if (!ok) {
    for (int k = 0; k < 2 * L; ++k) j.out[e * 2 * L + k] = 0u;
    atomicOr(err, pc2k::ERR_RANGE);
  }
}

// The end of a decryption, one wavefront per position (n = Ls limbs): from
// y_s = c^(s-1) mod s^2 (canonical, nl words at ys + (2 pos + half) stride),
// m_s = L_s(y) h_s mod s for both primes, where L_s(y) = (y - 1) / s is u =
// (y - 1) s^-1 mod 2^(32 n) if u s == y - 1 (else c is not coprime to s), and
// m = m_q + q ((m_p - m_q) q^-1 mod p).  A lane per element waited for its
// private arrays: 3.5 of 18 ms at 2051 decryptions of 4096 bits, now
// 0.08; 65536 of 2048 bits: 1.66 ms, now 0.43.
template <int N, int NC>
__global__ __launch_bounds__(64) void k_rns_dec_finish(pc2k::SkConst sk, pc2k::RnsJobs J,
                                                       const uint32_t* __restrict__ ys,
                                                       size_t stride, int* err) {
  const uint32_t pos = blockIdx.x;
  const int lane = threadIdx.x;
  pc2k::RnsJob j;
  size_t e;
  if (!find_job(J, pos, j, e)) return;
  const int n = sk.h[0].Ls, L2 = 2 * sk.pk.L;
  bool good = pc2w::less(j.x + e * L2, sk.pk.n2.Nl, L2, lane);
  uint32_t m[2][N], s[N], sinv[N];
  // q first, so that p's constants stay for the recombination
#pragma unroll 1
  for (int half = 1; half >= 0; --half) {
    const pc2k::HalfConst& H = sk.h[half];
    uint32_t y[NC], us[NC], y1[NC], u[N], lo[N], h[N];
    pc2w::load<NC>(y, ys + (2 * (size_t)pos + half) * stride, H.s2.nl, lane);
#pragma unroll
    for (int i = 0; i < NC; ++i) us[i] = i == 0 && lane == 0 ? 1u : 0u;
    good &= pc2w::sub<NC>(y1, y, us, lane) == 0;
    pc2w::load<N>(s, H.s, n, lane);
    pc2w::load<N>(sinv, H.sinv, n, lane);
    pc2w::load<N>(h, H.H, n, lane);
#pragma unroll
    for (int i = 0; i < N; ++i) lo[i] = y1[i];
    pc2w::clip<N>(lo, n, lane);
    pc2w::mul<N>(u, lo, n, sinv, lane);
    pc2w::clip<N>(u, n, lane);
    pc2w::mul<NC>(us, u, n, s, lane);
    uint32_t diff = 0;
#pragma unroll
    for (int i = 0; i < NC; ++i) diff |= us[i] ^ y1[i];
    good &= __ballot(diff != 0) == 0;
    pc2w::mont<N, NC>(lo, u, h, s, sinv, n, lane);
#pragma unroll
    for (int i = 0; i < N; ++i) m[1][i] = half ? lo[i] : m[1][i], m[0][i] = lo[i];
  }
  uint32_t d[N], x[N], qi[N], prod[NC], add[NC];
  if (pc2w::sub<N>(d, m[0], m[1], lane)) {
    pc2w::add<N>(x, d, s, lane);
    pc2w::clip<N>(x, n, lane);
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = x[i];
  }
  pc2w::load<N>(qi, sk.QI, n, lane);
  pc2w::mont<N, NC>(x, d, qi, s, sinv, n, lane);
  pc2w::load<N>(qi, sk.h[1].s, n, lane);
  pc2w::mul<NC>(prod, x, n, qi, lane);
#pragma unroll
  for (int i = 0; i < NC; ++i) add[i] = i < N ? m[1][i < N ? i : 0] : 0u;
  uint32_t out[NC];
  pc2w::add<NC>(out, prod, add, lane);
  const int L = sk.pk.L;
#pragma unroll
  for (int i = 0; i < NC; ++i)
    if (64 * i + lane < L) j.out[e * L + 64 * i + lane] = good ? out[i] : 0u;
  for (int k = 64 * NC + lane; k < L; k += 64) j.out[e * L + k] = 0u;
  if (!good && lane == 0) atomicOr(err, pc2k::ERR_RANGE);
}

// Recombination of key-holder encryption halves, one wavefront per position (n
// = limbs of p^2): c = c_q + q^2 ((c_p - c_q) (q^2)^-1 mod p^2); the checks of
// both halves stand behind their words.  16384 of 2048 bits: 1.65 ms with a
// lane per element, now 0.11.
template <int N, int NC>
__global__ __launch_bounds__(64) void k_rns_garner_crt(pc2k::SkConst sk, pc2k::RnsJobs J,
                                                       const uint32_t* __restrict__ stage,
                                                       int* err) {
  const uint32_t pos = blockIdx.x;
  const int lane = threadIdx.x;
  pc2k::RnsJob j;
  size_t e;
  if (!find_job(J, pos, j, e)) return;
  const int n = sk.h[0].s2.nl, L2 = 2 * sk.pk.L;
  const uint32_t* cp = stage + pos * 2 * (size_t)(n + 1);
  const uint32_t* cq = cp + n + 1;
  const bool good = cp[n] && cq[n];
  uint32_t a[N], b[N], d[N], p2[N], pinv[N], x[N], prod[NC], add[NC], out[NC];
  pc2w::load<N>(a, cp, n, lane);
  pc2w::load<N>(b, cq, n, lane);
  pc2w::load<N>(p2, sk.h[0].s2.Nl, n, lane);
  pc2w::load<N>(pinv, sk.P2inv, n, lane);
  // c_q < q^2 < p^2: one conditional addition of p^2 reduces the difference
  if (pc2w::sub<N>(d, a, b, lane)) {
    pc2w::add<N>(x, d, p2, lane);
    pc2w::clip<N>(x, n, lane);
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = x[i];
  }
  pc2w::load<N>(a, sk.Q2I, n, lane);
  pc2w::mont<N, NC>(x, d, a, p2, pinv, n, lane);
  pc2w::load<N>(a, sk.h[1].s2.Nl, sk.h[1].s2.nl < n ? sk.h[1].s2.nl : n, lane);
  pc2w::mul<NC>(prod, x, n, a, lane);
#pragma unroll
  for (int i = 0; i < NC; ++i) add[i] = i < N ? b[i < N ? i : 0] : 0u;
  pc2w::add<NC>(out, prod, add, lane);
#pragma unroll
  for (int i = 0; i < NC; ++i)
    if (64 * i + lane < L2) j.out[e * L2 + 64 * i + lane] = good ? out[i] : 0u;
  for (int k = 64 * NC + lane; k < L2; k += 64) j.out[e * L2 + k] = 0u;
  if (!good && lane == 0) atomicOr(err, pc2k::ERR_RANGE);
}

}  // namespace

namespace pc2k {

// The geometries (T, NB, wavefronts, two sides), one per T and NB, and the wide
// ones beside them for T = 9: eight wavefronts as two sides finish a group
// sooner, four alone leave room for a second workgroup on the unit (65536
// decryptions of 2048 bits: 35.9 ms wide, 32.7; 8192: 5.5 wide, 6.0; 10000:
// 6.4 wide, 7.4; rns_plan chooses).
#define PC2_RNS_GEOS(D)                                                       \
  D(5, 1, 4, false) D(5, 2, 4, false) D(5, 4, 4, false)                       \
  D(9, 1, 8, false) D(9, 2, 4, false) D(9, 3, 4, false) D(9, 4, 4, false)     \
  D(13, 1, 8, false) D(13, 2, 4, false)                                       \
  D(17, 1, 8, true) D(17, 2, 8, true) D(17, 3, 8, true) D(17, 4, 8, true)     \
  D(26, 1, 8, true) D(26, 2, 8, true)                                         \
  D(34, 1, 8, true) D(34, 2, 8, true)
#define PC2_RNS_WIDE_GEOS(D) D(9, 2, 8, true) D(9, 3, 8, true) D(9, 4, 8, true)
#define PC2_RNS_CASE(T, NB, W, XY)  \
  if (t == T && nb == NB) {         \
    using G = RGeo<T, NB, W, XY>;   \
    PC2_RNS_DO;                     \
  }

const void* rns_pow_kernel(int t, int nb, bool wide) {
#define PC2_RNS_DO return (const void*)&k_rns_pow<G>
  if (wide) {
    PC2_RNS_WIDE_GEOS(PC2_RNS_CASE)
  } else {
    PC2_RNS_GEOS(PC2_RNS_CASE)
  }
#undef PC2_RNS_DO
  return nullptr;
}
// The kernels with a multiplier per element: one or two column blocks (two where
// the multipliers fit the registers), the fixed-base tables one.
const void* rns_gather_kernel(int t, int nb, int which) {
#define PC2_RNS_DO                                                                        \
  if constexpr (G::NB == 1 || (G::NB == 2 && (G::T == 5 || G::T == 9 || G::T == 17))) {   \
    if (which == RNS_SMUL) return (const void*)&k_rns_smul<G>;                            \
    if (which == RNS_MV) return (const void*)&k_rns_mv<G>;                                \
    if (which == RNS_CHAIN) return (const void*)&k_rns_chain<G>;                          \
  }                                                                                       \
  if constexpr (G::NB == 1) {                                                             \
    if (which == RNS_MVTAB) return (const void*)&k_rns_mvtab<G>;                          \
    if (which == RNS_MVBLK) return (const void*)&k_rns_mvblk<G>;                          \
  }                                                                                       \
  return nullptr
  PC2_RNS_GEOS(PC2_RNS_CASE)
#undef PC2_RNS_DO
  return nullptr;
}

int rns_pow_threads(int t, int nb, bool wide) {
#define PC2_RNS_DO return G::W * 64
  if (wide) {
    PC2_RNS_WIDE_GEOS(PC2_RNS_CASE)
  } else {
    PC2_RNS_GEOS(PC2_RNS_CASE)
  }
#undef PC2_RNS_DO
  return 0;
}

hipError_t launch_rns_to(const RnsTo& c, int T, int nb, const RnsJobs& jobs, bool plain,
                         int limbs, uint8_t* out, void* stream) {
  const uint32_t per = nb * 32;
  const uint32_t total = (jobs.npos + per - 1) / per * per;
  const int chunks = plain ? c.nchunk : std::min(c.nchunk, (limbs + 7) / 8);
  hipLaunchKernelGGL(k_rns_to, dim3((total + 63) / 64), dim3(512), (size_t)chunks * 2048,
                     (hipStream_t)stream, c, jobs, plain, limbs, T, nb, out);
  return hipGetLastError();
}

hipError_t launch_rns_pow(int t, int nb, bool wide, int grid, const RnsPow& p, void* stream) {
  const void* k = rns_pow_kernel(t, nb, wide);
  if (!k) return hipErrorInvalidValue;
  void* args[] = {(void*)&p};
  return hipLaunchKernel(k, dim3(grid), dim3(rns_pow_threads(t, nb, wide)), args, 0,
                         (hipStream_t)stream);
}

hipError_t launch_rns_gather(int t, int nb, int which, int grid, const void* p, void* stream) {
  const void* k = rns_gather_kernel(t, nb, which);
  if (!k) return hipErrorInvalidValue;
  void* args[] = {const_cast<void*>(p)};
  return hipLaunchKernel(k, dim3(grid), dim3(rns_pow_threads(t, nb, false)), args, 0,
                         (hipStream_t)stream);
}
hipError_t launch_rns_row_check(const uint32_t* x, const uint32_t* n2, int L2, uint32_t* bad,
                                size_t rows, void* stream) {
  hipLaunchKernelGGL(k_rns_row_check, dim3((unsigned)((rows + 63) / 64)), dim3(64), 0,
                     (hipStream_t)stream, x, n2, L2, bad, rows);
  return hipGetLastError();
}
hipError_t launch_rns_row_clear(const uint32_t* bad, uint32_t* out, int L2, size_t rows, int* err,
                                void* stream) {
  hipLaunchKernelGGL(k_rns_row_clear, dim3((unsigned)((rows + 63) / 64)), dim3(64), 0,
                     (hipStream_t)stream, bad, out, L2, rows, err);
  return hipGetLastError();
}

hipError_t launch_rns_from(const RnsFrom& c, int T, int nb, const uint8_t* in,
                           const RnsJobs& jobs, uint32_t* stage, size_t stride, void* stream) {
  const size_t lds = (size_t)c.nblk * (512 * 4 + 64 * 8);
  hipLaunchKernelGGL(k_rns_from, dim3((jobs.npos + 63) / 64), dim3(512), lds,
                     (hipStream_t)stream, c, in, jobs, T, nb, stage, stride);
  return hipGetLastError();
}

hipError_t launch_rns_enc_check(const PkConst& pk, const RnsJobs& jobs, uint32_t* okw,
                                size_t stride, int* err, void* stream) {
  hipLaunchKernelGGL(k_rns_enc_check, dim3((jobs.npos + 63) / 64), dim3(64), 0,
                     (hipStream_t)stream, pk, jobs, okw, stride, err);
  return hipGetLastError();
}

// kernel<N, NC>: N registers hold n limbs, NC 2 n
#define PC2_RNS_WIDE(n, KERNEL, GRID, ...)                                                \
  do {                                                                                    \
    const dim3 g(GRID), b(64);                                                            \
    if ((n) <= 32)                                                                        \
      hipLaunchKernelGGL((KERNEL<1, 1>), g, b, 0, (hipStream_t)stream, __VA_ARGS__);      \
    else if ((n) <= 64)                                                                   \
      hipLaunchKernelGGL((KERNEL<1, 2>), g, b, 0, (hipStream_t)stream, __VA_ARGS__);      \
    else if ((n) <= 96)                                                                   \
      hipLaunchKernelGGL((KERNEL<2, 3>), g, b, 0, (hipStream_t)stream, __VA_ARGS__);      \
    else if ((n) <= 128)                                                                  \
      hipLaunchKernelGGL((KERNEL<2, 4>), g, b, 0, (hipStream_t)stream, __VA_ARGS__);      \
    else if ((n) <= 160)                                                                  \
      hipLaunchKernelGGL((KERNEL<3, 5>), g, b, 0, (hipStream_t)stream, __VA_ARGS__);      \
    else                                                                                  \
      return hipErrorInvalidValue;                                                        \
  } while (0)

hipError_t launch_rns_dec_finish(const SkConst& sk, const RnsJobs& jobs, const uint32_t* ys,
                                 size_t stride, int* err, void* stream) {
  PC2_RNS_WIDE(sk.h[0].Ls, k_rns_dec_finish, jobs.npos, sk, jobs, ys, stride, err);
  return hipGetLastError();
}

hipError_t launch_rns_garner_crt(const SkConst& sk, const RnsJobs& jobs, const uint32_t* stage,
                                 int* err, void* stream) {
  PC2_RNS_WIDE(sk.h[0].s2.nl, k_rns_garner_crt, jobs.npos, sk, jobs, stage, err);
  return hipGetLastError();
}

}  // namespace pc2k
