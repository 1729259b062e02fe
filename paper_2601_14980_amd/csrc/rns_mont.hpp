// Montgomery products in a residue number system, batched over elements on
// the i8 matrix cores of gfx950.
//
// A value X (any representative of a residue mod N, |X| < 2^26 N) is held by
// its residues x_i = X mod a_i in base A and w_j = X s_j mod b_j in base B
// (s_j = MA^-1 mod b_j), each centred and 16 bits wide.  A product
// Z = (X Y + q N) / MA, q = -X Y N^-1 mod MA, is
//
//     xi_i = x_i y_i mod a_i                                     (16 T products)
//     w_j  = w_j y_j + sum_i xi_i E1[j][i]       mod b_j         (a matrix product)
//     z_i  = sum_j w_j E2[i][j] - beta MB        mod a_i         (a matrix product)
//
// with constant matrices, the same for every element: E1[j][i] =
// k_i N s_j / a_i mod b_j, k_i = -N^-1 (MA/a_i)^-1 mod a_i, and E2[i][j] =
// g_j MB/b_j mod a_i, g_j = MA (MB/b_j)^-1 mod b_j.  q = sum_i xi_i k_i MA/a_i
// is not reduced mod MA: it only adds multiples of N, |Z| < 2^23 N.  The
// second extension is exact: beta = round(sum_j w_j g_j / b_j), a fixed-point
// sum whose error (< 0.2) and the remainder |Z| / MB (< 2^-4) cannot reach
// one half.  So the quadratic part of a modular product is two dense int8
// matrix products whose left operand is shared by the whole device, and what
// belongs to an element alone is linear in its length: no limb product, no
// carry and no lane exchange.
//
// Matrix layout (v_mfma_i32_32x32x32_i8).  A residue r is two signed bytes,
// the low one with its top bit flipped (r = 256 h + l + 128).  For xi the 128
// is added to x y before its reduction, so that 256 h + l is the residue; for
// w, which is also read back as a factor, the 128 sum_j E2[i][j] sits in the
// initial accumulators of the second extension.  Both bytes of a
// channel are rows of the right operand: the low byte meets E, the high byte
// 256 E mod m.  The left operand's rows are the low and the high byte of a
// channel's constants, in adjacent accumulators of one lane, so that
// sum = c0 + 256 c1.  Lane (n, h) of an output tile holds the eight channels
// 16 t + 8 h + 0..7 of element n; packed to 16 bits they are exactly the 16
// bytes that the lane has to supply as right operand of the next product's
// chunk t.  The residues therefore stay in one LDS slot per lane and tile
// (16 bytes, linear, no bank conflict), written by the wavefront that owns
// the tile and read by all.
//
// Reductions are centred: q = round(W / m) in float (W < 2^31, so the
// quotient is off by less than 2^-6), r = W - q m of which the low 16 bits
// are kept, |r| < 0.52 m < 2^15.  The bounds on W hold for every input: the
// host checks sum_i |E[j][i]| for each row when the key is made.
//
// Work split.  A workgroup of W wavefronts takes NB column blocks of 32
// elements; the output tiles are split over the wavefronts, so each fragment
// of the constant matrices (1 KB) is read from L2 by one wavefront only and
// serves NB matrix instructions, while the LDS serves the elements' residues:
// two tiles by four column blocks per wavefront read 1 KB of LDS per two
// matrix instructions, half of the LDS rate at full matrix rate.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rns_types.hpp"

namespace pc2r {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// T tiles, NB column blocks, W wavefronts.  A wavefront owns MT tiles over all
// column blocks; each of the R = T - W MT tiles left is split into its NB
// column blocks ("units"), one per wavefront.
//
// XY: the wavefronts 0..3 (X) and 4..7 (Y; one of each per SIMD) run half a
// phase apart, so that one's reductions (vector ALUs) run beside the other's
// matrix instructions.  X owns tiles 0 .. NX - 1 and starts a phase with the
// chunks of its own tiles while Y still reduces the previous phase; Y joins
// for the whole matrix product, and reduces while X has gone on.
template <int T_, int NB_, int W_, bool XY_>
struct RGeo {
  static constexpr int T = T_, NB = NB_, W = W_;
  static constexpr bool XY = XY_;
  static constexpr int MT = T_ / W_;
  static constexpr int R = T_ - W_ * MT;               // tiles split into units
  static constexpr int RX = XY_ ? (R + 1) / 2 : R;     // ... of X
  static constexpr int RY = R - RX;
  static constexpr int NX = XY_ ? W_ / 2 * MT + RX : T_;  // tiles of X
  static constexpr int PART = T_ * NB_ * 64;           // 16-byte slots of one base
  // the channel constants (448 bytes a tile) in LDS beside the residues where
  // they fit without costing a resident workgroup
  static constexpr int LDS = 2 * PART * 16 + NB_ * 512;
  static constexpr int WG = W_ == 8 ? 1 : 2;           // workgroups a CU is planned for
  static constexpr bool KL = (LDS + T_ * 448) * WG <= 160 * 1024;
  static_assert(MT >= 1 && (!XY_ || W_ == 8), "wavefronts");
  static_assert(MT <= pc2k::rns_mt(T_), "the bound on a lane's sums of beta");
  static_assert(RX * NB_ <= (XY_ ? W_ / 2 : W_) && RY * NB_ <= W_ / 2, "one unit a wavefront");
};

template <class G>
struct RWork {
  v4u xi[G::PART];                          // xi (base A), low bytes flipped
  v4u om[G::PART];                          // w (base B), low bytes flipped
  unsigned long long beta[2][G::NB * 32];   // sum_j w_j g_j / b_j in 2^-25
  v4u kb[G::KL ? G::T * 12 : 1], ka[G::KL ? G::T * 12 : 1];  // channel constants
  v4u c2[G::KL ? G::T * 4 : 1];             // initial sums of the second extension
};

constexpr uint32_t FLIP = 0x00800080u;
constexpr int BIAS = 128;  // FLIP's value in a residue

__device__ __forceinline__ uint32_t pack16(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
// signed 16-bit halves of packed words
template <int H>
__device__ __forceinline__ int mad16(uint32_t a, uint32_t b, int c) {
  int r;
  if constexpr (H == 0)
    asm("v_mad_i32_i16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  else
    asm("v_mad_i32_i16 %0, %1, %2, %3 op_sel:[1,1,0,0]" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// a b + bias (a scalar register)
template <int H>
__device__ __forceinline__ int mul16_biased(uint32_t a, uint32_t b, int bias) {
  int r;
  if constexpr (H == 0)
    asm("v_mad_i32_i16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(bias));
  else
    asm("v_mad_i32_i16 %0, %1, %2, %3 op_sel:[1,1,0,0]" : "=v"(r) : "v"(a), "v"(b), "s"(bias));
  return r;
}
// W mod m, centred, in the low 16 bits (the high bits are not meaningful):
// the float sum has round(W / m) + 2^22 in its low 24 bits, and 2^22 m only
// touches bits 22 and up.
__device__ __forceinline__ uint32_t reduce(int W, uint32_t inv, uint32_t negm) {
  const float g = __builtin_fmaf((float)W, __builtin_bit_cast(float, inv), 12582912.0f);
  uint32_t r;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(g), "v"(negm), "v"(W));
  return r;
}

// Workgroup barrier for LDS data only (every global array of the engine is
// read by the lane that wrote it).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A global array by buffer addressing: a uniform (scalar) offset beside one
// lane offset, so that no vector register holds an address.
struct Buf {
  __amdgpu_buffer_rsrc_t r;
  Buf() = default;
  __device__ __forceinline__ Buf(const void* p, uint32_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000)) {}
  __device__ __forceinline__ v4u load(uint32_t lane_off, uint32_t off) const {
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)off, 0);
  }
  // (no scalar offset here: with one the compiler takes a wide store's data
  // as safe to overwrite in the next vector instruction, which on this chip
  // it is not -- the last lanes stored the new value)
  __device__ __forceinline__ void store(v4u v, uint32_t lane_off, uint32_t off) const {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)(lane_off + off), 0, 0);
  }
};

// The constants of a modulus.
template <class G>
struct RConst {
  Buf E1, E2, c2, kb, ka;
  __device__ __forceinline__ explicit RConst(const pc2k::RnsMod& M)
      : E1(M.E1, G::T * G::T * 1024), E2(M.E2, G::T * G::T * 1024), c2(M.c2, G::T * 64),
        kb(M.kb, G::T * 192), ka(M.ka, G::T * 192) {}
};

// the channel constants to LDS (they depend on T alone, not on the modulus)
template <class G>
__device__ __forceinline__ void load_constants(const pc2k::RnsMod& M, RWork<G>& ws) {
  if constexpr (G::KL) {
    const v4u *kb = reinterpret_cast<const v4u*>(M.kb), *ka = reinterpret_cast<const v4u*>(M.ka),
              *c2 = reinterpret_cast<const v4u*>(M.c2);
    for (int i = threadIdx.x; i < G::T * 12; i += G::W * 64) {
      ws.kb[i] = kb[i];
      ws.ka[i] = ka[i];
      if (i < G::T * 4) ws.c2[i] = c2[i];
    }
  }
}

// Channel constants of one tile half: three groups of eight words, from LDS
// (loc) or global memory.
template <class G>
struct ChanConst {
  uint32_t w[24];
  __device__ __forceinline__ void load(const v4u* loc, const Buf& k, int t, int lane) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      v4u v;
      if constexpr (G::KL)
        v = loc[(t * 2 + (lane >> 5)) * 6 + i];
      else
        v = k.load((lane >> 5) * 96, t * 192 + 16 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[4 * i + j] = v[j];
    }
  }
};

// A wavefront's share of a phase: the tiles t0 .. t0 + MT - 1 over all column
// blocks and (U) the unit (tu, bu), with its accumulators and the fragments of
// the constant matrix in flight (PD chunks ahead).
template <class G, bool U>
struct Share {
  static constexpr int T = G::T, MT = G::MT, NB = G::NB, PD = 3, MA = MT + (U ? 1 : 0);
  v16i acc[MT][NB];
  v16i accu;
  v4i a[PD][MA];
  ChanConst<G> k;  // of tile t0, loaded ahead of the reductions

  // fragment row of accumulator m (opaque, so that the scalar offsets of a
  // product's fragments are formed where they are used and not kept)
  __device__ __forceinline__ static uint32_t row(int t0, int tu, int m) {
    uint32_t r = (uint32_t)(m < MT ? t0 + m : tu) * (T * 1024);
    asm volatile("" : "+s"(r));
    return r;
  }
  // issue the first loads of a product with E
  __device__ __forceinline__ void prime(const Buf& E, int t0, int tu, int lane) {
    uint32_t at[MA];
#pragma unroll
    for (int m = 0; m < MA; ++m) at[m] = row(t0, tu, m);
#pragma unroll
    for (int c = 0; c < PD; ++c)
#pragma unroll
      for (int m = 0; m < MA; ++m)
        a[c][m] = __builtin_bit_cast(v4i, E.load(lane * 16, at[m] + c * 1024));
  }
  // initial sums: zero, or (CST) the second extension's constants
  template <bool CST>
  __device__ __forceinline__ void init(const v4u* loc, const Buf& cst, int t0, int tu, int lane) {
#pragma unroll
    for (int m = 0; m < MA; ++m) {
      v16i c0{};
      if constexpr (CST) {
        const int t = m < MT ? t0 + m : tu;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          v4u v;
          if constexpr (G::KL)
            v = loc[(t * 2 + (lane >> 5)) * 2 + i];
          else
            v = cst.load((lane >> 5) * 32, t * 64 + 16 * i);
#pragma unroll
          for (int j = 0; j < 4; ++j) c0[8 * i + 2 * j] = (int)v[j];
        }
      }
      if (m < MT)
        acc[m][0] = c0;
      else
        accu = c0;
    }
  }
  // chunks C0 .. C1 - 1 of the product; src: the residues in LDS; kc: the
  // channel constants that the reductions after the last chunk need
  template <int C0, int C1>
  __device__ __forceinline__ void part(const Buf& E, const v4u* kloc, const Buf& kc,
                                       const v4u* src, int t0, int tu, int bu, int lane) {
    const v4i* s = reinterpret_cast<const v4i*>(src) + lane;
    const v4i* su = s + bu * 64;
    uint32_t at[MA];
#pragma unroll
    for (int m = 0; m < MA; ++m) at[m] = row(t0, tu, m);
    v4i y[2][NB], yu[2];
#pragma unroll
    for (int b = 0; b < NB; ++b) y[C0 & 1][b] = s[(C0 * NB + b) * 64];
    if constexpr (U) yu[C0 & 1] = su[C0 * NB * 64];
#pragma unroll
    for (int c = C0; c < C1; ++c) {
      if (c + 1 < C1) {
#pragma unroll
        for (int b = 0; b < NB; ++b) y[(c + 1) & 1][b] = s[((c + 1) * NB + b) * 64];
        if constexpr (U) yu[(c + 1) & 1] = su[(c + 1) * NB * 64];
      }
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int b = NB - 1; b >= 0; --b)
          acc[m][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
              a[c % PD][m], y[c & 1][b], c == 0 ? acc[m][0] : acc[m][b], 0, 0, 0);
      if constexpr (U)
        accu = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[c % PD][MT], yu[c & 1], accu, 0, 0, 0);
      if (c + PD < T) {
#pragma unroll
        for (int m = 0; m < MA; ++m)
          a[c % PD][m] = __builtin_bit_cast(v4i, E.load(lane * 16, at[m] + (c + PD) * 1024));
      }
      if (c == T - 2) k.load(kloc, kc, t0, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// The multiplier of a product (mul; else the running value itself) and the
// destination of a copy of its result (store), both in a group's layout.
// pre_b / pre_a run before the matrix product whose reductions use the
// multiplier's residues in that base, f_b / f_a in them (m: the tile's index in
// the wavefront's share, MT for its unit).
template <class G>
struct Operands {
  bool mul, store;
  Buf y, dst;
  __device__ __forceinline__ void pre_b(int, int, int, int) {}
  __device__ __forceinline__ void pre_a(int, int, int, int) {}
  template <int NBN>
  __device__ __forceinline__ void f_b(v4u (&f)[NBN], int, int t, int nb0, int lane) const {
#pragma unroll
    for (int b = 0; b < NBN; ++b) f[b] = y.load(lane * 16, ((t * G::NB + nb0 + b) * 64) * 16);
  }
  template <int NBN>
  __device__ __forceinline__ void f_a(v4u (&f)[NBN], int, int t, int nb0, int lane) const {
#pragma unroll
    for (int b = 0; b < NBN; ++b)
      f[b] = y.load(lane * 16, (G::PART + (t * G::NB + nb0 + b) * 64) * 16);
  }
  __device__ __forceinline__ void st_b(const v4u& z, int t, int b, bool, int lane) const {
    dst.store(z, lane * 16, ((t * G::NB + b) * 64) * 16);
  }
  __device__ __forceinline__ void st_a(const v4u& z, int t, int b, bool, int lane) const {
    dst.store(z, lane * 16, (G::PART + (t * G::NB + b) * 64) * 16);
  }
};

// A multiplier per element: lane's element of column block b has its residues
// at y + off[b] (offu: of the unit's block), tile stride ts, base A at ps.
// PRE (where the registers allow it): they are loaded a matrix product ahead
// of their use, which hides the latency of entries that come from HBM.
template <class G, bool PRE>
struct Gather {
  bool mul, store;
  Buf y, dst;
  uint32_t off[G::NB], offu, ts, ps;
  v4u pre[PRE ? G::MT + 1 : 1][G::NB];
  __device__ __forceinline__ void pre_any(uint32_t part, int t0, bool unit, int tu) {
    if (!PRE || !mul) return;
#pragma unroll
    for (int m = 0; m < G::MT; ++m)
#pragma unroll
      for (int b = 0; b < G::NB; ++b) pre[m][b] = y.load(off[b], part + (t0 + m) * ts);
    if (unit) pre[PRE ? G::MT : 0][0] = y.load(offu, part + tu * ts);
  }
  __device__ __forceinline__ void pre_b(int t0, bool unit, int tu, int) { pre_any(0, t0, unit, tu); }
  __device__ __forceinline__ void pre_a(int t0, bool unit, int tu, int) {
    pre_any(ps, t0, unit, tu);
  }
  template <int NBN>
  __device__ __forceinline__ void get(v4u (&f)[NBN], int m, int t, uint32_t part) const {
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
      if constexpr (PRE)
        f[b] = pre[m][b];
      else
        f[b] = y.load(m == G::MT ? offu : off[b], part + t * ts);
    }
  }
  template <int NBN>
  __device__ __forceinline__ void f_b(v4u (&f)[NBN], int m, int t, int, int) const {
    get(f, m, t, 0);
  }
  template <int NBN>
  __device__ __forceinline__ void f_a(v4u (&f)[NBN], int m, int t, int, int) const {
    get(f, m, t, ps);
  }
  // one entry for every element
  __device__ __forceinline__ void single(const Buf& e, int lane) {
    y = e;
    ts = 32;
    ps = G::T * 32;
    offu = (lane >> 5) * 16;
#pragma unroll
    for (int b = 0; b < G::NB; ++b) off[b] = offu;
  }
  __device__ __forceinline__ void st_b(const v4u& z, int t, int b, bool, int lane) const {
    dst.store(z, lane * 16, ((t * G::NB + b) * 64) * 16);
  }
  __device__ __forceinline__ void st_a(const v4u& z, int t, int b, bool, int lane) const {
    dst.store(z, lane * 16, (G::PART + (t * G::NB + b) * 64) * 16);
  }
};

// The multiplier as in Operands; the results go to an entry of each element's
// own at p[b] (pu: of the unit's block; null: none), zero where ok is not
// set, and (group) to dst as well.
template <class G>
struct Scatter : Operands<G> {
  bool group, single;  // single: y is one entry, the same for every element
  uint8_t* p[G::NB];
  uint8_t* pu;
  bool ok[G::NB], oku;
  template <int NBN>
  __device__ __forceinline__ void f_b(v4u (&f)[NBN], int m, int t, int nb0, int lane) const {
    if (!single) return Operands<G>::template f_b<NBN>(f, m, t, nb0, lane);
#pragma unroll
    for (int b = 0; b < NBN; ++b) f[b] = this->y.load((lane >> 5) * 16, t * 32);
  }
  __device__ __forceinline__ void put(const v4u& z, uint32_t at, int b, bool unit) const {
    uint8_t* q = unit ? pu : p[b];
    const bool good = unit ? oku : ok[b];
    if (q) *reinterpret_cast<v4u*>(q + at) = good ? z : v4u{0u, 0u, 0u, 0u};
  }
  __device__ __forceinline__ void st_b(const v4u& z, int t, int b, bool unit, int lane) const {
    if (group) Operands<G>::st_b(z, t, b, unit, lane);
    put(z, t * 32, b, unit);
  }
  __device__ __forceinline__ void st_a(const v4u& z, int t, int b, bool unit, int lane) const {
    if (group) Operands<G>::st_a(z, t, b, unit, lane);
    put(z, (G::T + t) * 32, b, unit);
  }
};

// The reductions after A -> B, tile t over column blocks nb0 ..: w <- w y +
// acc, and the tile's share of beta into s1, s2.
template <class G, int NBN, class OP>
__device__ __forceinline__ void reduce_b(const v16i (&acc)[NBN], const ChanConst<G>& k, RWork<G>& ws,
                                         int m, int t, int nb0, const OP& o, int (&s1)[NBN],
                                         int (&s2)[NBN], int lane) {
  const int at = (t * G::NB + nb0) * 64;
  v4u x[NBN], f[NBN];
#pragma unroll
  for (int b = 0; b < NBN; ++b) x[b] = f[b] = ws.om[at + b * 64 + lane] ^ FLIP;
  if (o.mul) o.template f_b<NBN>(f, m, t, nb0, lane);
#pragma unroll
  for (int b = 0; b < NBN; ++b) {
    v4u z;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t r0 =
          reduce(mad16<0>(x[b][i], f[b][i], (acc[b][4 * i + 1] << 8) + acc[b][4 * i]),
                 k.w[2 * i], k.w[8 + 2 * i]);
      const uint32_t r1 =
          reduce(mad16<1>(x[b][i], f[b][i], (acc[b][4 * i + 3] << 8) + acc[b][4 * i + 2]),
                 k.w[2 * i + 1], k.w[9 + 2 * i]);
      z[i] = pack16(r0, r1);
      s1[b] = mad16<1>(z[i], k.w[16 + i], mad16<0>(z[i], k.w[16 + i], s1[b]));
      s2[b] = mad16<1>(z[i], k.w[20 + i], mad16<0>(z[i], k.w[20 + i], s2[b]));
    }
    if (o.store) o.st_b(z, t, nb0 + b, m == G::MT, lane);
    ws.om[at + b * 64 + lane] = z ^ FLIP;
  }
}
template <class G>
__device__ __forceinline__ void add_beta(RWork<G>& ws, int par, int b, int s1, int s2, int lane) {
  const long long s = (long long)s1 * 8192 + s2;
  __hip_atomic_fetch_add(&ws.beta[par][b * 32 + (lane & 31)], (unsigned long long)s,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class G, bool U, class OP>
__device__ __forceinline__ void finish_b(Share<G, U>& h, const RConst<G>& M, RWork<G>& ws,
                                         int par, int t0, bool unit, int tu, int bu,
                                         const OP& o, int lane) {
  int s1[G::NB] = {}, s2[G::NB] = {};
  ChanConst<G> k[2];
  k[0] = h.k;
#pragma unroll
  for (int m = 0; m < G::MT; ++m) {
    if (m + 1 < G::MT)
      k[(m + 1) & 1].load(ws.kb, M.kb, t0 + m + 1, lane);
    else if (U)
      k[(m + 1) & 1].load(ws.kb, M.kb, tu, lane);
    reduce_b<G, G::NB>(h.acc[m], k[m & 1], ws, m, t0 + m, 0, o, s1, s2, lane);
  }
#pragma unroll
  for (int b = 0; b < G::NB; ++b) add_beta<G>(ws, par, b, s1[b], s2[b], lane);
  if constexpr (U) {
    if (unit) {
      int u1[1] = {}, u2[1] = {};
      const v16i au[1] = {h.accu};
      reduce_b<G, 1>(au, k[G::MT & 1], ws, G::MT, tu, bu, o, u1, u2, lane);
      add_beta<G>(ws, par, bu, u1[0], u2[0], lane);
    }
  }
}

// beta of column block b, as the pair (low 12 bits, rest)
template <class G>
__device__ __forceinline__ uint32_t read_beta(const RWork<G>& ws, int par, int b, int lane) {
  const long long s = (long long)ws.beta[par][b * 32 + (lane & 31)];
  const int beta = (int)((s + (1 << 24)) >> 25);
  const int lo = (int)((uint32_t)beta << 20) >> 20;
  return pack16((uint32_t)lo, (uint32_t)((beta - lo) >> 12));
}

// The reductions after B -> A: x <- acc - beta MB, then xi <- x y for the next
// product, whose multiplier o names (o.dst: where this product's x goes).
template <class G, int NBN, class OP>
__device__ __forceinline__ void reduce_a(const v16i (&acc)[NBN], const uint32_t (&bp)[NBN],
                                         const ChanConst<G>& k, RWork<G>& ws, int m, int t,
                                         int nb0, const OP& o, int lane) {
  const int at = (t * G::NB + nb0) * 64;
  v4u x[NBN], f[NBN];
#pragma unroll
  for (int b = 0; b < NBN; ++b) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t r[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        r[j] = reduce(mad16<1>(bp[b], k.w[16 + 2 * i + j],
                               mad16<0>(bp[b], k.w[16 + 2 * i + j],
                                        (acc[b][4 * i + 2 * j + 1] << 8) +
                                            acc[b][4 * i + 2 * j])),
                      k.w[2 * i + j], k.w[8 + 2 * i + j]);
      x[b][i] = pack16(r[0], r[1]);
    }
    f[b] = x[b];
  }
  if (o.store) {
#pragma unroll
    for (int b = 0; b < NBN; ++b) o.st_a(x[b], t, nb0 + b, m == G::MT, lane);
  }
  if (o.mul) o.template f_a<NBN>(f, m, t, nb0, lane);
#pragma unroll
  for (int b = 0; b < NBN; ++b) {
    v4u z;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      z[i] = pack16(reduce(mul16_biased<0>(x[b][i], f[b][i], BIAS), k.w[2 * i], k.w[8 + 2 * i]),
                    reduce(mul16_biased<1>(x[b][i], f[b][i], BIAS), k.w[2 * i + 1], k.w[9 + 2 * i]));
    ws.xi[at + b * 64 + lane] = z ^ FLIP;
  }
}
template <class G, bool U, class OP>
__device__ __forceinline__ void finish_a(Share<G, U>& h, const RConst<G>& M, RWork<G>& ws,
                                         int par, int t0, bool unit, int tu, int bu,
                                         const OP& o, int lane) {
  uint32_t bp[G::NB];
#pragma unroll
  for (int b = 0; b < G::NB; ++b) bp[b] = read_beta<G>(ws, par, b, lane);
  ChanConst<G> k[2];
  k[0] = h.k;
#pragma unroll
  for (int m = 0; m < G::MT; ++m) {
    if (m + 1 < G::MT)
      k[(m + 1) & 1].load(ws.ka, M.ka, t0 + m + 1, lane);
    else if (U)
      k[(m + 1) & 1].load(ws.ka, M.ka, tu, lane);
    reduce_a<G, G::NB>(h.acc[m], bp, k[m & 1], ws, m, t0 + m, 0, o, lane);
  }
  if constexpr (U) {
    if (unit) {
      const uint32_t bpu[1] = {read_beta<G>(ws, par, bu, lane)};
      const v16i au[1] = {h.accu};
      reduce_a<G, 1>(au, bpu, k[G::MT & 1], ws, G::MT, tu, bu, o, lane);
    }
  }
}

// One wavefront's run of products over its workgroup's current group; SIDE 0:
// X (or the only group of wavefronts), 1: Y.  Both sides meet at the same
// barriers (see RGeo), so every wavefront of a workgroup makes the same calls.
template <class G, int SIDE, class OP>
struct Stepper {
  static constexpr bool X = SIDE == 0;
  static constexpr bool U = (X ? G::RX : G::RY) > 0;
  int lane, t0, tu, bu, par = 0;
  bool unit, first;
  bool pending = false;  // Y: the last product's reductions in base A (with def)
  OP def;
  Share<G, U> h;

  __device__ __forceinline__ Stepper(int wave, int lane_) : lane(lane_) {
    const int w = X ? wave : wave - G::W / 2;
    t0 = (X ? 0 : G::NX) + w * G::MT;
    unit = w < (X ? G::RX : G::RY) * G::NB;
    const int u = unit ? w : 0;
    tu = (X ? 0 : G::NX) + (G::XY ? G::W / 2 : G::W) * G::MT + (U ? u / G::NB : 0);
    bu = U ? u % G::NB : 0;
    first = (int)threadIdx.x < G::NB * 32;  // (X wavefronts) clears beta
  }

  // f(tile, column block, index in the share) over the wavefront's units
  template <class F>
  __device__ __forceinline__ void each(F f) const {
#pragma unroll 1
    for (int m = 0; m < G::MT; ++m)
#pragma unroll
      for (int b = 0; b < G::NB; ++b) f(t0 + m, b, false);
    if (U && unit) f(tu, bu, true);
  }

  // the running value <- w and x as load(tile, block, unit, x) gives them, with
  // xi for a product by mul(tile, block, unit, x)
  template <class L, class F>
  __device__ __forceinline__ void load(const RConst<G>& M, RWork<G>& ws, L value, F mul) {
    if constexpr (G::XY && !X) {
      if (pending) {
        finish_a(h, M, ws, par ^ 1, t0, unit, tu, bu, def, lane);
        pending = false;
      }
    }
    lds_barrier();  // beta is read, and the residues, before they are overwritten
    each([&](int t, int b, bool u) {
      const int at = (t * G::NB + b) * 64;
      v4u x;
      ws.om[at + lane] = value(t, b, u, x) ^ FLIP;
      const v4u y = mul(t, b, u, x);
      ChanConst<G> k;
      k.load(ws.ka, M.ka, t, lane);
      v4u o;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = pack16(reduce(mul16_biased<0>(x[i], y[i], BIAS), k.w[2 * i], k.w[8 + 2 * i]),
                      reduce(mul16_biased<1>(x[i], y[i], BIAS), k.w[2 * i + 1], k.w[9 + 2 * i]));
      ws.xi[at + lane] = o ^ FLIP;
    });
    for (int i = threadIdx.x; i < 2 * G::NB * 32; i += G::W * 64) (&ws.beta[0][0])[i] = 0;
    par = 0;
    if (X) h.prime(M.E1, t0, tu, lane);
    lds_barrier();
  }

  // One product: o names its multiplier and where its w goes, n the next
  // product's multiplier and where this product's x goes.  last: w only.
  __device__ __forceinline__ void product(const RConst<G>& M, RWork<G>& ws, OP& o, OP& n,
                                          bool last) {
    if constexpr (!G::XY || X) {
      o.pre_b(t0, unit, tu, lane);
      h.template init<false>(ws.c2, M.c2, t0, tu, lane);
      if constexpr (G::XY) {
        __builtin_amdgcn_s_setprio(1);
        h.template part<0, G::NX>(M.E1, ws.kb, M.kb, ws.xi, t0, tu, bu, lane);
        lds_barrier();
        __builtin_amdgcn_s_setprio(2);
      }
      h.template part<G::XY ? G::NX : 0, G::T>(M.E1, ws.kb, M.kb, ws.xi, t0, tu, bu, lane);
      if constexpr (G::XY) __builtin_amdgcn_s_setprio(0);
      finish_b(h, M, ws, par, t0, unit, tu, bu, o, lane);
      h.prime(M.E2, t0, tu, lane);
      lds_barrier();
      if (last) return;
      n.pre_a(t0, unit, tu, lane);
      h.template init<true>(ws.c2, M.c2, t0, tu, lane);
      if constexpr (G::XY) {
        __builtin_amdgcn_s_setprio(1);
        h.template part<0, G::NX>(M.E2, ws.ka, M.ka, ws.om, t0, tu, bu, lane);
        lds_barrier();
        __builtin_amdgcn_s_setprio(2);
      }
      h.template part<G::XY ? G::NX : 0, G::T>(M.E2, ws.ka, M.ka, ws.om, t0, tu, bu, lane);
      if constexpr (G::XY) __builtin_amdgcn_s_setprio(0);
      finish_a(h, M, ws, par, t0, unit, tu, bu, n, lane);
      par ^= 1;
      if (first) ws.beta[par][threadIdx.x] = 0;
      h.prime(M.E1, t0, tu, lane);
      lds_barrier();
    } else {
      if (pending) finish_a(h, M, ws, par ^ 1, t0, unit, tu, bu, def, lane);
      pending = false;
      h.prime(M.E1, t0, tu, lane);
      lds_barrier();
      o.pre_b(t0, unit, tu, lane);
      __builtin_amdgcn_s_setprio(1);
      h.template init<false>(ws.c2, M.c2, t0, tu, lane);
      h.template part<0, G::T>(M.E1, ws.kb, M.kb, ws.xi, t0, tu, bu, lane);
      __builtin_amdgcn_s_setprio(0);
      lds_barrier();
      finish_b(h, M, ws, par, t0, unit, tu, bu, o, lane);
      if (last) return;
      h.prime(M.E2, t0, tu, lane);
      lds_barrier();
      n.pre_a(t0, unit, tu, lane);
      __builtin_amdgcn_s_setprio(1);
      h.template init<true>(ws.c2, M.c2, t0, tu, lane);
      h.template part<0, G::T>(M.E2, ws.ka, M.ka, ws.om, t0, tu, bu, lane);
      __builtin_amdgcn_s_setprio(0);
      par ^= 1;
      pending = true;
      def = n;
      lds_barrier();
    }
  }

  // after the last product if its x is wanted
  __device__ __forceinline__ void flush(const RConst<G>& M, RWork<G>& ws) {
    if constexpr (G::XY && !X) {
      if (pending) finish_a(h, M, ws, par ^ 1, t0, unit, tu, bu, def, lane);
      pending = false;
    }
  }
};

// run R<SIDE>::go(...) of a workgroup's wavefronts
#define PC2R_SIDES(G, wave, CALL)   \
  do {                              \
    if constexpr (G::XY) {          \
      if ((wave) < G::W / 2) {      \
        constexpr int SIDE = 0;     \
        CALL;                       \
      } else {                      \
        constexpr int SIDE = 1;     \
        CALL;                       \
      }                             \
    } else {                        \
      constexpr int SIDE = 0;       \
      CALL;                         \
    }                               \
  } while (0)

}  // namespace pc2r
