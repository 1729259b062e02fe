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
// the low one with its top bit flipped (r = 256 h + l + 128; the 128 sum_i
// E[j][i] this adds sits in the initial accumulators).  Both bytes of a
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
typedef short v2s __attribute__((ext_vector_type(2)));

// T tiles, NB column blocks, W wavefronts.  Of the T x NB (tile, column
// block) units, P pairs of tiles and Q single tiles are taken over all column
// blocks at once (wavefront p % W), the units of the remaining tiles one by
// one (wavefront (u + UO) % W; the single tile q goes to wavefront (P + q) %
// W): chosen so that the four SIMDs get the same
// number of units.
template <int T_, int NB_, int W_, int P_, int Q_, int UO_>
struct RGeo {
  static constexpr int T = T_, NB = NB_, W = W_, P = P_, Q = Q_, UO = UO_;
  static constexpr int NU = (T_ - 2 * P_ - Q_) * NB_;  // single units
  static constexpr int PART = T_ * NB_ * 64;           // 16-byte slots of one base
  static_assert(2 * P_ + Q_ <= T_, "tiles");
};

template <class G>
struct RWork {
  v4u xi[G::PART];                          // xi (base A), low bytes flipped
  v4u om[G::PART];                          // w (base B), low bytes flipped
  unsigned long long beta[2][G::NB * 32];   // sum_j w_j g_j / b_j in 2^-25
};

constexpr uint32_t FLIP = 0x00800080u;

__device__ __forceinline__ uint32_t pack16(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
__device__ __forceinline__ int dot2(uint32_t a, uint32_t b, int c) {
  return __builtin_amdgcn_sdot2(__builtin_bit_cast(v2s, a), __builtin_bit_cast(v2s, b), c, false);
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
  __device__ __forceinline__ Buf(const void* p, uint32_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000)) {}
  __device__ __forceinline__ v4u load(uint32_t lane_off, uint32_t off) const {
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)off, 0);
  }
  __device__ __forceinline__ void store(v4u v, uint32_t lane_off, uint32_t off) const {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)lane_off, (int)off, 0);
  }
};

// The constants of a modulus.
template <class G>
struct RConst {
  Buf E1, E2, c1, c2, kb, ka;
  __device__ __forceinline__ explicit RConst(const pc2k::RnsMod& M)
      : E1(M.E1, G::T * G::T * 1024), E2(M.E2, G::T * G::T * 1024), c1(M.c1, G::T * 128),
        c2(M.c2, G::T * 128), kb(M.kb, G::T * 192), ka(M.ka, G::T * 192) {}
};

// acc[m][b] = tile t0 + m of the matrix E times column block nb0 + b of src
template <class G, int MT, int NBN>
__device__ __forceinline__ void gemm(v16i (&acc)[MT][NBN], const Buf& E, const Buf& cst,
                                     const v4u* src, int t0, int nb0, int lane) {
  constexpr int T = G::T, PD = 3;
  const v4i* s = reinterpret_cast<const v4i*>(src) + nb0 * 64 + lane;
  const uint32_t lo = lane * 16;
  v4i a[PD][MT];
#pragma unroll
  for (int c = 0; c < PD; ++c)
#pragma unroll
    for (int m = 0; m < MT; ++m)
      a[c][m] = __builtin_bit_cast(v4i, E.load(lo, ((t0 + m) * T + c) * 1024));
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    v16i c0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const v4u v = cst.load((lane >> 5) * 64, (t0 + m) * 128 + 16 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) c0[4 * i + j] = (int)v[j];
    }
#pragma unroll
    for (int b = 0; b < NBN; ++b) acc[m][b] = c0;
  }
#pragma unroll
  for (int c = 0; c < T; ++c) {
    v4i y[NBN];
#pragma unroll
    for (int b = 0; b < NBN; ++b) y[b] = s[(c * G::NB + b) * 64];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int b = 0; b < NBN; ++b)
        acc[m][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[c % PD][m], y[b], acc[m][b], 0, 0, 0);
    if (c + PD < T) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
        a[c % PD][m] = __builtin_bit_cast(v4i, E.load(lo, ((t0 + m) * T + c + PD) * 1024));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Channel constants of one tile half: three groups of eight words.
struct ChanConst {
  uint32_t w[24];
  __device__ __forceinline__ ChanConst(const Buf& k, int t, int lane) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const v4u v = k.load((lane >> 5) * 96, t * 192 + 16 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[4 * i + j] = v[j];
    }
  }
};

// A -> B: tiles t0 .. t0 + MT - 1 of w <- w y + E1 xi, for NBN column blocks.
// y: the multiplier (mul; else w itself); dst: where a copy of the result
// goes (store); the tiles' share of beta is added to ws.beta[par].
template <class G, int MT, int NBN>
__device__ __forceinline__ void ext1(const RConst<G>& M, RWork<G>& ws, int par, int t0, int nb0,
                                     bool mul, const Buf& y, bool store, const Buf& dst,
                                     int lane) {
  v16i acc[MT][NBN];
  gemm<G, MT, NBN>(acc, M.E1, M.c1, ws.xi, t0, nb0, lane);
  int s1[NBN], s2[NBN];
#pragma unroll
  for (int b = 0; b < NBN; ++b) s1[b] = s2[b] = 0;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const ChanConst k(M.kb, t0 + m, lane);
    const int at = ((t0 + m) * G::NB + nb0) * 64;
    v4u x[NBN], f[NBN];
#pragma unroll
    for (int b = 0; b < NBN; ++b) x[b] = f[b] = ws.om[at + b * 64 + lane] ^ FLIP;
    if (mul) {
#pragma unroll
      for (int b = 0; b < NBN; ++b) f[b] = y.load(lane * 16, (at + b * 64) * 16);
    }
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
      v4u o;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t r[2];
        r[0] = reduce(mad16<0>(x[b][i], f[b][i], (acc[m][b][4 * i + 1] << 8) + acc[m][b][4 * i]),
                      k.w[2 * i], k.w[8 + 2 * i]);
        r[1] = reduce(
            mad16<1>(x[b][i], f[b][i], (acc[m][b][4 * i + 3] << 8) + acc[m][b][4 * i + 2]),
            k.w[2 * i + 1], k.w[8 + 2 * i + 1]);
        o[i] = pack16(r[0], r[1]);
        s1[b] = dot2(o[i], k.w[16 + i], s1[b]);
        s2[b] = dot2(o[i], k.w[20 + i], s2[b]);
      }
      if (store) dst.store(o, lane * 16, (at + b * 64) * 16);
      ws.om[at + b * 64 + lane] = o ^ FLIP;
    }
  }
#pragma unroll
  for (int b = 0; b < NBN; ++b) {
    const long long s = (long long)s1[b] * 8192 + s2[b];
    __hip_atomic_fetch_add(&ws.beta[par][(nb0 + b) * 32 + (lane & 31)], (unsigned long long)s,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// B -> A: tiles of x <- E2 w - beta MB, then xi <- x y for the next product
// (y: its multiplier if mul, else x itself); a copy of x goes to dst (store).
template <class G, int MT, int NBN>
__device__ __forceinline__ void ext2(const RConst<G>& M, RWork<G>& ws, int par, int t0, int nb0,
                                     bool mul, const Buf& y, bool store, const Buf& dst,
                                     int lane) {
  v16i acc[MT][NBN];
  gemm<G, MT, NBN>(acc, M.E2, M.c2, ws.om, t0, nb0, lane);
  uint32_t bp[NBN];
#pragma unroll
  for (int b = 0; b < NBN; ++b) {
    const long long s = (long long)ws.beta[par][(nb0 + b) * 32 + (lane & 31)];
    const int beta = (int)((s + (1 << 24)) >> 25);
    const int lo = (int)((uint32_t)beta << 20) >> 20;
    bp[b] = pack16((uint32_t)lo, (uint32_t)((beta - lo) >> 12));
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const ChanConst k(M.ka, t0 + m, lane);
    const int at = ((t0 + m) * G::NB + nb0) * 64;
    v4u x[NBN], f[NBN];
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t r[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
          r[j] = reduce(dot2(bp[b], k.w[16 + 2 * i + j],
                             (acc[m][b][4 * i + 2 * j + 1] << 8) + acc[m][b][4 * i + 2 * j]),
                        k.w[2 * i + j], k.w[8 + 2 * i + j]);
        x[b][i] = pack16(r[0], r[1]);
      }
      f[b] = x[b];
    }
    if (store) {
#pragma unroll
      for (int b = 0; b < NBN; ++b) dst.store(x[b], lane * 16, (G::PART + at + b * 64) * 16);
    }
    if (mul) {
#pragma unroll
      for (int b = 0; b < NBN; ++b) f[b] = y.load(lane * 16, (G::PART + at + b * 64) * 16);
    }
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
      v4u o;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = pack16(
            reduce(mad16<0>(x[b][i], f[b][i], 0), k.w[2 * i], k.w[8 + 2 * i]),
            reduce(mad16<1>(x[b][i], f[b][i], 0), k.w[2 * i + 1], k.w[9 + 2 * i]));
      ws.xi[at + b * 64 + lane] = o ^ FLIP;
    }
  }
}

// Load a value: w, and xi for the next product (as in ext2).
template <class G>
__device__ __forceinline__ void load_unit(const RConst<G>& M, RWork<G>& ws, int t, int b,
                                          const Buf& e, bool mul, const Buf& yb, int lane) {
  const int at = (t * G::NB + b) * 64;
  ws.om[at + lane] = e.load(lane * 16, at * 16) ^ FLIP;
  const v4u x = e.load(lane * 16, (G::PART + at) * 16);
  v4u y = x;
  if (mul) y = yb.load(lane * 16, (G::PART + at) * 16);
  const ChanConst k(M.ka, t, lane);
  v4u o;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    o[i] = pack16(reduce(mad16<0>(x[i], y[i], 0), k.w[2 * i], k.w[8 + 2 * i]),
                  reduce(mad16<1>(x[i], y[i], 0), k.w[2 * i + 1], k.w[9 + 2 * i]));
  ws.xi[at + lane] = o ^ FLIP;
}

// run F<MT, NBN>(t0, nb0) over the wavefront's share of the units
#define PC2R_FOR_ITEMS(G, wave, CALL)                                        \
  do {                                                                       \
    for (int u_ = (wave); u_ < G::P; u_ += G::W) {                           \
      constexpr int MT = 2, NBN = G::NB;                                     \
      const int t0 = 2 * u_, nb0 = 0;                                        \
      CALL;                                                                  \
    }                                                                        \
    for (int u_ = ((wave) + G::W - G::P % G::W) % G::W; u_ < G::Q; u_ += G::W) { \
      constexpr int MT = 1, NBN = G::NB;                                     \
      const int t0 = 2 * G::P + u_, nb0 = 0;                                 \
      CALL;                                                                  \
    }                                                                        \
    for (int u_ = ((wave) + G::W - G::UO % G::W) % G::W; u_ < G::NU; u_ += G::W) { \
      constexpr int MT = 1, NBN = 1;                                         \
      const int t0 = 2 * G::P + G::Q + u_ / G::NB, nb0 = u_ % G::NB;         \
      CALL;                                                                  \
    }                                                                        \
  } while (0)

}  // namespace pc2r
