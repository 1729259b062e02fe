// One element's Montgomery product (mfma_mont.hpp: the same digits, operand
// bands and bounds) on a workgroup of several wavefronts, for calls of few
// elements, where the time is that of a single chain of products.
//
// Each wavefront owns one column tile of 64 limbs: the low ones cover T's limbs
// below S and then q, the high ones the limbs from S up and then U.  A tile
// starts two limbs below the first one that it owns: the first gives the carry
// into the second, and the second the low neighbour that the reversed copies
// want, so no value crosses wavefronts inside a phase.  The
// constants' operand chunks stay in registers (N' in the low wavefronts, N in
// the high ones), x's forward digits are kept as four copies, one limb apart,
// so that every operand is one aligned 16-byte LDS read.
//
// What bounds a product are its three phases' latencies (LDS write, barrier,
// operand reads, the chain of matrix products, the fold).
#pragma once
#include "mfma_mont.hpp"

namespace pc2m {

template <int S>
struct TeamGeo : MGeo<S> {
  using M = MGeo<S>;
  static constexpr int NLOW = (S + 62) / 62;             // limbs 0 .. S, 62 to a tile
  static constexpr int NHIGH = (S + 63) / 62;            // S .. 2 S, 61 in the first tile
  static constexpr int W = NLOW + NHIGH;
  // forward copies: limb i of copy c at dword PFL / 4 + i + c
  static constexpr int PFL = 80;                         // zero bytes before limb 0 (c = 0)
  static constexpr int FC = ((PFL + M::D8 + 48 + 127) & ~127) + 32;
};

template <class G>
struct TeamWork {
  uint8_t xr[G::RBT], tr[G::RBT], qr[G::RBT];
  uint8_t xf[4 * G::FC];
  uint32_t u[G::S];
  uint32_t ok;
};

// A wavefront's tile: whether it is low, its first limb (lane 0) and column.
template <class G, int ROLE>
struct Tile {
  static constexpr bool LOW = ROLE < G::NLOW;
  static constexpr int K = LOW ? ROLE : ROLE - G::NLOW;
  static constexpr int BASE = LOW ? 62 * K - 2 : G::S - 3 + 62 * K;
  static constexpr int OWN = !LOW && K == 0 ? 3 : 2;     // first lane that is owned
  static constexpr int C0 = 4 * BASE;
  // operand chunk v = -t: digits C0 + 64 v + 4 j + 16 g ..
  static constexpr bool used(int v) { return C0 + 64 * v + 123 >= 0 && C0 + 64 * v < G::D; }
  static constexpr int VLO = [] { int v = -64; while (!used(v)) ++v; return v; }();
  static constexpr int VUP = [] { int v = VLO; while (used(v + 1)) ++v; return v; }();
  static constexpr int VHI = VUP < -G::TMIN ? VUP : -G::TMIN;
  static constexpr int VMIN = VLO > -G::TMAX ? VLO : -G::TMAX;
  static constexpr int NV = VHI - VMIN + 1;
  // the constant's chunks in registers (three wavefronts to a SIMD leave no room)
  static constexpr bool KEEP = G::W <= 8;
  static constexpr int NK = KEEP ? NV : 1;
};

// chunk offsets whose lanes may leave [lo, hi) read `zero` instead
__device__ __forceinline__ int in_range(int o, int base, int lo, int hi, int zero) {
  const int off = o + base;
  if (o >= lo && o + 108 < hi) return off;
  return off < lo || off >= hi ? zero : off;
}
// B chunk k of a forward digit array in global memory
template <class G, class P>
__device__ __forceinline__ v4i team_b_global(const uint8_t* y, int lane, int k) {
  const int off = in_range(P::C0 + 64 * (P::VMIN + k), 4 * (lane & 15) + 16 * (lane >> 4),
                           -G::PF, G::D8, -G::PF);
  const uint32_t* w = reinterpret_cast<const uint32_t*>(y + G::PF + off);
  return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
}
// ... chunk k of x's forward copies in LDS: the copy in which the lane's first
// limb is 16-byte aligned
template <class G, class P>
__device__ __forceinline__ v4i team_b_lds(const uint8_t* xf, int lane, int k) {
  const int base = 4 * (lane & 15) + 16 * (lane >> 4);
  const int c = (0 - (P::BASE + (lane & 15))) & 3;
  const uint8_t* at = xf + c * G::FC + 4 * c + G::PFL;
  // (out of range: the zeros of the front pad)
  const int off = in_range(P::C0 + 64 * (P::VMIN + k), base, -64, G::D8,
                           -64 + (base & 12) + ((4 * P::BASE) & 12));
  return *reinterpret_cast<const v4i*>(__builtin_assume_aligned(at + off, 16));
}

// Digit sums of the tile onto C; A operands from the reversed array xr, B
// operands from bf(chunk).  Two chains of accumulators: one alone waits for its
// own result at every step (34 cycles against 16).  The operands are read six
// chunks ahead: left to itself the compiler keeps two reads in flight (0.57 ms
// of 3.2 in a 2048-bit encryption).
template <class G, class P, class BF>
__device__ __forceinline__ void team_mma(v4i& C, const uint8_t* xr, int lane, BF bf) {
  constexpr int DEEP = 6, NG = (P::NV + DEEP - 1) / DEEP;
  const int i = lane & 15;
  const uint8_t* bp = xr + (3 - (i & 3)) * G::PR + G::X0 - 3 - 64 * (i >> 2) + 16 * (lane >> 4);
  v4i C2 = {0, 0, 0, 0};
  v4i A[2][DEEP], B[2][DEEP];
  auto load = [&](int g) {
#pragma unroll
    for (int u = 0; u < DEEP; ++u) {
      const int k = g * DEEP + u;
      if (k >= P::NV) break;
      A[g & 1][u] = *reinterpret_cast<const v4i*>(
          __builtin_assume_aligned(bp + 64 * (P::VMIN + k), 16));
      B[g & 1][u] = bf(k);
    }
  };
  load(0);
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (g + 1 < NG) load(g + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < DEEP; ++u) {
      const int k = g * DEEP + u;
      if (k >= P::NV) break;
      v4i& c = k & 1 ? C2 : C;
      c = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[g & 1][u], B[g & 1][u], c, 0, 0, 0);
    }
  }
  C += C2;
}

// One balanced split of the tile's biased column values (see split): the limb
// and the carry that it took.
__device__ __forceinline__ int32_t team_split(int64_t vb, int32_t& cin) {
  cin = (int32_t)rotate_up(
      __builtin_amdgcn_alignbit((uint32_t)((uint64_t)vb >> 32), (uint32_t)vb, 28));
  return (int32_t)((uint32_t)vb & M28) + cin - BIAS;
}

// The owned limbs as limbs of a reversed array (gi: the lane's limb in it);
// limb S takes part with a zero, as its lane writes the copies' dwords that
// reach into the limb below.  Returns the limb's digits.
template <class G, class P>
__device__ __forceinline__ uint32_t team_write_rev(uint8_t* xr, int32_t o, int lane, int gi) {
  const uint32_t d = gi < G::S ? limb_digits((uint32_t)o) : 0u;
  const uint32_t w = gi >= 0 ? __builtin_bswap32(d) : 0u;
  const uint32_t wp = rotate_up(w);
  if (lane >= P::OWN && gi <= G::S) put_rev<G>(xr, gi, w, wp);
  return d;
}

// x <- x y R^-1 by the wavefront of role ROLE (every wavefront of the workgroup
// calls it; x in ws.xr and ws.xf, y null: x itself).  kp: the
// wavefront's constant (N' or N), KB: its chunks.
// U: the result's limbs (high wavefronts).
template <class G, int ROLE>
__device__ __forceinline__ void team_mul(TeamWork<G>& ws, const v4i (&KB)[Tile<G, ROLE>::NK],
                                         const uint8_t* kp, const uint8_t* y, int lane, uint8_t* out,
                                         bool plus_one, int32_t& U) {
  using P = Tile<G, ROLE>;
  const FoldK k;
  v4i C = {0, 0, 0, 0};
  int32_t cin;
  auto constant = [&](int i) {
    if constexpr (P::KEEP)
      return KB[i];
    else
      return team_b_global<G, P>(kp, lane, i);
  };
  if (y) {
    team_mma<G, P>(C, ws.xr, lane, [&](int i) { return team_b_global<G, P>(y, lane, i); });
  } else {
    team_mma<G, P>(C, ws.xr, lane, [&](int i) { return team_b_lds<G, P>(ws.xf, lane, i); });
  }
  if constexpr (P::LOW) {
    const int32_t l = team_split(fold_biased(C, k.k7, k.k14, k.k21), cin);
    team_write_rev<G, P>(ws.tr, l, lane, P::BASE + lane);
  } else if constexpr (P::K == 0) {
    // the carry out of limb S - 1 joins column S; T mod R below it
    const int32_t l = team_split(fold_biased(C, k.k7, k.k14, k.k21), cin);
    if (lane == 3) C[0] += cin;
    if (lane < 3) C = v4i{l, 0, 0, 0};
  }
  __syncthreads();
  if constexpr (P::LOW) {
    v4i Q = {0, 0, 0, 0};
    team_mma<G, P>(Q, ws.tr, lane, constant);
    const int32_t l = team_split(fold_biased(Q, k.k7, k.k14, k.k21), cin);
    team_write_rev<G, P>(ws.qr, l, lane, P::BASE + lane);
  }
  __syncthreads();
  if constexpr (!P::LOW) {
    team_mma<G, P>(C, ws.qr, lane, constant);
    int64_t vb = fold_biased(C, k.k7, k.k14, k.k21);
    if constexpr (P::K == 0) {
      // c = (the part of T + q N below limb S) / R
      const int64_t a = (int64_t)read_lane64((uint64_t)vb, 2) - BIAS;
      const int64_t b = (int64_t)read_lane64((uint64_t)vb, 1) - BIAS;
      const int64_t c = (a + (b >> 28) + BIAS) >> 28;
      if (lane == 3) vb += c + (plus_one ? 1 : 0);
    }
    U = team_split(vb, cin);
    if constexpr (P::K == 0) {
      if (lane == 3) U -= cin;  // limb S takes no carry from below
    }
    const int gi = P::BASE - G::S + lane;
    const uint32_t d = team_write_rev<G, P>(ws.xr, U, lane, gi);
    if (lane >= P::OWN && gi < G::S) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        *reinterpret_cast<uint32_t*>(ws.xf + c * G::FC + G::PFL + 4 * (gi + c)) = d;
      if (out) *reinterpret_cast<uint32_t*>(out + G::PF + 4 * gi) = d;
    }
  }
  __syncthreads();
}

// limb i's digits d and the limb below's dp -> ws.xr and ws.xf
template <class G>
__device__ __forceinline__ void team_put(TeamWork<G>& ws, int i, uint32_t d, uint32_t dp) {
  put_rev<G>(ws.xr, i, __builtin_bswap32(d), __builtin_bswap32(dp));
  if (i < G::S)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      *reinterpret_cast<uint32_t*>(ws.xf + c * G::FC + G::PFL + 4 * (i + c)) = d;
}
template <class G>
__device__ __forceinline__ void team_load_x(TeamWork<G>& ws, const uint32_t* x, int n) {
  for (int i = threadIdx.x; i <= G::S; i += G::W * 64)
    team_put<G>(ws, i, i < G::S ? limb_digits(limb28_of(x, n, i)) : 0u,
                i > 0 ? limb_digits(limb28_of(x, n, i - 1)) : 0u);
  __syncthreads();
}
template <class G>
__device__ __forceinline__ void team_load_fwd(TeamWork<G>& ws, const uint8_t* y) {
  const uint32_t* d = reinterpret_cast<const uint32_t*>(y + G::PF);
  for (int i = threadIdx.x; i <= G::S; i += G::W * 64)
    team_put<G>(ws, i, i < G::S ? d[i] : 0u, i > 0 ? d[i - 1] : 0u);
  __syncthreads();
}

}  // namespace pc2m
