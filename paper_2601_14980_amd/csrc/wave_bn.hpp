// Multi-precision arithmetic with one wavefront per number: limb 64 r + lane
// (32 bits) in register r of the lane, zero from the number's length on.  For
// the few once-per-element steps after a powering, whose serial form in one
// lane (bn_scalar.hpp) waits for its own memory at every limb.
//
// Products go by columns: a's limbs are broadcast one after another through
// scalar registers while b moves up one lane, each lane adding its column's
// products in 96 bits.  Carries (and borrows) cross the lanes through the
// scalar unit: a lane that overflows and the lanes that pass a carry on are two
// 64-bit masks, and one addition of them gives every lane's carry.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pc2w {

// lane's value from the lane below; lane 0 of register r from lane 63 of r - 1
template <int N>
__device__ __forceinline__ void up1(uint32_t (&x)[N]) {
#pragma unroll
  for (int r = N - 1; r >= 0; --r) {
    const int in = r ? __builtin_amdgcn_readlane((int)x[r - 1], 63) : 0;
    x[r] = (uint32_t)__builtin_amdgcn_update_dpp(in, (int)x[r], 0x138 /* wave_shr:1 */, 0xF, 0xF,
                                                 false);
  }
}

// carries into the lanes: g lanes that overflow, p lanes that pass one on (no
// lane both); carry: into lane 0, then out of lane 63
__device__ __forceinline__ uint64_t lookahead(uint64_t g, uint64_t p, uint32_t& carry) {
  const uint64_t x = (g << 1) | carry, s = x + p;
  carry = (uint32_t)(g >> 63) | (s < x ? 1u : 0u);
  return s ^ p;
}

// r <- a + b (carry out of register N - 1 dropped)
template <int N>
__device__ __forceinline__ void add(uint32_t (&r)[N], const uint32_t (&a)[N],
                                    const uint32_t (&b)[N], int lane) {
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t t = a[i] + b[i];
    const uint64_t in = lookahead(__ballot(t < b[i]), __ballot(t == 0xFFFFFFFFu), c);
    r[i] = t + ((uint32_t)(in >> lane) & 1u);
  }
}
// r <- a - b; returns the borrow out of register N - 1
template <int N>
__device__ __forceinline__ uint32_t sub(uint32_t (&r)[N], const uint32_t (&a)[N],
                                        const uint32_t (&b)[N], int lane) {
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t t = a[i] - b[i];
    const uint64_t in = lookahead(__ballot(a[i] < b[i]), __ballot(t == 0u), c);
    r[i] = t - ((uint32_t)(in >> lane) & 1u);
  }
  return c;
}

// r <- a b mod 2^(32 64 NC), na limbs of a
template <int NC, int NA, int NB>
__device__ __forceinline__ void mul(uint32_t (&r)[NC], const uint32_t (&a)[NA], int na,
                                    const uint32_t (&b)[NB], int lane) {
  uint32_t bs[NC], hi[NC], mid[NC];
  uint64_t s[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    bs[i] = i < NB ? b[i] : 0u;
    s[i] = 0;
    hi[i] = 0;
  }
#pragma unroll
  for (int w = 0; w < NA; ++w) {
    const int n = na - 64 * w < 64 ? na - 64 * w : 64;
    for (int k = 0; k < n; ++k) {
      const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)a[w], k);
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const uint64_t p = (uint64_t)x * bs[i];
        s[i] += p;
        hi[i] += s[i] < p ? 1u : 0u;
      }
      up1<NC>(bs);
    }
  }
  // columns -> limbs
  uint32_t h1[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    mid[i] = (uint32_t)(s[i] >> 32);
    h1[i] = hi[i];
  }
  up1<NC>(mid);
  up1<NC>(h1);
  up1<NC>(h1);
  uint32_t over[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const uint64_t v = (uint64_t)(uint32_t)s[i] + mid[i] + h1[i];
    r[i] = (uint32_t)v;
    over[i] = (uint32_t)(v >> 32);
  }
  up1<NC>(over);
  uint32_t tmp[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) tmp[i] = r[i];
  add<NC>(r, tmp, over, lane);
}

// n limbs from memory
template <int N>
__device__ __forceinline__ void load(uint32_t (&r)[N], const uint32_t* x, int n, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i) r[i] = 64 * i + lane < n ? x[64 * i + lane] : 0u;
}
// limbs n .. zeroed
template <int N>
__device__ __forceinline__ void clip(uint32_t (&r)[N], int n, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (64 * i + lane >= n) r[i] = 0u;
}
// limbs n .. 2 n - 1 of x as limbs 0 .. n - 1
template <int N, int NC>
__device__ __forceinline__ void high(uint32_t (&r)[N], const uint32_t (&x)[NC], int n, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    r[i] = 0u;
#pragma unroll
    for (int k = 0; k < NC; ++k) {  // limb 64 i + lane + n: register k of lane (lane + n) & 63
      const uint32_t v = (uint32_t)__builtin_amdgcn_ds_bpermute(((lane + n) & 63) * 4, (int)x[k]);
      if ((64 * i + lane + n) >> 6 == k) r[i] = v;
    }
  }
  clip<N>(r, n, lane);
}

// r <- a b 2^(-32 n) mod m for a, b < m of n limbs; minv = m^-1 mod 2^(32 n)
template <int N, int NC>
__device__ __forceinline__ void mont(uint32_t (&r)[N], const uint32_t (&a)[N],
                                     const uint32_t (&b)[N], const uint32_t (&m)[N],
                                     const uint32_t (&minv)[N], int n, int lane) {
  uint32_t t[NC], q[N], lo[N], qm[NC], hi[N], qh[N];
  mul<NC>(t, a, n, b, lane);
#pragma unroll
  for (int i = 0; i < N; ++i) lo[i] = t[i];
  clip<N>(lo, n, lane);
  mul<N>(q, lo, n, minv, lane);
  clip<N>(q, n, lane);
  mul<NC>(qm, q, n, m, lane);
  // T - q m has zeros below limb n, and its upper part lies in (-m, m)
  high<N, NC>(hi, t, n, lane);
  high<N, NC>(qh, qm, n, lane);
  if (sub<N>(r, hi, qh, lane)) {
    uint32_t d[N];
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = r[i];
    add<N>(r, d, m, lane);
    clip<N>(r, n, lane);  // (the borrow ran through the zeros above)
  }
}

// a < b, n limbs in memory (uniform)
__device__ __forceinline__ bool less(const uint32_t* a, const uint32_t* b, int n, int lane) {
  for (int at = (n - 1) & ~63; at >= 0; at -= 64) {
    const uint32_t x = at + lane < n ? a[at + lane] : 0u, y = at + lane < n ? b[at + lane] : 0u;
    const uint64_t ne = __ballot(x != y);
    if (ne) {
      const uint64_t lt = __ballot(x < y);
      return (lt >> (63 - __builtin_clzll(ne))) & 1;
    }
  }
  return false;
}

}  // namespace pc2w
