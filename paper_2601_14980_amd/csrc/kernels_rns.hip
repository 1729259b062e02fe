// Powering kernels of the RNS engine (rns_mont.hpp) and its conversions.
//
//   k_rns_to    integers (32-bit limbs) -> residues of both bases, in
//               Montgomery form (times MA) or times another constant
//   k_rns_pow   runs a program of Montgomery products over groups of 32 NB
//               elements, one group at a time per workgroup: the table of
//               odd powers, sliding windows, the closing product
//   k_rns_from  residues of base B -> the canonical integer mod N
//
// Both conversions are plain sums over constants on the vector ALUs (together
// a few products' worth of a powering of thousands).
#include <hip/hip_runtime.h>

#include "bn_scalar.hpp"
#include "paillier_ops.hpp"
#include "rns_launch.hpp"
#include "rns_mont.hpp"

using namespace pc2r;
using pc2k::RnsFrom;
using pc2k::RnsPow;
using pc2k::RnsTo;

namespace {

// One wavefront's run over its workgroup's groups; SIDE 0: X (or the only
// group of wavefronts), 1: Y.  Both sides meet at the same barriers; see RGeo.
template <class G, int SIDE>
__device__ __forceinline__ void pow_run(const RnsPow& P, RWork<G>& ws, int wave, int lane) {
  constexpr bool X = SIDE == 0;
  constexpr bool U = (X ? G::RX : G::RY) > 0;
  constexpr size_t GB = 2 * (size_t)G::PART * 16;  // bytes of one group's residues
  const int w = X ? wave : wave - G::W / 2;
  const int t0 = (X ? 0 : G::NX) + w * G::MT;
  const bool unit = w < (X ? G::RX : G::RY) * G::NB;
  const int u = unit ? w : 0;
  const int tu = (X ? 0 : G::NX) + (G::XY ? G::W / 2 : G::W) * G::MT + (U ? u / G::NB : 0);
  const int bu = U ? u % G::NB : 0;
  const bool first = (int)threadIdx.x < G::NB * 32;  // (X wavefronts) clears beta
  uint8_t* slot = P.table + (size_t)blockIdx.x * P.entries * GB;
  const int nitems = P.ngroups * P.nmod;
  Share<G, U> h;
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const int mod = P.nmod == 2 ? (it & 1) : 0;
    const int g = P.nmod == 2 ? it >> 1 : it;
    const RConst<G> M(P.M[mod]);
    const uint32_t* ops = P.ops[mod];
    uint8_t* in = P.in[mod] + (size_t)g * GB;
    uint8_t* gm = P.gm[mod] ? P.gm[mod] + (size_t)g * GB : in;
    auto entry = [&](uint32_t e) {
      uint8_t* p = slot + (size_t)(e - 1) * GB;
      if (e == pc2k::RNS_GM) p = gm;
      if (e == 0 || e >= pc2k::RNS_OUT) p = in;
      return Buf(p, (uint32_t)GB);
    };
    auto is_mul = [](uint32_t op) { return op >> 16 == pc2k::RNS_MUL && (op & 0xFF) != pc2k::RNS_SQ; };
    auto stores = [](uint32_t op) { return ((op >> 8) & 0xFF) != pc2k::RNS_NODST; };
    // operands of the reductions of product `op` in base B, and in base A,
    // where the multiplier is the next product's
    auto ops_b = [&](uint32_t op) {
      return Operands{is_mul(op), stores(op), entry(op & 0xFF), entry((op >> 8) & 0xFF)};
    };
    auto ops_a = [&](uint32_t op, uint32_t next) {
      return Operands{is_mul(next), stores(op), entry(next & 0xFF), entry((op >> 8) & 0xFF)};
    };
    int par = 0;
    int k = 0;
    uint32_t op = ops[0], prev = 0;
    for (;;) {
      // op is a load: every wavefront its own tiles
      {
        const uint32_t next = ops[k + 1];
        const Buf e = entry(op & 0xFF), y = entry(next & 0xFF);
        for (int m = 0; m < G::MT; ++m)
          for (int b = 0; b < G::NB; ++b)
            load_unit<G>(M, ws, t0 + m, b, e, is_mul(next), y, lane);
        if (U && unit) load_unit<G>(M, ws, tu, bu, e, is_mul(next), y, lane);
        for (int i = threadIdx.x; i < 2 * G::NB * 32; i += G::W * 64) (&ws.beta[0][0])[i] = 0;
        op = next;
        ++k;
        if (X) h.prime(M.E1, t0, tu, lane);
        lds_barrier();
      }
      bool pending = false;  // Y: the last product's reductions in base A
      for (;;) {
        // products: A -> B
        const uint32_t next = ops[++k];
        if constexpr (!G::XY) {
          h.template init<false>(ws.c2, M.c2, t0, tu, lane);
          h.template part<0, G::T>(M.E1, ws.kb, M.kb, ws.xi, t0, tu, bu, lane);
          finish_b(h, M, ws, par, t0, unit, tu, bu, ops_b(op), lane);
          h.prime(M.E2, t0, tu, lane);
          lds_barrier();
          if (next >> 16 == pc2k::RNS_END) break;
          h.template init<true>(ws.c2, M.c2, t0, tu, lane);
          h.template part<0, G::T>(M.E2, ws.ka, M.ka, ws.om, t0, tu, bu, lane);
          finish_a(h, M, ws, par, t0, unit, tu, bu, ops_a(op, next), lane);
          par ^= 1;
          if (first) ws.beta[par][threadIdx.x] = 0;
          h.prime(M.E1, t0, tu, lane);
          lds_barrier();
        } else if constexpr (X) {
          __builtin_amdgcn_s_setprio(1);
          h.template init<false>(ws.c2, M.c2, t0, tu, lane);
          h.template part<0, G::NX>(M.E1, ws.kb, M.kb, ws.xi, t0, tu, bu, lane);
          lds_barrier();
          __builtin_amdgcn_s_setprio(2);
          h.template part<G::NX, G::T>(M.E1, ws.kb, M.kb, ws.xi, t0, tu, bu, lane);
          __builtin_amdgcn_s_setprio(0);
          finish_b(h, M, ws, par, t0, unit, tu, bu, ops_b(op), lane);
          h.prime(M.E2, t0, tu, lane);
          lds_barrier();
          if (next >> 16 == pc2k::RNS_END) break;
          __builtin_amdgcn_s_setprio(1);
          h.template init<true>(ws.c2, M.c2, t0, tu, lane);
          h.template part<0, G::NX>(M.E2, ws.ka, M.ka, ws.om, t0, tu, bu, lane);
          lds_barrier();
          __builtin_amdgcn_s_setprio(2);
          h.template part<G::NX, G::T>(M.E2, ws.ka, M.ka, ws.om, t0, tu, bu, lane);
          __builtin_amdgcn_s_setprio(0);
          finish_a(h, M, ws, par, t0, unit, tu, bu, ops_a(op, next), lane);
          par ^= 1;
          if (first) ws.beta[par][threadIdx.x] = 0;
          h.prime(M.E1, t0, tu, lane);
          lds_barrier();
        } else {
          if (pending) finish_a(h, M, ws, par ^ 1, t0, unit, tu, bu, ops_a(prev, op), lane);
          h.prime(M.E1, t0, tu, lane);
          lds_barrier();
          __builtin_amdgcn_s_setprio(1);
          h.template init<false>(ws.c2, M.c2, t0, tu, lane);
          h.template part<0, G::T>(M.E1, ws.kb, M.kb, ws.xi, t0, tu, bu, lane);
          __builtin_amdgcn_s_setprio(0);
          lds_barrier();
          finish_b(h, M, ws, par, t0, unit, tu, bu, ops_b(op), lane);
          if (next >> 16 == pc2k::RNS_END) break;
          h.prime(M.E2, t0, tu, lane);
          lds_barrier();
          __builtin_amdgcn_s_setprio(1);
          h.template init<true>(ws.c2, M.c2, t0, tu, lane);
          h.template part<0, G::T>(M.E2, ws.ka, M.ka, ws.om, t0, tu, bu, lane);
          __builtin_amdgcn_s_setprio(0);
          par ^= 1;
          pending = true;
          lds_barrier();
        }
        prev = op;
        op = next;
        if (op >> 16 != pc2k::RNS_MUL) break;
      }
      if (ops[k] >> 16 == pc2k::RNS_END) break;
      if constexpr (G::XY) {
        if (!X) finish_a(h, M, ws, par ^ 1, t0, unit, tu, bu, ops_a(prev, op), lane);
        lds_barrier();  // beta is read before the load clears it
      }
    }
    lds_barrier();  // the next group's load overwrites the residues
  }
}

template <class G>
__global__ __launch_bounds__(G::W * 64, 2) void k_rns_pow(RnsPow P) {
  __shared__ __align__(16) RWork<G> ws;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_constants<G>(P.M[0], ws);
  lds_barrier();
  if constexpr (G::XY) {
    if (wave < G::W / 2)
      pow_run<G, 0>(P, ws, wave, lane);
    else
      pow_run<G, 1>(P, ws, wave, lane);
  } else {
    pow_run<G, 0>(P, ws, wave, lane);
  }
}

// Residues of one wavefront's slot (part, tile, half: eight channels) for 64
// elements, one per lane: sum_i half_i P[i] + add.  The constants are uniform
// (scalar loads); elements past `count` repeat the last one, so that every
// column of a group holds valid residues.
__global__ __launch_bounds__(256) void k_rns_to(RnsTo C, const uint32_t* __restrict__ x,
                                                int limbs, size_t count, int T, int nb,
                                                uint8_t* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int slot = __builtin_amdgcn_readfirstlane(blockIdx.y * 4 + (threadIdx.x >> 6));
  if (slot >= 4 * T) return;
  const size_t pos = (size_t)blockIdx.x * 64 + lane;  // position in the padded groups
  const size_t per = (size_t)nb * 32;
  const size_t total = (count + per - 1) / per * per;
  if (pos >= total) return;
  const size_t e = pos < count ? pos : count - 1;
  const int nhalf = 2 * limbs < C.nhalf ? 2 * limbs : C.nhalf;
  const uint32_t* P = C.P + (size_t)slot * C.nhalf * 8;
  const uint32_t* xe = x + e * limbs;
  uint64_t acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = C.add[slot * 8 + c];
  for (int i = 0; i < nhalf; i += 2) {
    const uint32_t w = xe[i >> 1];
    const uint32_t lo = w & 0xFFFFu, hi = w >> 16;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] += (uint64_t)lo * P[i * 8 + c];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] += (uint64_t)hi * P[i * 8 + 8 + c];
  }
  v4u o;
  uint32_t r[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    // acc < 2^42: the quotient by the modulus is exact to +-1 in double
    const uint32_t m = C.m[slot * 8 + c];
    const uint64_t q = (uint64_t)((double)acc[c] * (1.0 / (double)m));
    int v = (int)(uint32_t)(acc[c] - q * m);  // in [-m, 2 m)
    if (v < 0) v += (int)m;
    if (v >= (int)m) v -= (int)m;
    if (2 * v > (int)m) v -= (int)m;
    r[c] = (uint32_t)v;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = pack16(r[2 * i], r[2 * i + 1]);
  // slot = (part T + tile) 2 + half
  const int h = slot & 1, pt = slot >> 1;
  const size_t grp = pos / per, b = pos % per / 32, n = pos & 31;
  uint8_t* g = out + grp * pc2k::rns_group_bytes(T, nb);
  reinterpret_cast<v4u*>(g)[((size_t)pt * nb + b) * 64 + h * 32 + n] = o;
}

// The value of base-B residues mod N, canonical.  A block handles 64
// elements, one per lane of every wavefront: the wavefronts form the columns
// sum_j w_j C_j[l] + beta D[l] + O[l] of eight limbs each (constants by
// scalar loads) and resolve the carries inside their block of limbs; the
// first wavefront then joins the blocks, subtracts the quotient by N, and
// all write the words.
__global__ __launch_bounds__(512) void k_rns_from(RnsFrom C, const uint8_t* __restrict__ in,
                                                  size_t count, int T, int nb,
                                                  uint32_t* __restrict__ out, size_t stride) {
  extern __shared__ __align__(16) uint32_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = C.nblk;
  uint32_t* limb = lds;                                              // [8 nblk][64]
  int64_t* cy = reinterpret_cast<int64_t*>(lds + (size_t)nblk * 512);  // [nblk][64]
  const size_t pos0 = (size_t)blockIdx.x * 64 + lane;
  const size_t pos = pos0 < count ? pos0 : count - 1;
  const size_t per = (size_t)nb * 32;
  const size_t grp = pos / per, b = pos % per / 32, n = pos & 31;
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
    const size_t p = (size_t)blockIdx.x * 64 + e;
    if (p >= count) break;
    for (int j = lane; j < C.nw; j += 64) {
      const int bit = 32 * j, i = bit / 28, sh = bit % 28;
      uint64_t v = limb[i * 64 + e];
      if (i + 1 < 8 * nblk) v |= (uint64_t)limb[(i + 1) * 64 + e] << 28;
      if (i + 2 < 8 * nblk) v |= (uint64_t)limb[(i + 2) * 64 + e] << 56;
      out[p * stride + j] = (uint32_t)(v >> sh);
    }
  }
}

// Input checks of an encryption, one lane per element: with c the element's
// ciphertext is zeroed if m >= n, r = 0 or r >= n, and ERR_RANGE latched;
// with okw the result of the check goes there instead (both halves' words).
__global__ __launch_bounds__(64) void k_rns_enc_check(pc2k::PkConst pk,
                                                      const uint32_t* __restrict__ m, int m_limbs,
                                                      const uint32_t* __restrict__ r,
                                                      uint32_t* __restrict__ c, size_t count,
                                                      uint32_t* __restrict__ okw, size_t stride,
                                                      int* err) {
  const size_t e = (size_t)blockIdx.x * 64 + threadIdx.x;
  if (e >= count) return;
  const int L = pk.L;
  const uint32_t* re = r + e * L;
  bool ok = pc2d::sc_cmp(m + e * m_limbs, m_limbs, pk.n, L) < 0 && pc2d::sc_cmp(re, L, pk.n, L) < 0;
  int i = L - 1;
  while (i >= 0 && re[i] == 0) --i;
  ok = ok && i >= 0;
  if (okw) {
    okw[2 * e * stride] = ok;
    okw[(2 * e + 1) * stride] = ok;
  } else if (!ok) {
    for (int j = 0; j < 2 * L; ++j) c[e * 2 * L + j] = 0u;
    atomicOr(err, pc2k::ERR_RANGE);
  }
}

// The scalar end of a decryption half, one lane per (element, prime): y =
// c^(s-1) mod s^2 (canonical, nl words at y + (2 e + half) stride) -> m_s =
// L_s(y) h_s mod s and its validity word at halves + (2 e + half)(Ls + 1).
__global__ __launch_bounds__(64) void k_rns_dec_finish(pc2k::SkConst sk,
                                                       const uint32_t* __restrict__ c,
                                                       const uint32_t* __restrict__ ys,
                                                       size_t stride, size_t count,
                                                       uint32_t* __restrict__ halves) {
  const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x;
  const int half = blockIdx.y;
  if (i >= count) return;
  const pc2k::HalfConst& H = sk.h[half];
  const int Ls = H.Ls, nl = H.s2.nl, L2 = 2 * sk.pk.L;
  const bool cv = pc2d::sc_cmp(c + i * L2, L2, sk.pk.n2.Nl, L2) < 0;
  uint32_t y[2 * pc2k::LS_MAX + 1], u[pc2k::LS_MAX], us[2 * pc2k::LS_MAX],
      tmp[pc2k::LS_MAX + 2];
  const uint32_t* src = ys + (2 * i + half) * stride;
  for (int j = 0; j < nl; ++j) y[j] = src[j];
  const uint32_t one = 1u;
  const uint32_t bor = pc2d::sc_sub(y, nl, &one, 1);
  pc2d::sc_mullo(u, y, H.sinv, Ls);
  pc2d::sc_mul(us, u, Ls, H.s, Ls);
  const bool good = bor == 0 && pc2d::sc_cmp(us, 2 * Ls, y, nl) == 0 && cv;
  uint32_t* dst = halves + (2 * i + half) * (size_t)(Ls + 1);
  pc2d::sc_montmul(u, u, H.H, H.s, H.s_n0, Ls, tmp);
  for (int j = 0; j < Ls; ++j) dst[j] = u[j];
  dst[Ls] = good ? 1u : 0u;
}

}  // namespace

namespace pc2k {

namespace {
// (T, NB) -> geometry: wavefronts, and whether they run as two sides.
template <int T, int NB>
struct Pick;
#define PC2_RNS_GEOS(D)                                                       \
  D(5, 1, 4, false) D(5, 2, 4, false) D(5, 4, 4, false)                       \
  D(9, 1, 8, false) D(9, 2, 4, false) D(9, 4, 4, false)                       \
  D(13, 1, 8, false) D(13, 2, 4, false) D(13, 3, 4, false)                    \
  D(17, 1, 8, true) D(17, 2, 8, true) D(17, 4, 8, true)                       \
  D(26, 1, 8, true) D(26, 2, 8, true) D(26, 3, 8, true)                       \
  D(34, 1, 8, true) D(34, 2, 8, true)
#define PC2_RNS_PICK(T, NB, W, XY) \
  template <>                      \
  struct Pick<T, NB> {             \
    using G = RGeo<T, NB, W, XY>;  \
  };
PC2_RNS_GEOS(PC2_RNS_PICK)
#undef PC2_RNS_PICK
}  // namespace

#define PC2_RNS_CASE(T, NB, W, XY) \
  if (t == T && nb == NB) {        \
    using G = Pick<T, NB>::G;      \
    PC2_RNS_DO;                    \
  }

const void* rns_pow_kernel(int t, int nb) {
#define PC2_RNS_DO return (const void*)&k_rns_pow<G>
  PC2_RNS_GEOS(PC2_RNS_CASE)
#undef PC2_RNS_DO
  return nullptr;
}

int rns_pow_threads(int t, int nb) {
#define PC2_RNS_DO return G::W * 64
  PC2_RNS_GEOS(PC2_RNS_CASE)
#undef PC2_RNS_DO
  return 0;
}

hipError_t launch_rns_to(const RnsTo& c, int T, int nb, const uint32_t* x, int limbs,
                         size_t count, uint8_t* out, void* stream) {
  const size_t per = (size_t)nb * 32;
  const size_t total = (count + per - 1) / per * per;
  hipLaunchKernelGGL(k_rns_to, dim3((unsigned)((total + 63) / 64), (unsigned)T), dim3(256), 0,
                     (hipStream_t)stream, c, x, limbs, count, T, nb, out);
  return hipGetLastError();
}

hipError_t launch_rns_pow(int t, int nb, int grid, const RnsPow& p, void* stream) {
  const void* k = rns_pow_kernel(t, nb);
  if (!k) return hipErrorInvalidValue;
  void* args[] = {(void*)&p};
  return hipLaunchKernel(k, dim3(grid), dim3(rns_pow_threads(t, nb)), args, 0,
                         (hipStream_t)stream);
}

hipError_t launch_rns_enc_check(const PkConst& pk, const uint32_t* m, int m_limbs,
                                const uint32_t* r, uint32_t* c, size_t count, uint32_t* okw,
                                size_t stride, int* err, void* stream) {
  hipLaunchKernelGGL(k_rns_enc_check, dim3((unsigned)((count + 63) / 64)), dim3(64), 0,
                     (hipStream_t)stream, pk, m, m_limbs, r, c, count, okw, stride, err);
  return hipGetLastError();
}

hipError_t launch_rns_dec_finish(const SkConst& sk, const uint32_t* c, const uint32_t* ys,
                                 size_t stride, size_t count, uint32_t* halves, void* stream) {
  hipLaunchKernelGGL(k_rns_dec_finish, dim3((unsigned)((count + 63) / 64), 2), dim3(64), 0,
                     (hipStream_t)stream, sk, c, ys, stride, count, halves);
  return hipGetLastError();
}

hipError_t launch_rns_from(const RnsFrom& c, int T, int nb, const uint8_t* in, size_t count,
                           uint32_t* out, size_t stride, void* stream) {
  const size_t lds = (size_t)c.nblk * (512 * 4 + 64 * 8);
  hipLaunchKernelGGL(k_rns_from, dim3((unsigned)((count + 63) / 64)), dim3(512), lds,
                     (hipStream_t)stream, c, in, count, T, nb, out, stride);
  return hipGetLastError();
}

}  // namespace pc2k
