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

// Residues of one wavefront's slot (part, tile, half: eight channels) for 64
// positions, one per lane: sum_i half_i P[i] + add.  The constants are uniform
// (scalar loads).
__global__ __launch_bounds__(256) void k_rns_to(RnsTo C, pc2k::RnsJobs J, bool plain, int limbs,
                                                int T, int nb, uint8_t* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int slot = __builtin_amdgcn_readfirstlane(blockIdx.y * 4 + (threadIdx.x >> 6));
  if (slot >= 4 * T) return;
  const uint32_t pos = blockIdx.x * 64 + lane;
  const uint32_t per = nb * 32;
  if (pos >= (J.npos + per - 1) / per * per) return;
  pc2k::RnsJob j;
  size_t e;
  const bool live = find_job(J, pos, j, e);
  if (plain) limbs = j.m_limbs;
  const int nhalf = !live ? 0 : 2 * limbs < C.nhalf ? 2 * limbs : C.nhalf;
  const uint32_t* P = C.P + (size_t)slot * C.nhalf * 8;
  const uint32_t* xe = (plain ? j.m : j.x) + e * limbs;
  uint64_t acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = C.add[slot * 8 + c];
  // (uniform bound: lanes of shorter or no inputs add zeros)
  const int top = plain ? C.nhalf : 2 * limbs < C.nhalf ? 2 * limbs : C.nhalf;
  for (int i = 0; i < top; i += 2) {
    if (plain && __ballot(i < nhalf) == 0) break;
    const uint32_t w = i < nhalf ? xe[i >> 1] : 0u;
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
  const uint32_t grp = pos / per, b = pos % per / 32, n = pos & 31;
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
    for (int j = lane; j < C.nw; j += 64) {
      const int bit = 32 * j, i = bit / 28, sh = bit % 28;
      uint64_t v = limb[i * 64 + e];
      if (i + 1 < 8 * nblk) v |= (uint64_t)limb[(i + 1) * 64 + e] << 28;
      if (i + 2 < 8 * nblk) v |= (uint64_t)limb[(i + 2) * 64 + e] << 56;
      out[j] = (uint32_t)(v >> sh);
    }
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

// The scalar end of a decryption half, one lane per (position, prime): y =
// c^(s-1) mod s^2 (canonical, nl words at y + (2 pos + half) stride) -> m_s =
// L_s(y) h_s mod s and its validity word at halves + (2 pos + half)(Ls + 1).
__global__ __launch_bounds__(64) void k_rns_dec_finish(pc2k::SkConst sk, pc2k::RnsJobs J,
                                                       const uint32_t* __restrict__ ys,
                                                       size_t stride,
                                                       uint32_t* __restrict__ halves) {
  const uint32_t pos = blockIdx.x * 64 + threadIdx.x;
  const int half = blockIdx.y;
  pc2k::RnsJob j;
  size_t e;
  if (pos >= J.npos || !find_job(J, pos, j, e)) return;
  const pc2k::HalfConst& H = sk.h[half];
  const int Ls = H.Ls, nl = H.s2.nl, L2 = 2 * sk.pk.L;
  const bool cv = pc2d::sc_cmp(j.x + e * L2, L2, sk.pk.n2.Nl, L2) < 0;
  uint32_t y[2 * pc2k::LS_MAX + 1], u[pc2k::LS_MAX], us[2 * pc2k::LS_MAX],
      tmp[pc2k::LS_MAX + 2];
  const size_t at = 2 * (size_t)pos + half;
  const uint32_t* src = ys + at * stride;
  for (int k = 0; k < nl; ++k) y[k] = src[k];
  const uint32_t one = 1u;
  const uint32_t bor = pc2d::sc_sub(y, nl, &one, 1);
  pc2d::sc_mullo(u, y, H.sinv, Ls);
  pc2d::sc_mul(us, u, Ls, H.s, Ls);
  const bool good = bor == 0 && pc2d::sc_cmp(us, 2 * Ls, y, nl) == 0 && cv;
  uint32_t* dst = halves + at * (size_t)(Ls + 1);
  pc2d::sc_montmul(u, u, H.H, H.s, H.s_n0, Ls, tmp);
  for (int k = 0; k < Ls; ++k) dst[k] = u[k];
  dst[Ls] = good ? 1u : 0u;
}

// CRT recombination of decryption halves, one lane per position.
__global__ __launch_bounds__(64) void k_rns_garner(pc2k::SkConst sk, pc2k::RnsJobs J,
                                                   const uint32_t* __restrict__ halves,
                                                   int* err) {
  const uint32_t pos = blockIdx.x * 64 + threadIdx.x;
  pc2k::RnsJob j;
  size_t e;
  if (pos >= J.npos || !find_job(J, pos, j, e)) return;
  const int Ls = sk.h[0].Ls;
  uint32_t work[5 * pc2k::LS_MAX + 2];
  const uint32_t* hp = halves + pos * 2 * (size_t)(Ls + 1);
  pc2ops::garner_elem(sk, hp, hp + Ls + 1, j.out + e * sk.pk.L, err, work);
}

// Recombination of key-holder encryption halves modulo n^2, one lane per position.
__global__ __launch_bounds__(64) void k_rns_garner_crt(pc2k::SkConst sk, pc2k::RnsJobs J,
                                                       const uint32_t* __restrict__ stage,
                                                       int* err) {
  const uint32_t pos = blockIdx.x * 64 + threadIdx.x;
  pc2k::RnsJob j;
  size_t e;
  if (pos >= J.npos || !find_job(J, pos, j, e)) return;
  const int n2 = sk.h[0].s2.nl;
  uint32_t work[10 * pc2k::LS_MAX + 2];
  const uint32_t* cp = stage + pos * 2 * (size_t)(n2 + 1);
  pc2ops::garner_crt_elem(sk, cp, cp + n2 + 1, j.out + e * 2 * (size_t)sk.pk.L, err, work);
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
  D(13, 1, 8, false) D(13, 2, 4, false)                                       \
  D(17, 1, 8, true) D(17, 2, 8, true) D(17, 4, 8, true)                       \
  D(26, 1, 8, true) D(26, 2, 8, true)                                         \
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

hipError_t launch_rns_to(const RnsTo& c, int T, int nb, const RnsJobs& jobs, bool plain,
                         int limbs, uint8_t* out, void* stream) {
  const uint32_t per = nb * 32;
  const uint32_t total = (jobs.npos + per - 1) / per * per;
  hipLaunchKernelGGL(k_rns_to, dim3((total + 63) / 64, (unsigned)T), dim3(256), 0,
                     (hipStream_t)stream, c, jobs, plain, limbs, T, nb, out);
  return hipGetLastError();
}

hipError_t launch_rns_pow(int t, int nb, int grid, const RnsPow& p, void* stream) {
  const void* k = rns_pow_kernel(t, nb);
  if (!k) return hipErrorInvalidValue;
  void* args[] = {(void*)&p};
  return hipLaunchKernel(k, dim3(grid), dim3(rns_pow_threads(t, nb)), args, 0,
                         (hipStream_t)stream);
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

hipError_t launch_rns_dec_finish(const SkConst& sk, const RnsJobs& jobs, const uint32_t* ys,
                                 size_t stride, uint32_t* halves, int* err, void* stream) {
  if (sk.h[0].Ls > LS_MAX || sk.h[0].s2.nl > 2 * LS_MAX) return hipErrorInvalidValue;
  const unsigned blocks = (jobs.npos + 63) / 64;
  hipLaunchKernelGGL(k_rns_dec_finish, dim3(blocks, 2), dim3(64), 0, (hipStream_t)stream, sk,
                     jobs, ys, stride, halves);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rns_garner, dim3(blocks), dim3(64), 0, (hipStream_t)stream, sk, jobs,
                     halves, err);
  return hipGetLastError();
}

hipError_t launch_rns_garner_crt(const SkConst& sk, const RnsJobs& jobs, const uint32_t* stage,
                                 int* err, void* stream) {
  if (sk.h[0].s2.nl > 2 * LS_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_rns_garner_crt, dim3((jobs.npos + 63) / 64), dim3(64), 0,
                     (hipStream_t)stream, sk, jobs, stage, err);
  return hipGetLastError();
}

}  // namespace pc2k
