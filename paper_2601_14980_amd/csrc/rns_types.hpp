// Device-visible constants of the residue-number-system (RNS) powering engine
// (rns_mont.hpp) and its launch plumbing.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pc2k {

// One odd modulus N in the RNS of T tiles: two bases of 16 T channels each, A
// (moduli a_i, product MA, the Montgomery R) and B (moduli b_j, product MB).
// "Half" h of tile t holds channels 16 t + 8 h .. + 7.
struct RnsMod {
  const uint8_t* E1;    // base extension A -> B: T x T fragments of 1 KB
  const uint8_t* E2;    // base extension B -> A
  const int32_t* c2;    // [T][2 halves][8] initial sums of E2
  const uint32_t* kb;   // [T][2][24]: 1/b_j (8 floats), -b_j (8), F1 pairs (4), F2 pairs (4)
  const uint32_t* ka;   // [T][2][24]: 1/a_i (8 floats), -a_i (8), -MB pairs (8)
};

// Input conversion: sum_i byte_i V_i + add over the input's bytes, V_i = 2^(8 i)
// f, as a product of the matrix cores: E holds the V_i's channel residues, two
// bytes each, as fragments of 32 rows (16 channels) by 32 input bytes; the
// input bytes go in less 128, and cst has what that takes away, and add.
struct RnsTo {
  const uint8_t* E;     // [2 parts][T][nchunk][64 lanes][16]
  const int32_t* cst;   // [chunks used: 0 .. nchunk][2 parts][T][2 halves][8]
  const uint32_t *kb, *ka;  // channel constants (RnsMod)
  int nchunk;           // 32-byte chunks of the longest input
};

// Output conversion: the value mod N (canonical) from the residues mod b_j.
struct RnsFrom {
  const uint32_t* C;    // [limb blocks of 8][16 T][8]: 28-bit limbs of C_j
  const uint32_t* D;    // 28-bit limbs of -MB (or -MB / MA) mod N, 8 blocks limbs
  const uint32_t* O;    // 28-bit limbs of 2^26 N
  const uint32_t* N28;  // 28-bit limbs of N
  const int64_t* F;     // [16 T]: round(2^36 g_j / b_j)
  int S;                // 28-bit limbs of 2^27 N
  int nblk;             // limb blocks: S <= 8 nblk
  int nw;               // 32-bit words of a result
  double ntop_inv;      // 1 / (N's limbs S - 4 .. S - 1 as a number)
};

// Word j of a number in n 28-bit limbs, `stride` words apart; zero past them.  A
// result's words come from the key's declared size, its limbs from the modulus,
// which may be shorter by any amount.
__host__ __device__ inline uint32_t rns_word28(const uint32_t* limb, int n, int stride, int j) {
  const int bit = 32 * j, i = bit / 28, sh = bit % 28;
  uint64_t v = 0;
  if (i < n) v = limb[(size_t)i * stride];
  if (i + 1 < n) v |= (uint64_t)limb[(size_t)(i + 1) * stride] << 28;
  if (i + 2 < n) v |= (uint64_t)limb[(size_t)(i + 2) * stride] << 56;
  return (uint32_t)(v >> sh);
}

// Powering programs (rns_mont.hpp): one word per operation.
constexpr uint32_t RNS_SQ = 0xFF;                          // multiplier: the running value
constexpr uint32_t RNS_GM = 0xFD;                          // multiplier: the second input
constexpr uint32_t RNS_NODST = 0xFF, RNS_OUT = 0xFE;       // destinations
constexpr uint32_t RNS_MUL = 0, RNS_LOAD = 1, RNS_END = 2; // kinds
constexpr uint32_t rns_op(uint32_t kind, uint32_t y, uint32_t dst) {
  return kind << 16 | dst << 8 | y;
}

// The elements of a launch: positions 0 .. npos - 1, cut into groups of 32 nb
// of them.  A job's elements first .. first + count - 1 stand at positions
// pos0 .. (pos0 a multiple of 32); positions of no job hold zeros and produce
// nothing.  One job travels by value, several in device memory, by ascending
// pos0.
struct RnsJob {
  const uint32_t* x;     // encryption: r; decryption: c
  const uint32_t* m;     // encryption: plaintexts
  uint32_t* out;
  uint64_t first;
  uint32_t count, pos0;
  int m_limbs;
};
struct RnsJobs {
  RnsJob one;
  const RnsJob* many;    // null: `one`
  int n;
  uint32_t npos;
};

// A launch of k_rns_pow: nmod moduli (1, or the two primes' squares), each
// with its program and its groups' inputs; item i is group i / nmod of
// modulus i % nmod.
struct RnsPow {
  RnsMod M[2];
  const uint32_t* ops[2];
  uint8_t* in[2];        // first input (Montgomery form) and the result, per group
  uint8_t* gm[2];        // second input, or null
  uint8_t* table;        // per workgroup: entries x one group's residues
  int nmod, ngroups, entries;
};

// one: single values, the same for every element (an entry of 2 T x 32 bytes
// each: base B, base A): MA, MA^2 and 1 mod N.
struct RnsSmul {         // c^k, k_rns_smul
  RnsMod M;
  const uint8_t* one;
  uint8_t* in;           // c, and the result (base B)
  uint8_t* table;        // 16 entries per workgroup
  const uint64_t* k;
  size_t count;
  int ngroups;
};
// A constant of the mat-vec, or (nblk > 1) a block of its bits, in n digits as even
// as the bits allow: the first x of them lo + 1 bits wide, the others lo, which
// holds the smallest tables for a number of digits.  A column's table is entry 0,
// the Montgomery one, for every digit that is zero, and then each digit's entries 1
// .. 2^width - 1.  The blocks share the table: a row takes them from the top, with a
// squaring per bit of a block between two.
struct RnsDigits {
  int n, lo, x, nblk;
  __host__ __device__ static RnsDigits of(int ebits, int n, int nblk) {
    const int bits = (ebits + nblk - 1) / nblk;
    return {n, bits / n, bits % n, nblk};
  }
  __host__ __device__ int bits() const { return lo * n + x; }  // of a block
  __host__ __device__ int wide(int t) const { return t < x ? t : x; }  // of the digits below t
  __host__ __device__ int width(int t) const { return lo + (t < x ? 1 : 0); }
  __host__ __device__ int shift(int t) const { return lo * t + wide(t); }
  // entry d >= 1 of digit t is before(t) + d
  __host__ __device__ uint32_t before(int t) const {
    return (uint32_t)t * ((1u << lo) - 1) + ((uint32_t)wide(t) << lo);
  }
  __host__ __device__ uint32_t entries() const { return before(n) + 1; }
};
struct RnsMvTab {        // k_rns_mvtab
  RnsMod M;
  const uint8_t* one;
  const uint8_t* in;     // c_j
  uint8_t* table;        // one entry per workgroup
  uint8_t* tab;          // [cols][dg.entries()]
  const uint32_t *c, *n2;
  RnsDigits dg;
  int L2, ngroups;
  size_t cols;
  int* err;
};
struct RnsMv {           // k_rns_mv, k_rns_chain
  RnsMod M;
  const uint8_t* one;
  uint8_t* in;           // [chunk][row group]: the running values
  const uint8_t* tab;
  const uint64_t* B;
  uint32_t* bad;         // per row
  size_t rows, cols, chunk_cols;
  RnsDigits dg;
  int alpha, ebits, nch, ngroups;  // alpha: the first chunk's values are set; ngroups: of rows
};

constexpr int RNS_NT = 6, RNS_NBMAX = 4;
constexpr int RNS_T[RNS_NT] = {5, 9, 13, 17, 26, 34};  // compiled tile counts
// the most tiles that a wavefront owns in their geometries: a lane sums over the
// channels of that many tile halves in 32 bits (RGeo, make_rns_base)
constexpr int RNS_MT[RNS_NT] = {1, 2, 3, 2, 3, 4};
constexpr int rns_mt(int T) {
  for (int i = 0; i < RNS_NT; ++i)
    if (RNS_T[i] == T) return RNS_MT[i];
  return 0;
}

// A modulus and its programs for window widths 2..6.
struct RnsKey {
  int T;                    // 0: the engine does not take this modulus
  RnsMod M;
  RnsTo x, gm;              // the power's base (times MA); 1 + m n
  RnsFrom from;
  RnsTo c;                  // modulo n^2: ciphertexts as they are,
  const uint8_t* one;       // and the single values MA, MA^2, 1 (see RnsSmul)
  const uint32_t* ops[5];
};

// bytes of the residues of one group of nb column blocks, both bases
constexpr size_t rns_group_bytes(int T, int nb) { return (size_t)T * nb * 2048; }

}  // namespace pc2k
