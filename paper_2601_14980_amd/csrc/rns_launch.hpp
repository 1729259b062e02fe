// Host-side entry points into the RNS kernels (kernels_rns.hip).
#pragma once
#include "pc2_types.hpp"
#include "rns_types.hpp"

namespace pc2k {

const void* rns_pow_kernel(int T, int nb);   // null if (T, nb) is not compiled
int rns_pow_threads(int T, int nb);

// x: [count][limbs] -> residues of both bases in groups of 32 nb elements
hipError_t launch_rns_to(const RnsTo& c, int T, int nb, const uint32_t* x, int limbs,
                         size_t count, uint8_t* out, void* stream);
hipError_t launch_rns_pow(int T, int nb, int grid, const RnsPow& p, void* stream);
// residues of base B in groups of 32 nb elements -> canonical words, element e
// at out + e stride
hipError_t launch_rns_from(const RnsFrom& c, int T, int nb, const uint8_t* in, size_t count,
                           uint32_t* out, size_t stride, void* stream);
// zero the ciphertexts of bad inputs and latch the error, or (okw) write the
// checks to both halves' words okw[(2 e + half) stride]
hipError_t launch_rns_enc_check(const PkConst& pk, const uint32_t* m, int m_limbs,
                                const uint32_t* r, uint32_t* c, size_t count, uint32_t* okw,
                                size_t stride, int* err, void* stream);
hipError_t launch_rns_dec_finish(const SkConst& sk, const uint32_t* c, const uint32_t* ys,
                                 size_t stride, size_t count, uint32_t* halves, void* stream);

}  // namespace pc2k
