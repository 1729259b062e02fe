// Host-side entry points into the RNS kernels (kernels_rns.hip).
#pragma once
#include "pc2_types.hpp"
#include "rns_types.hpp"

namespace pc2k {

// null (0) if (T, nb) is not compiled; wide: the geometry for one workgroup a CU
const void* rns_pow_kernel(int T, int nb, bool wide);
int rns_pow_threads(int T, int nb, bool wide);

// the jobs' x (or m) as residues of both bases; limbs: words of an x
hipError_t launch_rns_to(const RnsTo& c, int T, int nb, const RnsJobs& jobs, bool plain,
                         int limbs, uint8_t* out, void* stream);
hipError_t launch_rns_pow(int T, int nb, bool wide, int grid, const RnsPow& p, void* stream);
// residues of base B -> canonical words: at the jobs' outputs (stage null), or
// at stage + position stride
hipError_t launch_rns_from(const RnsFrom& c, int T, int nb, const uint8_t* in,
                           const RnsJobs& jobs, uint32_t* stage, size_t stride, void* stream);
// zero the ciphertexts of bad inputs and latch the error, or (okw) write the
// checks to both halves' words okw[(2 position + half) stride]
hipError_t launch_rns_enc_check(const PkConst& pk, const RnsJobs& jobs, uint32_t* okw,
                                size_t stride, int* err, void* stream);
// the end of a decryption (both halves' y to m), and the recombination of
// key-holder encryption halves
hipError_t launch_rns_dec_finish(const SkConst& sk, const RnsJobs& jobs, const uint32_t* ys,
                                 size_t stride, int* err, void* stream);
hipError_t launch_rns_garner_crt(const SkConst& sk, const RnsJobs& jobs, const uint32_t* stage,
                                 int* err, void* stream);

// kernels with a multiplier per element (null if not compiled for (T, nb));
// rns_pow_threads (not wide) threads; p: the kernel's argument (RnsSmul, RnsMvTab, RnsMv)
enum { RNS_SMUL, RNS_MVTAB, RNS_MV, RNS_MVBLK, RNS_CHAIN, RNS_NGATHER };
const void* rns_gather_kernel(int T, int nb, int which);
hipError_t launch_rns_gather(int T, int nb, int which, int grid, const void* p, void* stream);
// bad[i] = x_i >= n2 (x null: 0); rows with bad[i] zeroed and ERR_RANGE latched
hipError_t launch_rns_row_check(const uint32_t* x, const uint32_t* n2, int L2, uint32_t* bad,
                                size_t rows, void* stream);
hipError_t launch_rns_row_clear(const uint32_t* bad, uint32_t* out, int L2, size_t rows, int* err,
                                void* stream);

}  // namespace pc2k
