// The part of the Householder chain that runs with the matrix on the chip (tridiag_resident.hip), called from spectrum.hip.
#pragma once
#include "aser_internal.h"

constexpr int kAserTridiagTail = 256;                     // rows left to the kernel of one workgroup that ends the chain
constexpr int kAserResidentMost = 4096;                   // rows that fit
struct AserTridiagResident {
    int64_t k, c0;                                        // matrix side; rows and columns from c0 on are left, 256 < k - c0 <= 4096
    double* B;                                            // k x k, both triangles
    const double *vn, *vp, *wp, *tau;                     // reflector to apply and its factor; the pair B still lacks, or null (k entries each)
    double *vn_out, *vp_out, *wp_out, *tau_out;           // the same for the last 256 rows (may be the same memory, tau apart)
    double *d, *e, *vstore, *taustore;                    // as in the chain
    uint64_t* ring;                                       // scratch, 6 (k - c0 + 3) + 2 words, 16-byte aligned (64 is faster)
    int gate_attempts;                                    // of the wait for all workgroups
    bool broken;                                          // as if a wait for an entry had run out of attempts
};
// Enqueues the columns c0 .. k - 257.  *done is false, with nothing enqueued that touches the matrix, where it cannot run: a stream under
// capture, fewer than 256 compute units, no cooperative launch.
int aser_tridiag_resident(aser_ctx* ctx, const AserTridiagResident& a, bool* done);
// Where the launches enqueued leave a word that is not zero when an exchange broke off and nothing they computed may be used.
__host__ __device__ static inline uint64_t* aser_tridiag_broken(const AserTridiagResident& a) { return a.ring + 6 * (a.k - a.c0 + 3) + 1; }
