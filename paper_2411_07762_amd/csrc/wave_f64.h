// fp64 helpers of the kernels behind the spectra: sums over a wavefront by lane shifts, a reciprocal, an LDS-only barrier.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Sum over the wavefront by lane-shifted additions; every lane returns it.
template <int CTRL, int ROWS>
__device__ __forceinline__ double shifted(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {       // lane: the same in the whole wavefront
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane), hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v += shifted<0x111, 0xf>(v);                          // within rows of 16 lanes: 1, 2, 4, 8 to the right
    v += shifted<0x112, 0xf>(v);
    v += shifted<0x114, 0xf>(v);
    v += shifted<0x118, 0xf>(v);
    v += shifted<0x142, 0xa>(v);                          // the last lane of rows 0 and 2 to rows 1 and 3
    v += shifted<0x143, 0xc>(v);                          // the last lane of row 1 to rows 2 and 3
    return lane_value(v, 63);
}

// a's sum over lanes l and l ^ 32 (l ^ 16) in the lanes where that bit is clear, b's where it is set.
__device__ __forceinline__ double fold32(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
// Sum over each row of 16 lanes, in all of its lanes.
__device__ __forceinline__ double row_sum(double v) {
    v += shifted<0x128, 0xf>(v);                          // rotations by 8, 4, 2, 1
    v += shifted<0x124, 0xf>(v);
    v += shifted<0x122, 0xf>(v);
    v += shifted<0x121, 0xf>(v);
    return v;
}
// The sums of eight values over the wavefront, two per row of 16 lanes: lane l returns those of a[t] and a[t + 4] with
// t = eight_sums_index(l).  18 exchanges instead of the 96 of eight separate sums.
__device__ __forceinline__ int eight_sums_index(int lane) { return ((lane >> 5) & 1) | (((lane >> 4) & 1) << 1); }
__device__ __forceinline__ void eight_sums(const double (&a)[8], double& s0, double& s1) {
    s0 = row_sum(fold16(fold32(a[0], a[1]), fold32(a[2], a[3])));
    s1 = row_sum(fold16(fold32(a[4], a[5]), fold32(a[6], a[7])));
}

__device__ __forceinline__ double rcp_f64(double q) {          // full precision: hardware estimate and two Newton steps
    double r = __builtin_amdgcn_rcp(q);
    r = fma(fma(-q, r, 1.0), r, r);
    return fma(fma(-q, r, 1.0), r, r);
}

__device__ __forceinline__ void lds_barrier() {           // leaves stores to memory on their way
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Sturm counts of a symmetric tridiagonal matrix.  The leading principal minors of T - x I follow p_{l+1} = (d_l - x) p_l - e_{l-1}^2 p_{l-1},
// and the number of eigenvalues below x is the number of sign changes along them.  The matrix is scaled by a power of two to a radius of at
// most one, so that sixteen terms cannot overflow and (p, its predecessor) are brought back to the size of one behind every sixteen; that
// changes no sign.  Three fp64 operations per term, one of them in the chain, against a reciprocal and its two Newton steps of the quotients
// q_l = p_{l+1} / p_l (a chain of 100 cycles).  Squares below kSturmLeast (an e of 1e-18 of the radius) are raised to it, so that a
// minor of exactly zero is followed by one that is not; either sign of the zero gives one change over the two terms.  Sixteen terms
// shrink a minor by 1e-288 at most.
constexpr double kSturmLeast = 1e-36;
constexpr int kSturmTerms = 16;
struct SturmChain {
    double p = 1.0, before = 0.0;
    uint32_t signs = 0;                                   // of the last terms, the newest in bit 0
    int count = 0;
};
// The entry of a term; past the end of the matrix: a positive quotient.
__device__ __forceinline__ double2 sturm_entry(double d, double e, double scale) {
    const double es = e * scale, e2 = es * es;
    return make_double2(d * scale, e2 < kSturmLeast ? kSturmLeast : e2);        // a NaN stays
}
__device__ __forceinline__ double2 sturm_past_end() { return make_double2(4.0, 0.0); }
// The next kSturmTerms terms of P chains that share the matrix: a term comes out of LDS, all lanes reading the same 16 bytes, once for all
// of them (eight cycles of the compute unit's LDS per wavefront).
template <int P>
__device__ __forceinline__ void sturm_terms(SturmChain (&c)[P], const double2* de, const double (&x)[P]) {
#pragma unroll
    for (int u = 0; u < kSturmTerms; ++u) {
        const double2 v = de[u];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const double next = fma(v.x - x[i], c[i].p, -(v.y * c[i].before));
            c[i].before = c[i].p;
            c[i].p = next;
            c[i].signs = __builtin_amdgcn_alignbit(c[i].signs, (uint32_t)__double2hiint(next), 31);
        }
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
        c[i].count += __popc((c[i].signs ^ (c[i].signs >> 1)) & ((1u << kSturmTerms) - 1));
        const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(c[i].p), fabs(c[i].before)));
        c[i].p = __builtin_amdgcn_ldexp(c[i].p, -ex);
        c[i].before = __builtin_amdgcn_ldexp(c[i].before, -ex);
    }
}
// A power of two that brings `radius` to [0.5, 1); 1 where there is none.
__device__ __forceinline__ double sturm_scale(double radius) {
    return (radius > 1e-290 && radius < 1e290) ? __builtin_amdgcn_ldexp(1.0, -__builtin_amdgcn_frexp_exp(radius)) : 1.0;
}
