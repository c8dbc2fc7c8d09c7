// Symmetric eigen-solver for the Rayleigh-Ritz step of the truncated SVD (Eq. 6): all eigenpairs
// of a b x b matrix (b <= 128), eigenvalues descending; the `need` largest are wanted.  Two kernels:
//
//   tridiag_kernel   one workgroup of 256 threads, the matrix lives in registers (8 x 8 elements per
//                    thread, rows and columns dealt cyclically).
//                    Householder tridiagonalisation M = Q T Q^T in fp32: per reflector one pass that
//                    applies the rank-2 update and forms the mat-vec, and one barrier.
//   ritz_pair_kernel one wavefront per wanted eigenvalue, spread over the chip.  In fp64:
//                    65-section on Sturm counts (9 rounds; wave_f64.h), twisted factorisation of T - lambda I
//                    (forward and backward recurrences side by side in two lanes), eigenvector from
//                    the twist index; then back-transformation through the b - 2 reflectors in fp32.
//
// The tridiagonal problem is solved in fp64 because the spectrum it sees (squared singular values
// of a quantisation-error matrix) has a dense bulk whose spacing is close to fp32 resolution of
// the largest eigenvalue; in fp64 the vectors of distinct eigenvalues come out orthogonal to about
// 1e-16 / relative gap.  If a wanted eigenvalue is closer than 1e-9 of the spectral radius to the next smaller one a flag is
// raised instead and the caller runs the Jacobi solver (2.6 ms), which does not care about clusters.  Nine rounds leave an interval of
// 5e-17 of the radius, below the rounding of the counts: neighbouring vectors at a distance of 1.3e-9 are orthogonal to 8e-8 (measured; the Jacobi solver's
// are to 2e-6 to 8e-6), against 3e-7 at 1e-8 with eight rounds (interval 3e-15; emulated in fp64 on the CPU).  With that limit, and the unwanted
// half of the block looked at too, bulk neighbours met it in four of six traced passes over one 14336 x 4096 layer whose leading eigenvalue is
// far above the bulk; with this one in none.
#include <type_traits>

#include "aser_internal.h"
#include "wave_f64.h"

namespace {

constexpr int kB = 128;

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// sum over each row of 16 lanes, result in every lane of the row
__device__ __forceinline__ float row16_sum(float v) {
    v += dpp_f<0xB1>(v);     // quad_perm [1,0,3,2]
    v += dpp_f<0x4E>(v);     // quad_perm [2,3,0,1]
    v += dpp_f<0x124>(v);    // row_ror 4
    v += dpp_f<0x128>(v);    // row_ror 8
    return v;
}

__device__ __forceinline__ float wave_sum(float v) {
    v = row16_sum(v);
    const int iv = __float_as_int(v);
    return (__int_as_float(__builtin_amdgcn_readlane(iv, 0)) + __int_as_float(__builtin_amdgcn_readlane(iv, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(iv, 32)) + __int_as_float(__builtin_amdgcn_readlane(iv, 48)));
}

// 256 threads in a 16 x 16 grid, thread (ti, tj) holds a[s][c] = A[ti + 16 s][tj + 16 c], s, c = 0..7.
// The 16 lanes of a DPP row share their matrix rows, so the sums of a row never leave it,
// and the cyclic layout lets every thread skip the slots that lie wholly inside the finished part
// (the work shrinks with the trailing block).  Vectors live in LDS in the same cyclic order
// (element i at (i % 16) * 8 + i / 16) so that a thread reads its 8 values as two float4.
//
// Step k starts from u, column k below the diagonal, and from the pair (v, w) of the step before, which A still lacks.  One pass applies the
// pair and sums A u on the way; the rows' sums and column k + 1 go through LDS, behind the only barrier, and as v = scal u +
// (1 - scal alpha) e_{k+1}, A v follows from the two, then w, and the next u from column k + 1, v and w.  Meanwhile the reflector has
// been formed from u.  Every thread forms v, w and u in its own rows and columns, and the wavefronts' sums in a third copy: the
// helpers below keep the copies the same to the last bit.
//
// A u and |u|^2 are of the size of the squared matrix, so its largest entry is brought to [2^54, 2^55) first: nothing in the loop then reaches 2^127, and a
// column counts down to 2^-106 of the largest entry, whatever the scale of the input.  A power of two, taken out of d and e again: no result
// that was in range before is another.
//
// What bounds it: latency, one wavefront per SIMD; a step is 1.2 us.  b = 128: 230 -> 147 us (before: the mat-vec with the normalised reflector behind the
// square root and two divisions, the update in a pass of its own, two barriers).
__device__ __forceinline__ int cyc(int i) { return (i & 15) * 8 + (i >> 4); }
__device__ __forceinline__ float tri_p(float f, float beta, float sum, float col) { return f * fmaf(-beta, col, sum); }
__device__ __forceinline__ float tri_w(float a2, float p, float v) { return fmaf(a2, v, p); }
__device__ __forceinline__ float tri_u(float col, float wj, float v, float w) { return fmaf(-wj, v, col) - w; }

__global__ __launch_bounds__(256) void tridiag_kernel(const float* __restrict__ Mb, int b, float* __restrict__ refl /* [k][128] */,
                                                      float* __restrict__ tri /* d | e | tau, 128 each */,
                                                      int* __restrict__ cluster_flag) {
    // Everything the loop produces stays in LDS until the end: a global store inside the loop
    // would have to drain before each barrier.
    extern __shared__ __align__(16) float sm[];
    __shared__ float largest[4];
    float (*sums)[kB] = (float (*)[kB])sm;              // [2][kB] A u (cyclic order), double-buffered
    float (*cols)[kB] = (float (*)[kB])(sm + 2 * kB);   // [2][kB] column k + 1 (cyclic order)
    float* td = sm + 4 * kB;
    float* te = td + kB;
    float* tt = te + kB;
    float* rs = tt + kB;                                // [b - 2][kB] reflectors (natural order)
    const int tid = threadIdx.x, lane = tid & 63;
    const int ti = tid >> 4, tj = tid & 15;
    const int i0 = (lane >> 3) + 16 * (lane & 7), i1 = i0 + 8;      // natural indices of the cyclic positions lane and lane + 64

    float a[8][8];
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            // unconditional loads from clamped indices: all 128 of a thread are in flight together
            const int r = ti + 16 * s, q = tj + 16 * c;
            const int rc = r < b ? r : b - 1, qc = q < b ? q : b - 1;
            const float lo = Mb[rc * b + qc], up = Mb[qc * b + rc];
            a[s][c] = (r < b && q < b) ? 0.5f * (lo + up) : 0.f;
        }
    float most = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int c = 0; c < 8; ++c) most = fmaxf(most, fabsf(a[s][c]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = fmaxf(most, __shfl_xor(most, o, 64));
    if (lane == 0) largest[tid >> 6] = most;
    if (tid == 0) *cluster_flag = 0;
    if (tid < kB) { td[tid] = 0.f; te[tid] = 0.f; tt[tid] = 0.f; }
    if (tj == 0) {
        *(float4*)(cols[1] + 8 * ti) = make_float4(a[0][0], a[1][0], a[2][0], a[3][0]);
        *(float4*)(cols[1] + 8 * ti + 4) = make_float4(a[4][0], a[5][0], a[6][0], a[7][0]);
    }
    __syncthreads();
    const int up = 55 - __builtin_amdgcn_frexp_expf(fmaxf(fmaxf(largest[0], largest[1]), fmaxf(largest[2], largest[3])));
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int c = 0; c < 8; ++c) a[s][c] = __builtin_amdgcn_ldexpf(a[s][c], up);
    auto eight = [](const float* at, float (&x)[8]) {
        const float4 p = *(const float4*)at, q = *(const float4*)(at + 4);
        x[0] = p.x; x[1] = p.y; x[2] = p.z; x[3] = p.w; x[4] = q.x; x[5] = q.y; x[6] = q.z; x[7] = q.w;
    };
    auto at_position = [](float lo, float hi, int pos) {            // pos: the same in the whole wavefront
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pos < 64 ? lo : hi), pos & 63));
    };
    float ur[8], uc[8], vr[8], vc[8], wr[8], wc[8];     // u, v, w in this thread's rows and columns; u is 0 up to row k
    eight(cols[1] + 8 * ti, ur);
    eight(cols[1] + 8 * tj, uc);
    float u0 = i0 > 0 ? __builtin_amdgcn_ldexpf(cols[1][lane], up) : 0.f, u1 = __builtin_amdgcn_ldexpf(cols[1][lane + 64], up);      // u at the positions lane and lane + 64
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        ur[s] = __builtin_amdgcn_ldexpf(ur[s], up);
        uc[s] = __builtin_amdgcn_ldexpf(uc[s], up);
    }
    if (ti == 0) ur[0] = 0.f;
    if (tj == 0) uc[0] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) vr[s] = vc[s] = wr[s] = wc[s] = 0.f;
    if (tid == 0) td[0] = a[0][0];

    int k = 0;
    // the steps whose row k + 1 lies in slot S0: the slots below are done with, those above hold rows and columns behind it only
    auto steps = [&](auto first) {
        constexpr int S0 = decltype(first)::value;
        for (; k + 2 < b && k + 1 < 16 * (S0 + 1); ++k) {
            float* const sum = sums[k & 1];
            float* const col = cols[k & 1];
            // A -= v w^T + w v^T on the trailing block, and A u
            float ps[8];
#pragma unroll
            for (int s = S0; s < 8; ++s) {
                ps[s] = 0.f;
#pragma unroll
                for (int c = S0; c < 8; ++c) {
                    a[s][c] = fmaf(-wr[s], vc[c], fmaf(-vr[s], wc[c], a[s][c]));
                    ps[s] = fmaf(a[s][c], uc[c], ps[s]);
                }
            }
#pragma unroll
            for (int s = S0; s < 8; ++s) ps[s] = row16_sum(ps[s]);
            if (tj == 0) {
#pragma unroll
                for (int s = S0; s < 8; ++s) sum[8 * ti + s] = ps[s];
            }
            if (tj == ((k + 1) & 15)) {
#pragma unroll
                for (int s = S0; s < 8; ++s) col[8 * ti + s] = a[s][S0];
            }
            // reflector k annihilates A[k+2.., k]
            const int jpos = cyc(k + 1);
            const float alpha = at_position(u0, u1, jpos);
            const float sigma = wave_sum((lane != jpos ? u0 * u0 : 0.f) + (lane + 64 != jpos ? u1 * u1 : 0.f));
            float beta = alpha, tk = 0.f, scal = 0.f;
            if (sigma > 1e-30f * alpha * alpha && sigma > 0.f) {
                beta = -copysignf(sqrtf(alpha * alpha + sigma), alpha);
                tk = (beta - alpha) / beta;
                scal = 1.0f / (alpha - beta);
            }
            const float f = tk * scal;
            const float v0 = lane == jpos ? 1.f : u0 * scal, v1 = lane + 64 == jpos ? 1.f : u1 * scal;
#pragma unroll
            for (int s = S0; s < 8; ++s) {
                vr[s] = (s == S0 && ti + 16 * s == k + 1) ? 1.f : ur[s] * scal;
                vc[s] = (s == S0 && tj + 16 * s == k + 1) ? 1.f : uc[s] * scal;
            }
            if (tj == 0) {
#pragma unroll
                for (int s = 0; s < 8; ++s) rs[k * kB + ti + 16 * s] = s < S0 ? 0.f : vr[s];
            }
            if (tid == 0) { te[k] = beta; tt[k] = tk; }
            __syncthreads();
            // w = p - (tau/2)(p^T v) v with p = tau A v, and the next u
            const float c0 = col[lane], c1 = col[lane + 64];
            const float p0 = i0 > k ? tri_p(f, beta, sum[lane], c0) : 0.f, p1 = i1 > k ? tri_p(f, beta, sum[lane + 64], c1) : 0.f;
            const float a2 = -0.5f * tk * wave_sum(p0 * v0 + p1 * v1);
            const float w0 = tri_w(a2, p0, v0), w1 = tri_w(a2, p1, v1);
            const float wj = at_position(w0, w1, jpos);
            u0 = i0 > k + 1 ? tri_u(c0, wj, v0, w0) : 0.f;
            u1 = i1 > k + 1 ? tri_u(c1, wj, v1, w1) : 0.f;
            float sr[8], sc[8], cr[8], cc[8];
            eight(sum + 8 * ti, sr);
            eight(sum + 8 * tj, sc);
            eight(col + 8 * ti, cr);
            eight(col + 8 * tj, cc);
#pragma unroll
            for (int s = S0; s < 8; ++s) {
                const bool rin = s > S0 || ti + 16 * s > k, cin = s > S0 || tj + 16 * s > k;
                wr[s] = rin ? tri_w(a2, tri_p(f, beta, sr[s], cr[s]), vr[s]) : 0.f;
                wc[s] = cin ? tri_w(a2, tri_p(f, beta, sc[s], cc[s]), vc[s]) : 0.f;
                ur[s] = (s > S0 || ti + 16 * s > k + 1) ? tri_u(cr[s], wj, vr[s], wr[s]) : 0.f;
                uc[s] = (s > S0 || tj + 16 * s > k + 1) ? tri_u(cc[s], wj, vc[s], wc[s]) : 0.f;
            }
            if (tid == 0) td[k + 1] = fmaf(-2.f, wj, col[jpos]);
        }
    };
    steps(std::integral_constant<int, 0>{});
    steps(std::integral_constant<int, 1>{});
    steps(std::integral_constant<int, 2>{});
    steps(std::integral_constant<int, 3>{});
    steps(std::integral_constant<int, 4>{});
    steps(std::integral_constant<int, 5>{});
    steps(std::integral_constant<int, 6>{});
    steps(std::integral_constant<int, 7>{});
    // the last 2 x 2 block
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        if (ti + 16 * s != b - 1) continue;
        if (tj == 0) te[b - 2] = ur[s];
        if (tj == ti) td[b - 1] = fmaf(-2.f * wr[s], vr[s], a[s][s]);
    }
    __syncthreads();
    for (int t = tid; t < (b - 2) * kB; t += 256) refl[t] = rs[t];
    for (int t = tid; t < 3 * kB; t += 256) tri[t] = t < 2 * kB ? __builtin_amdgcn_ldexpf(td[t], -up) : td[t];
}

__device__ __forceinline__ double wave_max_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_min_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}

// number of eigenvalues of the tridiagonal (padded to a multiple of kSturmTerms) below x
__device__ __forceinline__ int sturm_count(const double2* de, int padded, double x) {
    SturmChain c[1];
    const double xs[1] = {x};
    for (int i = 0; i < padded; i += kSturmTerms) sturm_terms(c, de + i, xs);
    return c[0].count;
}

// One wavefront: eigenvalue number blockIdx.x (descending; m counts ascending) of the tridiagonal and its eigenvector,
// mapped back through the reflectors.  Writes lambda[b - 1 - m] and column b - 1 - m of Vout.
__global__ __launch_bounds__(64) void ritz_pair_kernel(const float* __restrict__ tri, const float* __restrict__ refl, int b,
                                                       float* __restrict__ lambda, float* __restrict__ Vout,
                                                       int* __restrict__ cluster_flag) {
    __shared__ __align__(16) double2 de[kB];        // (d_i, e_{i-1}^2), scaled by a power of two
    __shared__ double es[kB], Dp[kB], Dm[kB], zz[kB];
    __shared__ float tau[kB];
    extern __shared__ __align__(16) float rl[];     // [b - 2][kB] reflectors, read once up front
    const int lane = threadIdx.x;
    const int m = b - 1 - (int)blockIdx.x;
    // the reflectors, 16 float4 per lane in flight at a time
    for (int t0 = 0; t0 < (b - 2) * (kB / 4); t0 += 64 * 16) {
        float4 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int t = t0 + u * 64 + lane;
            v[u] = (t < (b - 2) * (kB / 4)) ? ((const float4*)refl)[t] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int t = t0 + u * 64 + lane;
            if (t < (b - 2) * (kB / 4)) ((float4*)rl)[t] = v[u];
        }
    }

    double glo = 1e300, ghi = -1e300;
    float df[2], el[2], ei[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + 64 * u;
        df[u] = (i < b) ? tri[i] : 0.f;
        ei[u] = (i + 1 < b) ? tri[kB + i] : 0.f;
        el[u] = (i > 0 && i < b) ? tri[kB + i - 1] : 0.f;
        tau[i] = (i + 2 < b) ? tri[2 * kB + i] : 0.f;
        if (i < b) {
            const double rad = fabs((double)ei[u]) + fabs((double)el[u]);
            glo = fmin(glo, (double)df[u] - rad);
            ghi = fmax(ghi, (double)df[u] + rad);
        }
    }
    glo = wave_min_d(glo);
    ghi = wave_max_d(ghi);
    const double scale = sturm_scale(fmax(fabs(glo), fabs(ghi)));
    glo *= scale;
    ghi *= scale;
    const double radius = fmax(fabs(glo), fabs(ghi));
    const double tiny = fmax(radius * 1e-60, 1e-290);
    const int padded = (b + kSturmTerms - 1) / kSturmTerms * kSturmTerms;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + 64 * u;
        de[i] = i < b ? sturm_entry((double)df[u], (double)el[u], scale) : sturm_past_end();
        es[i] = (double)ei[u] * scale;
    }
    __syncthreads();

    // ---- eigenvalue: 64 interior points per round
    double lo = glo - 1e-12 * radius - tiny, hi = ghi + 1e-12 * radius + tiny;
    for (int round = 0; round < 9; ++round) {
        const double x = lo + (hi - lo) * ((double)(lane + 1) * (1.0 / 65.0));
        const int cnt = sturm_count(de, padded, x);
        const double clo = wave_max_d((cnt <= m) ? x : lo);
        const double chi = wave_min_d((cnt > m) ? x : hi);
        lo = clo;
        hi = chi;
    }
    const double lam = 0.5 * (lo + hi);
    int bad = 0;
    if (m > 0) bad = sturm_count(de, padded, lam - 1e-9 * radius) < m;

    // ---- twisted factorisation: lane 0 runs D+ downwards, lane 1 runs D- upwards
    {
        const int dir = lane & 1;
        double q = 0.0;
        for (int t = 0; t < b; ++t) {
            const int i = dir ? (b - 1 - t) : t;
            const double dx = de[i].x - lam;
            q = (t == 0) ? dx : fma(-de[dir ? i + 1 : i].y, rcp_f64(q), dx);
            if (fabs(q) < tiny) q = tiny;
            if (lane < 2) (dir ? Dm : Dp)[i] = q;
        }
    }
    __syncthreads();
    int twist;
    {
        double best = 1e300;
        int bi = 0;
        for (int i = lane; i < b; i += 64) {
            const double g = fabs(Dp[i] + Dm[i] - (de[i].x - lam));
            if (g < best) { best = g; bi = i; }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double ob = __shfl_xor(best, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (ob < best || (ob == best && oi < bi)) { best = ob; bi = oi; }
        }
        twist = bi;
    }
    // z_twist = 1; z_i = -(e_i / D+_i) z_{i+1} above it, z_i = -(e_{i-1} / D-_i) z_{i-1} below it
    for (int i = lane; i < b; i += 64) {
        double rat = 1.0;
        if (i < twist) rat = -es[i] * rcp_f64(Dp[i]);
        if (i > twist) rat = -es[i - 1] * rcp_f64(Dm[i]);
        zz[i] = rat;
    }
    __syncthreads();
    {
        const int dir = lane & 1;
        const int steps = max(twist, b - 1 - twist);
        double z = 1.0;
        for (int t = 1; t <= steps; ++t) {
            const int i = dir ? twist + t : twist - t;
            if (i >= 0 && i < b && lane < 2) {
                z *= zz[i];
                zz[i] = z;
            }
        }
    }
    __syncthreads();
    float y0, y1;
    {
        const double z0 = (lane < b) ? zz[lane] : 0.0, z1 = (lane + 64 < b) ? zz[lane + 64] : 0.0;
        double nrm = z0 * z0 + z1 * z1;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) nrm += __shfl_xor(nrm, o, 64);
        if (!(nrm < 1e300)) bad = 1;
        const double inv = 1.0 / sqrt(nrm);
        y0 = (float)(z0 * inv);
        y1 = (float)(z1 * inv);
    }
    if (bad && lane == 0) *cluster_flag = 1;

    // ---- back-transformation y <- H_0 H_1 ... H_{b-3} y
    if (b >= 3) {
        float v0 = rl[(b - 3) * kB + lane], v1 = rl[(b - 3) * kB + lane + 64];
        for (int k = b - 3; k >= 0; --k) {
            const int kn = k > 0 ? k - 1 : 0;
            const float n0 = rl[kn * kB + lane], n1 = rl[kn * kB + lane + 64];
            const float s = tau[k] * wave_sum(v0 * y0 + v1 * y1);
            y0 -= s * v0;
            y1 -= s * v1;
            v0 = n0;
            v1 = n1;
        }
    }
    const int c = b - 1 - m;
    if (lane == 0) lambda[c] = (float)(lam / scale);
    if (lane < b) Vout[lane * b + c] = y0;
    if (lane + 64 < b) Vout[(lane + 64) * b + c] = y1;
}

}  // namespace

int aser_tridiag_eig(aser_ctx* ctx, const float* Mb, int b, float* lambda, float* V, float* refl, float* tri, int* cluster_flag, int need) {
    if (need < 1 || need > b) ASER_FAIL(ctx, ASER_ERR_SHAPE, "sym_eig: 1 to b eigenpairs");
    if (b < 2 || b > kB) ASER_FAIL(ctx, ASER_ERR_SHAPE, "sym_eig: block size must be in [2, 128]");
    static bool attr_set[16] = {false};
    const size_t lds = (size_t)(7 + (kB - 2)) * kB * sizeof(float);
    const size_t lds_r = (size_t)(kB - 2) * kB * sizeof(float);
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)tridiag_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)ritz_pair_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_r));
        attr_set[ctx->device] = true;
    }
    hipLaunchKernelGGL(tridiag_kernel, dim3(1), dim3(256), lds, ctx->stream, Mb, b, refl, tri, cluster_flag);
    hipLaunchKernelGGL(ritz_pair_kernel, dim3(need), dim3(64), lds_r, ctx->stream, (const float*)tri, (const float*)refl, b, lambda, V,
                       cluster_flag);
    return aser_check_launch(ctx, "tridiag_eig");
}
