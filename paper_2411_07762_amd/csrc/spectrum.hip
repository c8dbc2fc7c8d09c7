// The whole singular spectrum of the whitened error T S (Eq. 6), and what the paper derives from it:
// the rank chosen by the threshold alpha on the cumulative sum of singular values (Eq. 9) and the
// effective rank, the exponential of the entropy of the normalised singular values (Eq. 3, Eq. 4).
//
// A truncated solver does not produce the sum over ALL singular values that Eq. 9 divides by, so this
// path computes every one of them, in fp64 behind the product T S:
//   B = Z Z^T  (k x k, k = min(m, n), Z = T S or its transpose)   fp64 accumulation of exact fp32 products
//   B -> tridiagonal (d, e) by Householder reflections            on the chip up to 4096 columns (tridiag_resident.hip), else see below
//   eigenvalues of (d, e) by multisection on Sturm counts         16 to 64 lanes per eigenvalue
//   sigma_i = sqrt(lambda_i), descending.
// The singular values of T S and of (T S)^T agree, so B is formed on the shorter side.
//
// Tridiagonalisation, where the matrix does not stay on the chip: more than 4096 columns left, fewer than kResidentLeast, several layers in
// flight (the cooperative launch would hold every compute unit), a stream under capture.  Step j turns column j into (d_j, e_j, 0, ...) with H = I - tau v v^T and needs
// p = tau B22 v and the rank-2 update B22 -= v w^T + w v^T with w = p - (tau / 2)(v^T p) v.  A step is one launch:
// a pass over the trailing matrix that forms B22 v with the updates of the last (up to four) steps applied on the fly, of
// which one in up to four also writes the updated matrix, and in the workgroup that finishes last the reflector of the next
// step.  A step moves 8 bytes per entry of the trailing matrix, or 16 when it writes: 10 on average while at least 2048 columns
// are left (one of four steps writes), 12 down to 1024 (one of two), 16 below, where the launch is what a step costs; the
// last 256 columns do not leave one workgroup.  Bound by HBM or the last-level cache when B fits.
// B is kept as a full symmetric matrix so that every pass walks rows with unit stride.
#include <math.h>

#include "aser_internal.h"
#include "tridiag_resident.h"
#include "wave_f64.h"

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------------
// B += P^T P for P: K x k fp32 (row-major, ldp), B: k x k fp64 (ld = k), lower-triangle tiles of
// 64 x 64 written to both (i, j) and (j, i).  256 threads as 16 x 16, a 4 x 4 block of B each.
// K is split over blockIdx.y; partial tiles are added with fp64 atomics (B is cleared first).
template <typename TIN>
__global__ __launch_bounds__(256) void gram_f64_kernel(const TIN* __restrict__ P, int64_t K, int64_t k, int64_t ldp,
                                                       double* __restrict__ B, int k_parts) {
    typedef TIN tin4_t __attribute__((ext_vector_type(4)));
    __shared__ __align__(32) TIN sa[16][64];
    __shared__ __align__(32) TIN sb[16][64];
    const int64_t t = blockIdx.x;
    int64_t bi = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (bi * (bi + 1) / 2 > t) --bi;
    while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
    const int64_t bj = t - bi * (bi + 1) / 2;
    const int64_t I0 = bi * 64, J0 = bj * 64;
    const int64_t per = (((K + 15) / 16 + k_parts - 1) / k_parts) * 16;
    const int64_t k0 = (int64_t)blockIdx.y * per;
    const int64_t k1 = (k0 + per < K) ? k0 + per : K;
    if (k0 >= k1) return;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int lr = tid >> 4, lc = (tid & 15) * 4;          // this thread's 4 floats of a 16 x 64 slab
    const bool vec_ok = (((uintptr_t)P & (4 * sizeof(TIN) - 1)) == 0) && ((ldp & 3) == 0);
    double acc[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
    for (int64_t kk = k0; kk < k1; kk += 16) {
        const int64_t row = kk + lr;
        tin4_t a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
        if (row < k1) {
            const TIN* pr = P + row * ldp;
            if (vec_ok && I0 + lc + 4 <= k) a = *(const tin4_t*)(pr + I0 + lc);
            else
                for (int e = 0; e < 4; ++e)
                    if (I0 + lc + e < k) a[e] = pr[I0 + lc + e];
            if (vec_ok && J0 + lc + 4 <= k) b = *(const tin4_t*)(pr + J0 + lc);
            else
                for (int e = 0; e < 4; ++e)
                    if (J0 + lc + e < k) b[e] = pr[J0 + lc + e];
        }
        __syncthreads();                                  // the previous slab has been consumed
        *(tin4_t*)&sa[lr][lc] = a;
        *(tin4_t*)&sb[lr][lc] = b;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const tin4_t av = *(const tin4_t*)&sa[s][ty * 4];
            const tin4_t bv = *(const tin4_t*)&sb[s][tx * 4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = fma((double)av[u], (double)bv[v], acc[u][v]);
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t i = I0 + ty * 4 + u, j = J0 + tx * 4 + v;
            if (i >= k || j >= k) continue;
            if (bi == bj && j > i) continue;              // diagonal tile: the lower half is mirrored below
            unsafeAtomicAdd(B + i * k + j, acc[u][v]);
            if (i != j) unsafeAtomicAdd(B + j * k + i, acc[u][v]);
        }
}

__device__ __forceinline__ double block_sum(double v, double* red) {   // blockDim.x multiple of 64, <= 1024
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();                                      // red may still be read from an earlier call
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double r = 0.0;
    for (int i = 0; i < nw; ++i) r += red[i];
    return r;
}

// Values that another workgroup of the same launch reads or wrote: agent-scope accesses, which do not stop in a cache that the
// other compute units do not share.
__device__ __forceinline__ void publish(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double published(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

constexpr int kTriThreads = 512, kTriRows = 8, kTriPairs = 4, kResidentLeast = 320;

struct TridiagStep {
    int64_t c0, k;
    double* B;
    const double* v[kTriPairs];           // pending pairs: B still lacks - v w^T - w v^T for each of them
    const double* w[kTriPairs];
    const double* vn;                     // the reflector of this step
    double *wn, *vnext;                   // out: its w, and the next reflector
    double *p, *eff;                      // B vn, and row c0 of the up-to-date matrix
    double *d, *e;
    const double* tau_cur; double* tau_next;
    int* counter;                         // workgroups that have finished (0 between launches)
    double *vstore, *taustore;            // reflectors kept for a back-transformation, or null
    const uint64_t* broken;               // not null and the word not zero: what the tail kernel is given may not be used
};

// The start of the chain: d_0 and the first reflector from row 0 of B (or the whole of a matrix of one or two rows).
__global__ __launch_bounds__(kTriThreads) void tridiag_first_kernel(TridiagStep a) {
    __shared__ double red[16];
    const int tid = threadIdx.x;
    const int64_t k = a.k;
    if (tid == 0) a.d[0] = a.B[0];
    if (k > 2) {
        double n2 = 0.0;
        for (int64_t i = 1 + tid; i < k; i += kTriThreads) {
            const double c = a.B[i];
            a.vnext[i] = c;
            if (a.vstore) a.vstore[i] = c;
            n2 += c * c;
        }
        n2 = block_sum(n2, red);
        __syncthreads();
        if (tid == 0) {
            const double x0 = a.B[1];
            const double alpha = (x0 > 0.0) ? -sqrt(n2) : sqrt(n2);
            const double v0 = x0 - alpha, vn2 = n2 - x0 * x0 + v0 * v0, tnew = vn2 > 0.0 ? 2.0 / vn2 : 0.0;
            a.vnext[1] = v0;
            *a.tau_next = tnew;
            a.e[0] = alpha;
            if (a.vstore) { a.vstore[1] = v0; a.taustore[0] = tnew; }
        }
    } else if (k == 2 && tid == 0) {
        a.e[0] = a.B[1];
        a.d[1] = a.B[3];
    }
}

// One step of the chain in one launch, while more than kTailRows rows are left.  Every workgroup takes 8 rows of the trailing matrix (rows and columns >= c0): it
// forms p_i = sum_l B_il vn_l on the up-to-date values, which are B minus the NP pending rank-2 updates; with
// WRITE they also go back to memory and nothing is pending any more, otherwise the pass only reads.  The workgroup
// that finishes last then has all of p: w = tau p - (tau^2 / 2)(vn^T p) vn, and from row c0 of the matrix after this
// step's own update the next diagonal entry, the next off-diagonal one and the next reflector.
// What bounds it: 8 (k - j)^2 bytes per read-only pass and twice that per writing one (one in up to four), from the last-level
// cache when B fits, and the tail of the last workgroup; a launch per column and role (pass, reflector) and a read and a
// write of B in every pass were 26.7 us per column at k = 4096, this is 19.7.
// W columns per thread and round: two where rows start on 16 bytes (k even): half as many loads, twice as wide (k = 4096: 84.6 -> 82.4 ms in all).
template <int NP, bool WRITE, int W>
__global__ __launch_bounds__(kTriThreads) void tridiag_step_kernel(TridiagStep a) {
    typedef double dvec __attribute__((ext_vector_type(W)));
    __shared__ double red[kTriThreads / 64][kTriRows];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t c0 = a.c0, k = a.k, r0 = c0 + (int64_t)blockIdx.x * kTriRows;
    const int nrows = (int)((k - r0 < kTriRows) ? k - r0 : kTriRows);
    {
        constexpr int NQ = NP > 0 ? NP : 1;
        double vi[NQ][kTriRows], wi[NQ][kTriRows], acc[kTriRows];
        double* rowp[kTriRows];
#pragma unroll
        for (int r = 0; r < kTriRows; ++r) {
            const int64_t i = (r0 + r < k) ? r0 + r : k - 1;       // rows past the end repeat the last row; their results are dropped
#pragma unroll
            for (int q = 0; q < NP; ++q) { vi[q][r] = a.v[q][i]; wi[q][r] = a.w[q][i]; }
            rowp[r] = a.B + i * k;
            acc[r] = 0.0;
        }
        for (int64_t l = (c0 & ~(int64_t)(W - 1)) + W * tid; l < k; l += W * kTriThreads) {
            dvec vl[NQ], wl[NQ], b[kTriRows], vnl = *(const dvec*)(a.vn + l);
#pragma unroll
            for (int r = 0; r < kTriRows; ++r) b[r] = *(const dvec*)(rowp[r] + l);
#pragma unroll
            for (int q = 0; q < NP; ++q) { vl[q] = *(const dvec*)(a.v[q] + l); wl[q] = *(const dvec*)(a.w[q] + l); }
            // the column before c0 belongs to the chain's past: what stands there is not touched and counts nothing
            const bool past = W == 2 && l < c0;
            if (past) vnl[0] = 0.0;
#pragma unroll
            for (int r = 0; r < kTriRows; ++r) {
                const double before = b[r][0];
#pragma unroll
                for (int q = 0; q < NP; ++q) b[r] -= vi[q][r] * wl[q] + wi[q][r] * vl[q];
                if (past) b[r][0] = before;
                if (WRITE && r < nrows) *(dvec*)(rowp[r] + l) = b[r];
                if (past) b[r][0] = 0.0;
#pragma unroll
                for (int u = 0; u < W; ++u) acc[r] = fma(b[r][u], vnl[u], acc[r]);
            }
            if (blockIdx.x == 0) {
#pragma unroll
                for (int u = 0; u < W; ++u) publish(a.eff + l + u, b[0][u]);
            }
        }
#pragma unroll
        for (int r = 0; r < kTriRows; ++r) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) acc[r] += __shfl_xor(acc[r], o, 64);
            if (lane == 0) red[wave][r] = acc[r];
        }
    }
    __syncthreads();
    if (tid < nrows) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < kTriThreads / 64; ++u) s += red[u][tid];
        publish(a.p + r0 + tid, s);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // what this wavefront published has arrived
    __syncthreads();
    if (tid == 0) last = (__hip_atomic_fetch_add(a.counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1) ? 1 : 0;
    __syncthreads();
    if (!last) return;

    // ---- the last workgroup: w of this step, and the next reflector from row c0
    double* flat = &red[0][0];
    if (tid == 0) *a.counter = 0;
    const int64_t row = c0;
    const double tau = *a.tau_cur;
    // The first 2048 entries of p, of the row and of the reflector are asked for together and kept; the rest of a longer
    // vector is read when it is needed.
    const double v_row = a.vn[row], p_row = published(a.p + row);
    double pv[4], vv[4], ev[4];
    auto fetch = [&](int64_t i0, bool with_row) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + u * kTriThreads;
            pv[u] = i < k ? published(a.p + i) : 0.0;
            if (with_row) ev[u] = i < k ? published(a.eff + i) : 0.0;
            vv[u] = i < k ? a.vn[i] : 0.0;
        }
    };
    double dot = 0.0;
    for (int64_t i0 = row + tid + 4 * kTriThreads; i0 < k; i0 += 4 * kTriThreads) {
        fetch(i0, false);
#pragma unroll
        for (int u = 0; u < 4; ++u) dot += vv[u] * pv[u];
    }
    fetch(row + tid, true);
#pragma unroll
    for (int u = 0; u < 4; ++u) dot += vv[u] * pv[u];
    dot = block_sum(dot, flat);
    const double kk = 0.5 * tau * tau * dot, w_row = tau * p_row - kk * v_row;
    double n2 = 0.0;
    for (int64_t i0 = row + tid; i0 < k; i0 += 4 * kTriThreads) {
        if (i0 != row + tid) fetch(i0, true);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + u * kTriThreads;
            if (i >= k) continue;
            const double w = tau * pv[u] - kk * vv[u], c = ev[u] - (v_row * w + w_row * vv[u]);
            a.wn[i] = w;
            if (i == row) a.d[row] = c;
            else {
                a.vnext[i] = c;
                if (a.vstore) a.vstore[row * k + i] = c;
                n2 += c * c;
                if (i == row + 1) red[kTriThreads / 64 - 1][kTriRows - 1] = c;      // behind what block_sum uses
            }
        }
    }
    n2 = block_sum(n2, flat);
    if (tid == 0) {
        const double x0 = red[kTriThreads / 64 - 1][kTriRows - 1];
        const double alpha = (x0 > 0.0) ? -sqrt(n2) : sqrt(n2);
        const double v0 = x0 - alpha, vn2 = n2 - x0 * x0 + v0 * v0, tnew = vn2 > 0.0 ? 2.0 / vn2 : 0.0;
        a.vnext[row + 1] = v0;
        *a.tau_next = tnew;
        a.e[row] = alpha;
        if (a.vstore) { a.vstore[row * k + row + 1] = v0; a.taustore[row] = tnew; }
    }
}

// The rest of the chain in one workgroup once at most 256 rows and columns are left, with at most one pair pending.  They are
// numbered so that the last one is 255.  Wavefront w owns the rows w + 16 q and lane l the columns l + 64 t, so that an
// element always belongs to the same thread, and nothing but the reflectors that the caller asked for leaves the
// compute unit: everything behind row and column 63 is in registers, the first 64 rows in LDS (half of their corner in
// registers too; their mirror image is not kept).  By symmetry p_j = sum_i B_ij vn_i: sums over a thread's
// rows without lane exchange, where the entries of vn, v and w that go with a row are LDS broadcasts; of the rows in LDS
// also their product with vn, for the columns of their mirror image.  The first four wavefronts form w and the next
// reflector, a column per lane: a wavefront issues an instruction every 7 cycles or so, and 150 of them with two more
// barriers are less than the 350 that one wavefront with four columns per lane needs (k = 256: 715 -> 665 us).  A step costs
// 1.6 us below 100 rows, 2.1 at 192 and 4.2 at 256; a launch per column is 7.7 us, the chain of k = 256 was 1960 us.
// Kept in B instead of LDS, the first 64 rows and columns made it 970.
constexpr int kTailRows = kAserTridiagTail, kTailWaves = 16, kTailMem = 64;
__global__ __launch_bounds__(64 * kTailWaves) void tridiag_tail_kernel(TridiagStep a) {
    constexpr int Q = kTailRows / kTailWaves, T = kTailRows / 64, Q0 = kTailMem / kTailWaves, T0 = kTailMem / 64;
    constexpr int kLow = kTailRows - kTailMem;
    static_assert(T == 4 && T0 == 1, "sums of four wavefronts, the corner");
    extern __shared__ double low[];                       // [kTailMem][kLow]
    __shared__ double2 vw[kTailRows];
    __shared__ double rowdot[kTailMem], nv[kTailRows], part[kTailWaves][kTailRows], rowbuf[kTailRows], diag[kTailRows], off[kTailRows],
        taus[kTailRows], red[2 * T], entry[2], corner, tau_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t k = a.k;
    if (a.broken && *a.broken != 0) {
        for (int64_t i = tid; i < k; i += 64 * kTailWaves) a.d[i] = a.e[i] = __builtin_nan("");
        return;
    }
    const int first = kTailRows - (int)(k - a.c0);        // 0 .. kTailRows - 2; row i here is row i + base of the matrix
    const int64_t base = a.c0 - first;
    const double* const Bo = a.B + base * k + base;       // entries from `first` on only
    double* const low0 = low + kTailMem * kLow + tid;     // [Q0 / 2][threads]
    double corner0[Q0 / 2], m[Q - Q0][T - T0];
#pragma unroll
    for (int q = Q0; q < Q; ++q)
#pragma unroll
        for (int t = T0; t < T; ++t) {
            const int i = wave + kTailWaves * q, j = lane + 64 * t;
            m[q - Q0][t - T0] = (i >= first && j >= first) ? Bo[i * k + j] : 0.0;
        }
#pragma unroll
    for (int q = 0; q < Q0; ++q) {
        const int i = wave + kTailWaves * q;
        const double x0 = (i >= first && lane >= first) ? Bo[i * k + lane] : 0.0;
        if (q < Q0 / 2) corner0[q] = x0;
        else low0[(q - Q0 / 2) * 64 * kTailWaves] = x0;
        if (i >= first)
#pragma unroll
            for (int t = T0; t < T; ++t) low[i * kLow + lane + 64 * (t - T0)] = Bo[i * k + lane + 64 * t];
    }
    // the loads are over here: without this the compiler waits for all memory before every use of an element
#pragma unroll
    for (int q = 0; q < Q0 / 2; ++q) asm volatile("" : "+v"(corner0[q]));
#pragma unroll
    for (int q = 0; q < Q - Q0; ++q)
#pragma unroll
        for (int t = 0; t < T - T0; ++t) asm volatile("" : "+v"(m[q][t]));
    if (tid < kTailRows) {
        const bool in = tid >= first;
        nv[tid] = in ? a.vn[base + tid] : 0.0;
        vw[tid] = (in && a.v[0]) ? make_double2(a.v[0][base + tid], a.w[0][base + tid]) : make_double2(0.0, 0.0);
        rowbuf[tid] = 0.0;
    }
    if (tid == 0) tau_s = *a.tau_cur;
    __syncthreads();

    for (int c = first;; ++c) {                           // row c: its reflector is nv
        const bool reflect = c + 2 < kTailRows;
        double acc[T - T0];
#pragma unroll
        for (int t = 0; t < T - T0; ++t) acc[t] = 0.0;
        if (c < kTailMem) {
            double acc0 = 0.0;
#pragma unroll
            for (int q = 0; q < Q0; ++q) {
                const int i = wave + kTailWaves * q;
                if (i < c) continue;
                asm volatile("" ::: "memory");            // nothing of another row is read ahead: the registers are full
                const double2 r = vw[i], u0 = vw[lane];
                const double n = nv[i];
                double& x0 = q < Q0 / 2 ? corner0[q] : low0[(q - Q0 / 2) * 64 * kTailWaves];
                const double y0 = x0 - (r.x * u0.y + r.y * u0.x);
                x0 = y0;
                acc0 = fma(y0, n, acc0);
                if (i == c) rowbuf[lane] = y0;
                double dot = 0.0;
#pragma unroll
                for (int t = T0; t < T; ++t) {
                    const int j = lane + 64 * t;
                    double* const at = low + i * kLow + j - kTailMem;
                    const double2 u = vw[j];
                    const double x = *at - (r.x * u.y + r.y * u.x);
                    *at = x;
                    acc[t - T0] = fma(x, n, acc[t - T0]);
                    dot = fma(x, nv[j], dot);
                    if (i == c) rowbuf[j] = x;
                }
                dot = wave_sum(dot);
                if (lane == 0) rowdot[i] = dot;
            }
            part[wave][lane] = acc0;
            asm volatile("" ::: "memory");
        }
        double2 u[T - T0];
#pragma unroll
        for (int t = T0; t < T; ++t) u[t - T0] = vw[lane + 64 * t];
#pragma unroll
        for (int q = Q0; q < Q; ++q) {
            const int i = wave + kTailWaves * q;
            if (i < c) continue;
            const double2 r = vw[i];
            const double n = nv[i];
#pragma unroll
            for (int t = 0; t < T - T0; ++t)
                if (64 * (t + T0) + 63 >= c) {
                    double& x = m[q - Q0][t];
                    x -= r.x * u[t].y + r.y * u[t].x;
                    acc[t] = fma(x, n, acc[t]);
                    if (i == c) rowbuf[lane + 64 * (t + T0)] = x;
                }
        }
        if (!reflect && tid == 64 * kTailWaves - 1) corner = m[Q - Q0 - 1][T - T0 - 1];
#pragma unroll
        for (int t = T0; t < T; ++t) part[wave][lane + 64 * t] = acc[t - T0];
        lds_barrier();
        // column j = tid on the first four wavefronts; the others only keep the barriers
        const bool head = wave < T;
        double vn = 0.0, p = 0.0, tau = 0.0, v_row = 0.0, w = 0.0, x = 0.0;
        if (head) {
            vn = nv[tid];
            tau = tau_s;
            v_row = nv[c];
            double q[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) q[g] = (part[4 * g][tid] + part[4 * g + 1][tid]) + (part[4 * g + 2][tid] + part[4 * g + 3][tid]);
            p = (q[0] + q[1]) + (q[2] + q[3]);
            if (wave == 0) p += rowdot[lane];
            p = tid < c ? 0.0 : p;
            const double dot = wave_sum(p * vn);
            if (lane == 0) red[wave] = dot;
            if (tid == c) entry[0] = p;
        }
        lds_barrier();
        if (head) {
            const double dot = (red[0] + red[1]) + (red[2] + red[3]);
            const double kk = 0.5 * tau * tau * dot, w_row = tau * entry[0] - kk * v_row;
            w = tau * p - kk * vn;
            x = rowbuf[tid] - (v_row * w + w_row * vn);
            if (tid == c) diag[c] = x;
            x = tid <= c ? 0.0 : x;
            if (tid == c + 1) entry[1] = x;
            const double n2 = wave_sum(x * x);
            if (lane == 0) red[T + wave] = n2;
        }
        if (!reflect) {                                   // the last 2 x 2 block: no reflector
            if (tid == kTailRows - 1) {
                off[c] = x;
                diag[c + 1] = corner - 2.0 * vn * w;
            }
            break;
        }
        lds_barrier();
        if (head) {
            const double n2 = (red[T] + red[T + 1]) + (red[T + 2] + red[T + 3]), x0 = entry[1], alpha = (x0 > 0.0) ? -sqrt(n2) : sqrt(n2);
            const double v0 = x0 - alpha, vn2 = n2 - x0 * x0 + v0 * v0, next = tid == c + 1 ? v0 : x;
            vw[tid] = make_double2(vn, w);
            nv[tid] = next;
            if (a.vstore && tid > c) a.vstore[(base + c) * k + base + tid] = next;
            if (tid == 0) {
                tau = vn2 > 0.0 ? 2.0 * rcp_f64(vn2) : 0.0;
                off[c] = alpha;
                taus[c] = tau_s = tau;
            }
        }
        lds_barrier();
    }
    lds_barrier();
    if (tid >= first && tid < kTailRows) {
        a.d[base + tid] = diag[tid];
        if (tid + 1 < kTailRows) a.e[base + tid] = off[tid];
        if (a.vstore && tid + 2 < kTailRows) a.taustore[base + tid] = taus[tid];
    }
}

// Every eigenvalue of the symmetric tridiagonal matrix (d, e) by multisection on Sturm counts (wave_f64.h).
// L lanes share an eigenvalue: they take the counts of L P points that cut its interval into L P + 1 parts, and
// the interval shrinks to the part where the count passes i; `rounds` rounds for 60 halvings.  The terms lie in LDS (in pieces of kSturmLds
// when k is larger).  More points per eigenvalue mean fewer rounds but more chains: one wavefront per SIMD hides nothing, a
// second chain in it costs a third more and shares the terms, and at k = 4096 sixteen lanes of two points are one wavefront per SIMD
// (2570 us with quotients and one point per lane in 15 rounds, 1110 now).  Where the chip is empty anyway a wavefront of 64 points takes an eigenvalue, alone in its workgroup (k = 256: 103 -> 40 us).
// sigma[k - 1 - i] = sqrt(max(lambda_i, 0)).  Where an entry of d or e is not finite every sigma is 0, which has no rank, and every eigenvalue NaN.
constexpr int kSturmLds = 4096;

template <int L, int P, int THREADS>
__global__ __launch_bounds__(THREADS) void tridiag_eigenvalues_kernel(int64_t k, const double* __restrict__ d, const double* __restrict__ e,
                                                                      int rounds, double* __restrict__ sigma, double* __restrict__ lam_desc) {
    extern __shared__ __align__(16) double2 de[];               // (d_l, e_{l-1}^2), scaled and padded to a multiple of kSturmTerms
    __shared__ double red[2][THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t i = (int64_t)blockIdx.x * (THREADS / L) + tid / L;
    const int sub = tid % L;
    // Gershgorin interval; none where an entry is not finite
    double lo = 1e300, hi = -1e300;
    int odd = 0;
    for (int64_t l = tid; l < k; l += THREADS) {
        const double dl = d[l], el = (l + 1 < k) ? fabs(e[l]) : 0.0, ep = (l > 0) ? fabs(e[l - 1]) : 0.0;
        lo = fmin(lo, dl - el - ep);
        hi = fmax(hi, dl + el + ep);
        odd |= !__builtin_isfinite(dl + el + ep);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o, 64));
        hi = fmax(hi, __shfl_xor(hi, o, 64));
    }
    if (lane == 0) { red[0][wave] = lo; red[1][wave] = hi; }
    if (__syncthreads_or(odd)) {
        if (sub == 0 && i < k) {
            sigma[k - 1 - i] = 0.0;
            if (lam_desc) lam_desc[k - 1 - i] = __builtin_nan("");
        }
        return;
    }
#pragma unroll
    for (int g = 0; g < THREADS / 64; ++g) {
        lo = fmin(lo, red[0][g]);
        hi = fmax(hi, red[1][g]);
    }
    const double radius = fmax(fabs(lo), fabs(hi)), scale = sturm_scale(radius);
    lo *= scale;
    hi *= scale;
    const double span = fmax(hi - lo, 1e-300);
    double a = lo - 1e-12 * span, b = hi + 1e-12 * span;
    const bool once = k <= kSturmLds;
    for (int it = 0; it < rounds; ++it) {
        double x[P];
        SturmChain c[P];
#pragma unroll
        for (int u = 0; u < P; ++u) x[u] = a + (b - a) * ((double)(P * sub + u + 1) * (1.0 / (L * P + 1)));
        for (int64_t l0 = 0; l0 < k; l0 += kSturmLds) {
            const int len = (int)((k - l0 < kSturmLds) ? k - l0 : kSturmLds), padded = (len + kSturmTerms - 1) / kSturmTerms * kSturmTerms;
            if (!once || it == 0) {
                __syncthreads();                                // the previous piece has been read
                for (int t = tid; t < padded; t += THREADS) {
                    const int64_t l = l0 + t;
                    de[t] = l < k ? sturm_entry(d[l], l > 0 ? e[l - 1] : 0.0, scale) : sturm_past_end();
                }
                __syncthreads();
            }
            for (int t = 0; t < padded; t += kSturmTerms) sturm_terms(c, de + t, x);
        }
        // the count grows with x: the points with cnt <= i are the first p of the group
        int mine = 0;
#pragma unroll
        for (int u = 0; u < P; ++u) mine += (int64_t)c[u].count <= i ? 1 : 0;
        int p = 0;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const uint64_t have = __builtin_amdgcn_ballot_w64(mine > u) >> (lane / L * L);
            p += __popcll(L == 64 ? have : (have & ((1ull << (L & 63)) - 1)));
        }
        const double na = p > 0 ? a + (b - a) * ((double)p * (1.0 / (L * P + 1))) : a, nb = p < L * P ? a + (b - a) * ((double)(p + 1) * (1.0 / (L * P + 1))) : b;
        a = na;
        b = nb;
    }
    if (sub == 0 && i < k) {
        const double lam = radius > 0.0 ? 0.5 * (a + b) / scale : 0.0;
        sigma[k - 1 - i] = lam > 0.0 ? sqrt(lam) : 0.0;
        if (lam_desc) lam_desc[k - 1 - i] = lam;
    }
}

template <int L, int P, int THREADS>
int launch_eigenvalues(aser_ctx* ctx, int64_t k, const double* d, const double* e, int rounds, double* sigma, double* lam_desc) {
    const size_t lds = (size_t)(k < kSturmLds ? (k + kSturmTerms - 1) / kSturmTerms * kSturmTerms : kSturmLds) * sizeof(double2);
    auto kern = tridiag_eigenvalues_kernel<L, P, THREADS>;
    ASER_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kSturmLds * sizeof(double2))));
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div64(k, THREADS / L)), dim3(THREADS), lds, ctx->stream, k, d, e, rounds, sigma, lam_desc);
    return aser_check_launch(ctx, "tridiag_eigenvalues");
}

int tridiag_eigenvalues(aser_ctx* ctx, int64_t k, const double* d, const double* e, double* sigma, double* lam_desc) {
    // 65^10 and 33^12 are above 2^60
    if (k <= 1024) return launch_eigenvalues<64, 1, 64>(ctx, k, d, e, 10, sigma, lam_desc);
    if (k <= 2048) return launch_eigenvalues<32, 2, 256>(ctx, k, d, e, 10, sigma, lam_desc);
    return launch_eigenvalues<16, 2, 256>(ctx, k, d, e, 12, sigma, lam_desc);
}

// Eq. 9 on a descending spectrum: running sums in index order; r = number of leading indices whose
// cumulative share stays below alpha, at least 1.  out: r, then sum, share(r), share(r + 1) as doubles.
// One wavefront: 64 values are loaded at a time and added one after the other (every lane carries the same sums), so the
// order and the rounding are those of a running sum; the shares are divided out only until the threshold is passed.
__global__ __launch_bounds__(64) void select_rank_kernel(const double* __restrict__ sigma, int64_t k, double alpha, int32_t* __restrict__ r_out,
                                                         double* __restrict__ stats) {
    const int lane = threadIdx.x;
    auto at = [&](double v, int l) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
    };
    double total = 0.0;
    double nv = lane < k ? sigma[lane] : 0.0;
    for (int64_t i0 = 0; i0 < k; i0 += 64) {
        const double v = nv;
        nv = i0 + 64 + lane < k ? sigma[i0 + 64 + lane] : 0.0;
#pragma unroll
        for (int l = 0; l < 64; ++l) total += at(v, l);      // past the end: + 0, which changes nothing
    }
    double cum = 0.0, at_r = 0.0, next = 0.0;
    int64_t r = 0;
    bool open = true;
    for (int64_t i0 = 0; i0 < k && open; i0 += 64) {
        const double v = i0 + lane < k ? sigma[i0 + lane] : 0.0;
        for (int l = 0; l < 64 && i0 + l < k && open; ++l) {
            cum += at(v, l);
            const double share = cum / total;
            if (share < alpha) { r = i0 + l + 1; at_r = share; }
            else { next = share; open = false; }
        }
    }
    if (lane != 0) return;
    if (open) next = 1.0;
    if (r < 1) {                                          // the threshold lies below the first share: rank one
        r = 1;
        at_r = sigma[0] / total;
        next = (k > 1) ? (sigma[0] + sigma[1]) / total : 1.0;
    }
    *r_out = (int32_t)r;
    stats[0] = total;
    stats[1] = at_r;
    stats[2] = next;
}

// Eq. 3 and Eq. 4: exp(-sum p ln p), p = sigma / sum(sigma) + eps.  One workgroup.
__global__ __launch_bounds__(1024) void effective_rank_kernel(const double* __restrict__ sigma, int64_t k, double eps,
                                                              double* __restrict__ out) {
    __shared__ double red[16];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < k; i += 1024) s += sigma[i];
    const double total = block_sum(s, red);
    double h = 0.0;
    for (int64_t i = threadIdx.x; i < k; i += 1024) {
        const double p = sigma[i] / total + eps;
        if (p > 0.0) h -= p * log(p);
    }
    h = block_sum(h, red);
    if (threadIdx.x == 0) *out = exp(h);
}

// B (k x k fp64, full symmetric) = P^T P, cleared first; K split so that the grid fills the device.
template <typename TIN>
int gram_f64(aser_ctx* ctx, const TIN* P, int64_t K, int64_t k, int64_t ldp, double* B) {
    ASER_TRY(aser_fill_bytes(ctx, B, (size_t)k * k * 8));
    const int64_t t64 = ceil_div64(k, 64), tiles = t64 * (t64 + 1) / 2, ksteps = ceil_div64(K, 16);
    int64_t parts = ceil_div64(2048, tiles);
    if (parts > ksteps / 8) parts = ksteps / 8;
    if (parts < 1) parts = 1;
    if (parts > 64) parts = 64;
    hipLaunchKernelGGL(gram_f64_kernel<TIN>, dim3((unsigned)tiles, (unsigned)parts), dim3(256), 0, ctx->stream, P, K, k, ldp, B,
                       (int)parts);
    return aser_check_launch(ctx, "gram_f64");
}

// write: the pending pairs are applied (one to four of them); otherwise zero to three stay pending.
void launch_tridiag_step(aser_ctx* ctx, bool write, int pairs, const TridiagStep& a) {
    const dim3 grid((unsigned)ceil_div64(a.k - a.c0, kTriRows)), block(kTriThreads);
    const bool two = (a.k & 1) == 0;
    switch (write ? pairs : -pairs) {
#define ASER_STEP(np, wr) \
        if (two) hipLaunchKernelGGL((tridiag_step_kernel<np, wr, 2>), grid, block, 0, ctx->stream, a); \
        else hipLaunchKernelGGL((tridiag_step_kernel<np, wr, 1>), grid, block, 0, ctx->stream, a); \
        break
        case 1: ASER_STEP(1, true);
        case 2: ASER_STEP(2, true);
        case 3: ASER_STEP(3, true);
        case 4: ASER_STEP(4, true);
        case 0: ASER_STEP(0, false);
        case -1: ASER_STEP(1, false);
        case -2: ASER_STEP(2, false);
        default: ASER_STEP(3, false);
#undef ASER_STEP
    }
}

// Householder chain on B (overwritten), one launch per column and one for the last 256.
// vec: eight zeroed arrays of k doubles; d = vec[4], e = vec[5] on return, vec[7] and the first ten rows of B are scratch.
// vstore (k x k) / taustore (k), both zeroed by the caller, receive the reflectors when not null.
int tridiagonalize(aser_ctx* ctx, double* B, int64_t k, double* const* vec, double* vstore, double* taustore) {
    // The pairs (v, w) of the last steps: five slots in rows of B that the chain has left behind, and until those exist
    // (kFirst steps) two v and one w in vec, with every pass writing.
    constexpr int64_t kSlots = kTriPairs + 1, kFirst = 2 * kSlots + 2;
    auto v_of = [&](int64_t s) { return s < kFirst ? vec[s & 1] : B + (2 * (s % kSlots)) * k; };
    auto w_of = [&](int64_t s) { return s < kFirst ? vec[2] : B + (2 * (s % kSlots) + 1) * k; };
    double* tau = vec[6];
    TridiagStep a{};
    a.k = k; a.B = B; a.p = vec[3]; a.eff = vec[7]; a.counter = (int*)(tau + 3);
    a.d = vec[4]; a.e = vec[5]; a.vstore = vstore; a.taustore = taustore;
    a.vnext = v_of(0); a.tau_next = tau;
    hipLaunchKernelGGL(tridiag_first_kernel, dim3(1), dim3(kTriThreads), 0, ctx->stream, a);
    ASER_TRY(aser_check_launch(ctx, "tridiag_first"));
    bool tried = false;
    int64_t pending = 0;                                   // steps s - pending .. s - 1 have not been applied to B
    for (int64_t s = 0; s + 2 < k; ++s) {                  // reflector s acts on rows and columns s + 1 ..
        a.c0 = s + 1;
        for (int64_t q = 0; q < pending; ++q) { a.v[q] = v_of(s - pending + q); a.w[q] = w_of(s - pending + q); }
        a.vn = v_of(s); a.wn = w_of(s); a.vnext = v_of(s + 1);
        a.tau_cur = tau + (s & 1); a.tau_next = tau + ((s + 1) & 1);
        // the columns up to the last 256 on the chip, once six rows that the chain has left behind (and that hold no pair) are there for the
        // exchange.  A column costs 2.8 us there against 7.7 (and more) for a launch; kResidentLeast: less than that is not worth two launches
        const int64_t gone = s < kFirst ? 0 : 2 * kSlots;
        if (!tried && k - a.c0 <= kAserResidentMost && k - a.c0 >= kResidentLeast && pending <= 1 && a.c0 >= gone + 6 && ctx->share == 1 && ctx->gate_attempts >= 0) {
            tried = true;
            const AserTridiagResident r{k, a.c0, B, a.vn, pending ? a.v[0] : nullptr, pending ? a.w[0] : nullptr, a.tau_cur,
                                        vec[0], vec[1], vec[2], a.tau_next, a.d, a.e, vstore, taustore, (uint64_t*)(B + gone * k),
                                        ctx->gate_attempts, ctx->exchange_broken};
            bool done = false;
            ASER_TRY(aser_tridiag_resident(ctx, r, &done));
            if (done) {
                s = k - kTailRows - 1;
                a.c0 = s + 1;
                a.vn = vec[0]; a.v[0] = vec[1]; a.w[0] = vec[2];
                a.tau_cur = r.tau_out;
                a.broken = aser_tridiag_broken(r);
                pending = 1;
            }
        }
        if (k - a.c0 <= kTailRows && pending <= 1) {       // what the registers and the LDS of one compute unit hold
            if (pending == 0) a.v[0] = a.w[0] = nullptr;
            constexpr int lds = (kTailMem * (kTailRows - kTailMem) + kTailMem * kTailMem / 2) * 8;
            ASER_HIP(ctx, hipFuncSetAttribute((const void*)tridiag_tail_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            hipLaunchKernelGGL(tridiag_tail_kernel, dim3(1), dim3(64 * kTailWaves), lds, ctx->stream, a);
            return aser_check_launch(ctx, "tridiag_tail");
        }
        // deferring the update pays where the traffic is what a pass costs.  Whole spectra in ms with 1 / 2 / 4 pairs pending at
        // most: k = 1024 10.60 / 10.63 / 11.31, 2048 27.3 / 26.2 / 27.2, 4096 101 / 90 / 88
        const int64_t rest = k - a.c0, most = rest >= 2048 ? kTriPairs : (rest >= 1024 ? 2 : 1);
        const bool write = pending > 0 && (pending >= most || s < kFirst + 1);
        launch_tridiag_step(ctx, write, (int)pending, a);
        if (write) pending = 0;
        ASER_TRY(aser_check_launch(ctx, "tridiag_step"));
        ++pending;
    }
    return ASER_OK;
}

// ---------------------------------------------------------------------------------------------
// Dense fp64 solver for small layers: the rank-r truncated SVD of A = T S from the complete
// eigen-decomposition of the Gram matrix of its shorter side.  Eigenvalues as above (every one, so the
// whitened error is the square root of their tail sum); eigenvectors of the r largest by inverse
// iteration on the tridiagonal matrix, made orthonormal among themselves, and carried back through the
// stored reflectors.  No iteration count, no start block: what the iterative path approximates.

// out[i][j] = sum_{l >= j} T[i][l] S[l][j] in fp64 (S lower triangular); TRANSPOSED: stored as out[j][i].
// 16 x 64 outputs per workgroup, four rows per thread; operands through LDS, the next 32 rows of S on their way while these are multiplied (a
// thread per output that read both operands from memory: 70 us at 256 x 256, this 20).  Sums run over l in ascending order.
template <bool TRANSPOSED>
__global__ __launch_bounds__(256) void ts_f64_kernel(const float* __restrict__ T, int64_t m, int64_t n, int64_t ldt,
                                                     const float* __restrict__ S, int64_t lds, double* __restrict__ out) {
    __shared__ float st[16][32], ss[32][64];
    const int tid = threadIdx.x, tx = tid & 63, ty = tid >> 6;
    const int64_t j = (int64_t)blockIdx.x * 64 + tx, i0 = (int64_t)blockIdx.y * 16;
    float rt[2], rs[8];
    auto load = [&](int64_t l0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t i = i0 + (tid >> 5) + 8 * u, l = l0 + (tid & 31);
            rt[u] = (i < m && l < n) ? T[i * ldt + l] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t l = l0 + ty + 4 * u;
            rs[u] = (l < n && j < n && l >= j) ? S[l * lds + j] : 0.f;
        }
    };
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t l0 = (int64_t)blockIdx.x * 64;                // the entries above the diagonal do not count
    load(l0);
    for (; l0 < n; l0 += 32) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) st[(tid >> 5) + 8 * u][tid & 31] = rt[u];
#pragma unroll
        for (int u = 0; u < 8; ++u) ss[ty + 4 * u][tx] = rs[u];
        __syncthreads();
        if (l0 + 32 < n) load(l0 + 32);
#pragma unroll 8
        for (int l = 0; l < 32; ++l) {
            const double b = (double)ss[l][tx];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = fma((double)st[4 * ty + q][l], b, acc[q]);
        }
    }
    if (j >= n) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t i = i0 + 4 * ty + q;
        if (i >= m) break;
        if (TRANSPOSED) out[j * m + i] = acc[q]; else out[i * n + j] = acc[q];
    }
}

__device__ __forceinline__ uint32_t hash32(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352dU; x ^= x >> 15; x *= 0x846ca68bU; x ^= x >> 16;
    return x;
}

// One step of inverse iteration on the symmetric tridiagonal matrix (d, e): x <- (T - shift I)^-1 x by Gaussian
// elimination with row interchanges (a zero pivot becomes `tiny`), then scaled to unit maximum.  dd (reciprocal pivots), du,
// du2: k doubles each of scratch.  One thread: the recurrence is a chain, and what it reads (eight entries at a time) is asked for
// before it is needed; 64-bit divisions and a load behind every store took three quarters of a microsecond per row.
__device__ __forceinline__ void invit_solve_one(int64_t k, const double* __restrict__ d, const double* __restrict__ e,
                                                double shift, double tiny, double* x, double* dd, double* du, double* du2) {
    double a = d[0] - shift, b = (k > 1) ? e[0] : 0.0, xi = x[0];      // current row: diagonal, super-diagonal, right-hand side
    for (int64_t i0 = 0; i0 + 1 < k; i0 += 8) {
        double sub[8], dn[8], en[8], xn[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = (i0 + u + 1 < k) ? i0 + u : k - 2;
            sub[u] = e[i];
            dn[u] = d[i + 1] - shift;
            en[u] = (i + 2 < k) ? e[i + 1] : 0.0;
            xn[u] = x[i + 1];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = i0 + u;
            if (i + 1 < k) {
                const bool keep = fabs(a) >= fabs(sub[u]);
                if (keep && fabs(a) < tiny) a = tiny;
                const double rp = rcp_f64(keep ? a : sub[u]), mult = (keep ? sub[u] : a) * rp;
                const double top = keep ? b : dn[u], top2 = keep ? 0.0 : en[u], xt = keep ? xi : xn[u];
                dd[i] = rp; du[i] = top; du2[i] = top2; x[i] = xt;
                xi = (keep ? xn[u] : xi) - mult * xt;
                a = (keep ? dn[u] : b) - mult * top;
                b = (keep ? en[u] : 0.0) - mult * top2;
            }
        }
    }
    if (fabs(a) < tiny) a = tiny;
    double x1 = xi * rcp_f64(a), x2 = 0.0, mx = fabs(x1);               // x_{i+1}, x_{i+2}
    x[k - 1] = x1;
    for (int64_t i0 = k - 2; i0 >= 0; i0 -= 8) {
        double rp[8], t1[8], t2[8], xv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = (i0 - u >= 0) ? i0 - u : 0;
            rp[u] = dd[i]; t1[u] = du[i]; t2[u] = du2[i]; xv[u] = x[i];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (i0 - u >= 0) {
                const double v = (xv[u] - t1[u] * x1 - t2[u] * x2) * rp[u];
                x2 = x1;
                x1 = v;
                x[i0 - u] = v;
                mx = fmax(mx, fabs(v));
            }
        }
    }
    const double sc = mx > 0.0 ? 1.0 / mx : 1.0;
#pragma unroll 8
    for (int64_t i = 0; i < k; ++i) x[i] *= sc;
}

// Largest row sum of the tridiagonal matrix (d, e), by a whole wavefront.
__device__ __forceinline__ double tridiag_norm(int64_t k, const double* d, const double* e) {
    double tnorm = 0.0;
    for (int64_t l = threadIdx.x & 63; l < k; l += 64) tnorm = fmax(tnorm, fabs(d[l]) + (l + 1 < k ? fabs(e[l]) : 0.0) + (l > 0 ? fabs(e[l - 1]) : 0.0));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tnorm = fmax(tnorm, __shfl_xor(tnorm, o, 64));
    return tnorm;
}

__device__ __forceinline__ double invit_start_value(int64_t t) {
    return (double)(hash32((uint32_t)t * 0x9E3779B9U + 12345u) >> 8) * (1.0 / 8388608.0) - 1.0;
}

// Eigenvectors of the symmetric tridiagonal matrix (d, e) for the r largest eigenvalues lam[0 .. r),
// as rows of X (r x k), k <= kInvitMost.  Three rounds of: (T - lam_c I) y = x_c for every c, then the vectors are orthonormalised in
// order, in two sweeps after the last solves and in one after the others, which only keep the vectors apart.
//
// The solves: a workgroup per vector, everything in LDS, the recurrences on its first lane.  What bounds them is the number of instructions, one every six
// cycles or so: the matrix is padded to a multiple of 16 rows that nothing couples to the others, so that no row asks where the matrix ends,
// a row's entries are read and written in pairs, sixteen rows ahead, and the triangular factors of the first round are kept (scr: r x 3 k doubles), which saves
// the later ones the elimination with row interchanges.  A multiplier is at most 1 in magnitude, so the top bit of its exponent is free: set where
// the rows were interchanged.  A zero pivot becomes `tiny`.
// All rounds together, before -> now (one workgroup for everything, a vector per thread, and classical Gram-Schmidt with two barriers per vector and pass):
// k = 256, r = 8: 250 -> 108 us; 512, 64: 6740 -> 572; whole reconstructions: 700 x 900, r = 128: 37.9 -> 4.5 ms, 512 x 512, r = 64: 8.6 -> 2.3.  A round of
// solves is 28, 56 and 107 us at k = 256, 512 and 1000 (78, 157 and 304 with bounds tests and selects on every row), a sweep of r = 64 rows 101 us at 512.
constexpr int kInvitMost = 1024, kInvitPad = 16;
constexpr uint64_t kSwapped = 1ull << 62;
__host__ __device__ static inline int invit_rows(int k) { return (k + kInvitPad - 1) / kInvitPad * kInvitPad; }
__host__ __device__ static inline int invit_lds_bytes(int k) { return (invit_rows(k) + 2 * kInvitPad) * 7 * (int)sizeof(double); }
__global__ __launch_bounds__(64) void invit_solve_lds_kernel(int k, const double* __restrict__ dg, const double* __restrict__ eg, const double* __restrict__ lam,
                                                             int round, double* __restrict__ X, double* __restrict__ scr) {
    extern __shared__ __align__(16) double2 mem2[];
    constexpr int C = kInvitPad / 2;                      // rows per buffer
    const int lane = threadIdx.x, c = blockIdx.x, rows = invit_rows(k), room = rows + 2 * kInvitPad;
    double2* const de = mem2;                             // d - lam, e
    double2* const up = de + room;                        // reciprocal pivot, super-diagonal of the triangular factor
    double2* const mu = up + room;                        // multiplier, second super-diagonal
    double* const x = (double*)(mu + room);
    double *Xc = X + (int64_t)c * k, *kept = scr + (int64_t)c * 3 * k;
    const double shift = lam[c], tiny = fmax(tridiag_norm(k, dg, eg) * 2.3e-16, 1e-300);
    for (int i = lane; i < room; i += 64) {
        de[i] = i < k ? make_double2(dg[i] - shift, i + 1 < k ? eg[i] : 0.0) : make_double2(1.0, 0.0);
        x[i] = i >= k ? 0.0 : round == 0 ? invit_start_value((int64_t)c * k + i) : Xc[i];
        if (round != 0) {
            const double m = i < k ? kept[2 * k + i] : 0.0;
            up[i] = i < k ? make_double2(kept[i], kept[k + i]) : make_double2(1.0, 0.0);
            mu[i] = make_double2(m, (__builtin_bit_cast(uint64_t, m) & kSwapped) && i + 2 < k ? eg[i + 1] : 0.0);
        }
    }
    __syncthreads();
    if (lane == 0) {
        if (round == 0) {
            double a = de[0].x, b = de[0].y, sub = b, xi = x[0];       // current row: diagonal, super-diagonal; sub-diagonal below it; right-hand side
            double2 r[2][C];
            double t[2][C];
            auto load = [&](int buf, int i0) {
#pragma unroll
                for (int u = 0; u < C; ++u) { r[buf][u] = de[i0 + u + 1]; t[buf][u] = x[i0 + u + 1]; }
            };
            auto eliminate = [&](int buf, int i0) {
#pragma unroll
                for (int u = 0; u < C; ++u) {
                    const double dn = r[buf][u].x, en = r[buf][u].y, xn = t[buf][u];
                    const bool keep = fabs(a) >= fabs(sub);
                    if (keep && fabs(a) < tiny) a = tiny;
                    const double q = rcp_f64(keep ? a : sub), mult = (keep ? sub : a) * q;
                    const double top = keep ? b : dn, top2 = keep ? 0.0 : en, xt = keep ? xi : xn;
                    up[i0 + u] = make_double2(q, top);
                    mu[i0 + u] = make_double2(__builtin_bit_cast(double, __builtin_bit_cast(uint64_t, mult) | (keep ? 0 : kSwapped)), top2);
                    x[i0 + u] = xt;
                    xi = (keep ? xn : xi) - mult * xt;
                    a = (keep ? dn : b) - mult * top;
                    b = (keep ? en : 0.0) - mult * top2;
                    sub = en;
                }
            };
            load(0, 0);
#pragma unroll 1
            for (int i0 = 0; i0 < rows; i0 += 2 * C) {
                load(1, i0 + C);
                eliminate(0, i0);
                load(0, i0 + 2 * C);
                eliminate(1, i0 + C);
            }
        } else {
            double xi = x[0], m[2][C], t[2][C];
            auto load = [&](int buf, int i0) {
#pragma unroll
                for (int u = 0; u < C; ++u) { m[buf][u] = mu[i0 + u].x; t[buf][u] = x[i0 + u + 1]; }
            };
            auto forward = [&](int buf, int i0) {
#pragma unroll
                for (int u = 0; u < C; ++u) {
                    const uint64_t bits = __builtin_bit_cast(uint64_t, m[buf][u]);
                    const bool keep = !(bits & kSwapped);
                    const double xn = t[buf][u], xt = keep ? xi : xn;
                    x[i0 + u] = xt;
                    xi = (keep ? xn : xi) - __builtin_bit_cast(double, bits & ~kSwapped) * xt;
                }
            };
            load(0, 0);
#pragma unroll 1
            for (int i0 = 0; i0 < rows; i0 += 2 * C) {
                load(1, i0 + C);
                forward(0, i0);
                load(0, i0 + 2 * C);
                forward(1, i0 + C);
            }
        }
        double x1 = 0.0, x2 = 0.0;                        // x_{i+1}, x_{i+2}
        double2 f[2][C];
        double w[2][C], t[2][C];
        auto load = [&](int buf, int i0) {                // rows i0 + C - 1 down to i0
#pragma unroll
            for (int u = 0; u < C; ++u) { f[buf][u] = up[i0 + u]; w[buf][u] = mu[i0 + u].y; t[buf][u] = x[i0 + u]; }
        };
        auto backward = [&](int buf, int i0) {
#pragma unroll
            for (int u = C - 1; u >= 0; --u) {
                const double v = (t[buf][u] - w[buf][u] * x2 - f[buf][u].y * x1) * f[buf][u].x;
                x2 = x1;
                x1 = v;
                x[i0 + u] = v;
            }
        };
        load(0, rows - C);
#pragma unroll 1
        for (int i0 = rows - C; i0 > 0; i0 -= 2 * C) {
            load(1, i0 - C);
            backward(0, i0);
            load(0, i0 >= 2 * C ? i0 - 2 * C : 0);
            backward(1, i0 - C);
        }
    }
    __syncthreads();
    double mx = 0.0;
    for (int i = lane; i < k; i += 64) mx = fmax(mx, fabs(x[i]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    const double sc = mx > 0.0 ? 1.0 / mx : 1.0;
    for (int i = lane; i < k; i += 64) {
        Xc[i] = x[i] * sc;
        if (round == 0) { kept[i] = up[i].x; kept[k + i] = up[i].y; kept[2 * k + i] = mu[i].x; }
    }
}

// The rows of X (r x k, k <= 64 PER) orthonormalised in order by modified Gram-Schmidt, `sweeps` times.  One workgroup; four rows at a time
// become a panel in LDS, a wavefront each, then every wavefront takes its share of the rows behind it through the panel.
template <int PER>
__global__ __launch_bounds__(1024) void invit_orthonormalize_kernel(int k, int r, int sweeps, double* __restrict__ X) {
    constexpr int P = 4, W = 16;
    __shared__ double pan[P][64 * PER];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto load = [&](int j, double (&v)[PER]) {
#pragma unroll
        for (int u = 0; u < PER; ++u) v[u] = lane + 64 * u < k ? X[(int64_t)j * k + lane + 64 * u] : 0.0;
    };
    auto store = [&](int j, const double (&v)[PER]) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (lane + 64 * u < k) X[(int64_t)j * k + lane + 64 * u] = v[u];
    };
    auto project = [&](int i, double (&v)[PER]) {          // v -= (v, panel i) panel i
        double p[PER], s = 0.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            p[u] = pan[i][lane + 64 * u];
            s = fma(v[u], p[u], s);
        }
        s = wave_sum(s);
#pragma unroll
        for (int u = 0; u < PER; ++u) v[u] = fma(-s, p[u], v[u]);
    };
    for (int sweep = 0; sweep < sweeps; ++sweep)
        for (int p0 = 0; p0 < r; p0 += P) {
            const int width = r - p0 < P ? r - p0 : P;
            double v[PER];
            if (wave < width) load(p0 + wave, v);
            for (int i = 0; i < width; ++i) {
                if (wave == i) {
                    double s = 0.0;
#pragma unroll
                    for (int u = 0; u < PER; ++u) s = fma(v[u], v[u], s);
                    const double nrm = sqrt(wave_sum(s)), inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
#pragma unroll
                    for (int u = 0; u < PER; ++u) {
                        v[u] *= inv;
                        pan[i][lane + 64 * u] = v[u];
                    }
                    store(p0 + i, v);
                }
                lds_barrier();
                if (wave > i && wave < width) project(i, v);
            }
            for (int j = p0 + P + wave; j < r; j += W) {
                load(j, v);
                for (int i = 0; i < P; ++i) project(i, v);
                store(j, v);
            }
            __syncthreads();                              // the next panel's rows have been written, this one has been read
        }
}

template <int PER>
int orthonormalize(aser_ctx* ctx, int64_t k, int r, int sweeps, double* X) {
    hipLaunchKernelGGL(invit_orthonormalize_kernel<PER>, dim3(1), dim3(1024), 0, ctx->stream, (int)k, r, sweeps, X);
    return aser_check_launch(ctx, "invit_orthonormalize");
}

// The same for k <= 8 in one launch of one wavefront: the five launches saved are a fifth of such a call, which is bound by its launches.  Lane 8 c + i holds
// entry i of vector c, lane c solves for it.  Whole calls (us, the launches above -> this): 3 x 40, r = 1: 93 -> 74, 8 x 64, r = 8: 106 -> 92.
constexpr int kInvitTiny = 8;
__global__ __launch_bounds__(64) void invit_tiny_kernel(int k, int r, const double* __restrict__ dg, const double* __restrict__ eg, const double* __restrict__ lam,
                                                        double* __restrict__ X) {
    constexpr int K = kInvitTiny;
    __shared__ double d[K], e[K], x[K][K + 1], factor[K][3 * K + 1];
    const int lane = threadIdx.x, c = lane / K, i = lane % K;
    const bool mine = c < r && i < k;
    const auto sum = [](double v) {                       // over the eight lanes of a vector
#pragma unroll
        for (int o = 1; o < K; o <<= 1) v += __shfl_xor(v, o, 64);
        return v;
    };
    if (lane < K) {
        d[lane] = lane < k ? dg[lane] : 0.0;
        e[lane] = lane + 1 < k ? eg[lane] : 0.0;
    }
    const double shift = lane < r ? lam[lane] : 0.0, tiny = fmax(tridiag_norm(k, dg, eg) * 2.3e-16, 1e-300);
    double v = mine ? invit_start_value((int64_t)c * k + i) : 0.0;
    for (int round = 0; round < 3; ++round) {
        x[c][i] = v;
        __syncthreads();
        if (lane < r) invit_solve_one(k, d, e, shift, tiny, x[lane], factor[lane], factor[lane] + K, factor[lane] + 2 * K);
        __syncthreads();
        v = mine ? x[c][i] : 0.0;
        for (int sweep = 0; sweep < (round == 2 ? 2 : 1); ++sweep)
            for (int j = 0; j < r; ++j) {
                const double nrm = sqrt(sum(v * v));
                if (c == j) v *= nrm > 0.0 ? 1.0 / nrm : 0.0;
                const double p = __shfl(v, K * j + i, 64), s = sum(v * p);
                if (c > j) v = fma(-s, p, v);
            }
    }
    if (mine) X[c * k + i] = v;
}

// The same computation for larger problems, one launch per step, because the orthonormalisation is r^2 k work that
// one workgroup takes most of a second for at k = 4096, r = 200: the start vectors, the r solves (one thread each),
// and per vector c and pass the dots against the vectors before it (one workgroup per earlier vector), the
// update (workgroups over the k entries) and, after the second pass, the normalisation (one workgroup).
__global__ void invit_start_kernel(int64_t total, double* __restrict__ X) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x)
        X[t] = invit_start_value(t);
}

__global__ __launch_bounds__(64) void invit_solve_kernel(int64_t k, int r, const double* __restrict__ d,
                                                         const double* __restrict__ e, const double* __restrict__ lam,
                                                         double* __restrict__ X, double* __restrict__ scr) {
    const int c = blockIdx.x * 64 + threadIdx.x;
    const double tiny = fmax(tridiag_norm(k, d, e) * 2.3e-16, 1e-300);
    if (c >= r) return;
    double* dd = scr + (int64_t)c * 3 * k;
    invit_solve_one(k, d, e, lam[c], tiny, X + (int64_t)c * k, dd, dd + k, dd + 2 * k);
}

__global__ __launch_bounds__(256) void invit_dots_kernel(int64_t k, int c, const double* __restrict__ X, double* __restrict__ dots) {
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = blockIdx.x;
    const double* y = X + (int64_t)j * k;
    const double* x = X + (int64_t)c * k;
    double s = 0.0;
    for (int64_t i = tid; i < k; i += 256) s += y[i] * x[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    if (tid == 0) dots[j] = red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(256) void invit_update_kernel(int64_t k, int c, double* __restrict__ X, const double* __restrict__ dots) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= k) return;
    double v = X[(int64_t)c * k + i];
    for (int j = 0; j < c; ++j) v -= dots[j] * X[(int64_t)j * k + i];
    X[(int64_t)c * k + i] = v;
}

__global__ __launch_bounds__(256) void invit_normalize_kernel(int64_t k, int c, double* __restrict__ X) {
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* x = X + (int64_t)c * k;
    double s = 0.0;
    for (int64_t i = tid; i < k; i += 256) s += x[i] * x[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    const double nrm = sqrt(red[0] + red[1] + red[2] + red[3]);
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    for (int64_t i = tid; i < k; i += 256) x[i] *= inv;
}

// x <- H_0 H_1 ... H_{k-3} x for every row x of X (one workgroup per row): eigenvectors of the tridiagonal
// matrix become eigenvectors of the Gram matrix.  H_j = I - tau_j v_j v_j^T, v_j in row j of vstore.
__global__ __launch_bounds__(256) void backtransform_kernel(int64_t k, const double* __restrict__ vstore,
                                                            const double* __restrict__ taustore, double* __restrict__ X) {
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* x = X + (int64_t)blockIdx.x * k;
    for (int64_t j = k - 3; j >= 0; --j) {
        const double* v = vstore + j * k;
        double s = 0.0;
        for (int64_t i = j + 1 + tid; i < k; i += 256) s += v[i] * x[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        __syncthreads();
        if (lane == 0) red[wave] = s;
        __syncthreads();
        const double f = taustore[j] * (red[0] + red[1] + red[2] + red[3]);
        for (int64_t i = j + 1 + tid; i < k; i += 256) x[i] -= f * v[i];
        __syncthreads();
    }
}

// The same for k <= 64 PER: one wavefront per vector with the vector in registers and the next four reflectors on their way, sums by
// lane shifts (k = 256: 194 us with a workgroup per vector and two barriers per reflector).  The loads stand behind no branch, what lies past the row's end
// is dropped at its use: with a test around every load the compiler waits for all of them where the branches meet, and nothing is on
// its way (k = 256: 63 -> 59 us, 512: 240 -> 134, 1000: 551 -> 348).
template <int PER>
__global__ __launch_bounds__(64) void backtransform_wave_kernel(int64_t k, const double* __restrict__ vstore,
                                                                const double* __restrict__ taustore, double* __restrict__ X) {
    constexpr int kAhead = 4;
    if (k < 3) return;                                               // no reflectors
    const int lane = threadIdx.x;
    double* x = X + (int64_t)blockIdx.x * k;
    uint32_t col[PER];
    double xv[PER], v[kAhead][PER], tau[kAhead];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        col[u] = lane + 64 * u < k ? lane + 64 * u : 0;
        xv[u] = x[col[u]];
        if (lane + 64 * u >= k) xv[u] = 0.0;
    }
    auto load = [&](int64_t j, double (&t)[PER], double& tt) {       // entries up to j are zero in the store
        if (j < 0) j = 0;                                            // not used
        const double* const row = vstore + j * k;
#pragma unroll
        for (int u = 0; u < PER; ++u) t[u] = row[col[u]];
        tt = taustore[j];
    };
#pragma unroll
    for (int q = 0; q < kAhead; ++q) load(k - 3 - q, v[q], tau[q]);
    for (int64_t j = k - 3; j >= 0; j -= kAhead) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            if (j - q < 0) break;
            double s[4] = {0.0, 0.0, 0.0, 0.0}, y[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                y[u] = lane + 64 * u < k ? v[q][u] : 0.0;
                s[u & 3] = fma(y[u], xv[u], s[u & 3]);
            }
            const double f = wave_sum((s[0] + s[1]) + (s[2] + s[3])) * tau[q];
            load(j - q - kAhead, v[q], tau[q]);
#pragma unroll
            for (int u = 0; u < PER; ++u) xv[u] = fma(-f, y[u], xv[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (lane + 64 * u < k) x[lane + 64 * u] = xv[u];
}

// Factors from the eigenvectors (rows of X, r x k) and eigenvalues lam (descending) of the Gram matrix.
//   k == m (left singular vectors u_c = X[c]):   L_A[i][c] = u_c[i] sigma_c,        L_B[c][j] = sum_i u_c[i] T[i][j] / sigma_c
//   k == n (right singular vectors v_c = X[c]):  L_A[i][c] = sum_j A[i][j] v_c[j],  L_B[c][j] = sum_i L_A[i][c] T[i][j] / sigma_c^2
// LA64: m x r fp64 scratch.  Two launches: phase 0 writes L_A (and LA64), phase 1 writes L_B, sigma and the error.
__global__ __launch_bounds__(256) void exact_factors_kernel(int phase, int left, int64_t m, int64_t n, int64_t k, int r,
                                                            const double* __restrict__ X, const double* __restrict__ lam,
                                                            const double* __restrict__ A64, const float* __restrict__ A32,
                                                            const float* __restrict__ T,
                                                            int64_t ldt, double* __restrict__ LA64, float* __restrict__ L_A,
                                                            float* __restrict__ L_B, float* __restrict__ sigma,
                                                            double* __restrict__ err2) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (phase == 0) {
        if (t >= m * r) return;
        const int64_t i = t / r;
        const int c = (int)(t % r);
        double v;
        if (left) {
            const double sg = lam[c] > 0.0 ? sqrt(lam[c]) : 0.0;
            v = X[(int64_t)c * k + i] * sg;
        } else {
            v = 0.0;
            if (A32) {
#pragma unroll 8
                for (int64_t j = 0; j < n; ++j) v = fma((double)A32[i * n + j], X[(int64_t)c * k + j], v);
            } else {
#pragma unroll 8
                for (int64_t j = 0; j < n; ++j) v = fma(A64[i * n + j], X[(int64_t)c * k + j], v);
            }
        }
        LA64[t] = v;
        L_A[t] = (float)v;
        return;
    }
    if (t == 0) {
        double tail = lam[0] != lam[0] ? lam[0] : 0.0;     // NaN: all of them are
        for (int64_t i = k - 1; i >= r; --i) tail += lam[i] > 0.0 ? lam[i] : 0.0;    // smallest first
        *err2 = tail;
    }
    if (t < r) sigma[t] = lam[t] > 0.0 ? (float)sqrt(lam[t]) : 0.f;
    if (t >= (int64_t)r * n) return;
    const int c = (int)(t / n);
    const int64_t j = t % n;
    double acc = 0.0;
#pragma unroll 8
    for (int64_t i = 0; i < m; ++i) acc = fma(LA64[i * r + c], (double)T[i * ldt + j], acc);
    L_B[t] = lam[c] > 0.0 ? (float)(acc / lam[c]) : 0.f;     // L_A^T T / sigma^2 in both cases (L_A = u sigma)
}

struct ExactPlan {
    int64_t k;
    bool big;           // a layer beyond the small ones the solver was made for: T S from the MFMA kernel, multi-launch inverse iteration
    size_t off_a, off_b, off_vs, off_vec, off_x, off_scr, off_la, off_tt, off_dots, total;
};

void exact_plan(int64_t m, int64_t n, int r, ExactPlan* p) {
    p->k = m < n ? m : n;
    const size_t kk = align_up((size_t)p->k * p->k * 8, 256), vb = align_up((size_t)p->k * 8, 256);
    size_t off = 0;
    p->off_a = off; off += align_up((size_t)m * n * 8, 256);        // A (m x n) or A^T (n x m), fp64
    p->off_b = off; off += kk;                                      // Gram matrix, then scratch of the chain
    p->off_vs = off; off += kk;                                     // reflectors
    p->off_vec = off; off += 10 * vb;                               // eight chain vectors, tau store, eigenvalues
    p->off_x = off; off += align_up((size_t)r * p->k * 8, 256);
    p->off_scr = off; off += align_up((size_t)r * 3 * p->k * 8, 256);
    p->off_la = off; off += align_up((size_t)m * r * 8, 256);
    p->off_dots = off; off += 2048;                                 // up to 256 dot products
    p->big = m * n > ((int64_t)1 << 20);
    p->off_tt = off; off += p->big ? align_up((size_t)m * n * 4, 256) : 0;    // T^T for the fp32 product (A and A^T share off_a)
    p->total = off;
}

struct SpecPlan {
    int64_t k;
    size_t off_tt, off_a, off_at, off_b, off_vec, total;
};

void spectrum_plan(int64_t m, int64_t n, bool with_s, SpecPlan* p) {
    p->k = m < n ? m : n;
    size_t off = 0;
    const size_t mat = align_up((size_t)m * n * 4, 256);
    p->off_tt = off; off += (with_s || m <= n) ? mat : 0;          // T^T
    p->off_a = off; off += with_s ? mat : 0;                       // A = T S
    p->off_at = off; off += with_s ? mat : 0;                      // A^T
    p->off_b = off; off += align_up((size_t)p->k * p->k * 8, 256);
    p->off_vec = off; off += 8 * align_up((size_t)p->k * 8, 256);  // v (two), w, p, d, e, tau, scratch
    p->total = off;
}

}  // namespace

size_t aser_exact_workspace(int64_t m, int64_t n, int r) {
    ExactPlan p;
    exact_plan(m, n, r, &p);
    return p.total;
}

// The dense fp64 solver on the bound workspace: L_A, L_B, sigma and, in *err2_dev (device), the squared
// whitened error.  Asynchronous.  The caller has checked shapes and the workspace size.
int aser_exact_reconstruct(aser_ctx* ctx, const float* T, int64_t m, int64_t n, int64_t ldt, const float* S, int64_t lds,
                           int r, float* L_A, float* L_B, float* sigma, double* err2_dev) {
    ExactPlan pl;
    exact_plan(m, n, r, &pl);
    char* ws = (char*)ctx->ws;
    const int64_t k = pl.k;
    const bool left = m <= n;
    double* A64 = (double*)(ws + pl.off_a);
    double* B = (double*)(ws + pl.off_b);
    double* vstore = (double*)(ws + pl.off_vs);
    const size_t vb = align_up((size_t)k * 8, 256);
    double* vec[8];
    for (int i = 0; i < 8; ++i) vec[i] = (double*)(ws + pl.off_vec + i * vb);
    double* taustore = (double*)(ws + pl.off_vec + 8 * vb);
    double* lam = (double*)(ws + pl.off_vec + 9 * vb);
    double* X = (double*)(ws + pl.off_x);
    double* scr = (double*)(ws + pl.off_scr);
    double* LA64 = (double*)(ws + pl.off_la);
    const float* A32 = nullptr;                            // m x n, row-major: the fp32 product of large layers
    if (pl.big) {
        // Large layers (a rank beyond the subspace iteration's): T S from the MFMA kernel (about 2^-16 relative per
        // product, as in the iteration and in aser_singular_values), its Gram matrix in fp64 from the widened entries
        float* Tt = (float*)(ws + pl.off_tt);
        float* A = (float*)(ws + pl.off_a);
        float* At = A + (size_t)m * n;
        ASER_TRY(aser_transpose_f32(ctx, T, m, n, ldt, Tt, m));
        GemmArgs g{};
        g.A = Tt; g.lda = m; g.B = S; g.ldb = lds; g.C = A; g.ldc = n; g.Ct = At; g.ldct = m;
        g.M = m; g.N = n; g.K = n; g.alpha = 1.f;
        g.in_type = aser_f32_form(ctx, m * n); g.epi = GEMM_EPI_STORE; g.tiles = GEMM_TILES_ALL; g.krange = GEMM_K_GE_COL;
        g.k_parts = 1;
        g.long_first = 1;
        g.bm = (m > 1024 && n > 1024) ? 256 : 128; g.bn = 128;
        ASER_TRY(aser_gemm_tn(ctx, g));
        A32 = A;
        if (left) ASER_TRY(gram_f64<float>(ctx, At, n, k, m, B));
        else ASER_TRY(gram_f64<float>(ctx, A, m, k, n, B));
    } else {
        // A = T S in fp64; for m <= n stored transposed (n x m), which is the K-major operand of A A^T
        dim3 grid((unsigned)ceil_div64(n, 64), (unsigned)ceil_div64(m, 16));
        if (left) hipLaunchKernelGGL(ts_f64_kernel<true>, grid, dim3(256), 0, ctx->stream, T, m, n, ldt, S, lds, A64);
        else hipLaunchKernelGGL(ts_f64_kernel<false>, grid, dim3(256), 0, ctx->stream, T, m, n, ldt, S, lds, A64);
        ASER_TRY(aser_check_launch(ctx, "ts_f64"));
        ASER_TRY(gram_f64<double>(ctx, A64, left ? n : m, k, k, B));
    }
    ASER_TRY(aser_fill_bytes(ctx, vstore, (size_t)k * k * 8));
    ASER_TRY(aser_fill_bytes(ctx, vec[0], 10 * vb));
    ASER_TRY(tridiagonalize(ctx, B, k, vec, vstore, taustore));
    double* sig64 = vec[7];
    ASER_TRY(tridiag_eigenvalues(ctx, k, vec[4], vec[5], sig64, lam));
    const double* dd = vec[4];
    const double* ee = vec[5];
    if (k <= kInvitTiny) {
        hipLaunchKernelGGL(invit_tiny_kernel, dim3(1), dim3(64), 0, ctx->stream, (int)k, r, dd, ee, (const double*)lam, X);
        ASER_TRY(aser_check_launch(ctx, "invit_tiny"));
    } else if (k <= kInvitMost) {
        for (int round = 0; round < 3; ++round) {
            hipLaunchKernelGGL(invit_solve_lds_kernel, dim3((unsigned)r), dim3(64), (unsigned)invit_lds_bytes((int)k), ctx->stream, (int)k, dd, ee, (const double*)lam,
                               round, X, scr);
            ASER_TRY(aser_check_launch(ctx, "invit_solve"));
            const int sweeps = round == 2 ? 2 : 1;
            ASER_TRY(k <= 256 ? orthonormalize<4>(ctx, k, r, sweeps, X) : k <= 512 ? orthonormalize<8>(ctx, k, r, sweeps, X) : orthonormalize<16>(ctx, k, r, sweeps, X));
        }
    } else {
        double* dots = (double*)(ws + pl.off_dots);
        const int64_t total = (int64_t)r * k;
        hipLaunchKernelGGL(invit_start_kernel, dim3((unsigned)(ceil_div64(total, 256) < 1024 ? ceil_div64(total, 256) : 1024)), dim3(256),
                           0, ctx->stream, total, X);
        for (int round = 0; round < 3; ++round) {
            hipLaunchKernelGGL(invit_solve_kernel, dim3((unsigned)ceil_div64(r, 64)), dim3(64), 0, ctx->stream, k, r, dd, ee,
                               (const double*)lam, X, scr);
            for (int c = 0; c < r; ++c) {
                for (int pass = 0; pass < 2 && c > 0; ++pass) {
                    hipLaunchKernelGGL(invit_dots_kernel, dim3((unsigned)c), dim3(256), 0, ctx->stream, k, c, (const double*)X, dots);
                    hipLaunchKernelGGL(invit_update_kernel, dim3((unsigned)ceil_div64(k, 256)), dim3(256), 0, ctx->stream, k, c, X,
                                       (const double*)dots);
                }
                hipLaunchKernelGGL(invit_normalize_kernel, dim3(1), dim3(256), 0, ctx->stream, k, c, X);
            }
            ASER_TRY(aser_check_launch(ctx, "tridiag_invit (multi-launch)"));
        }
    }
    if (k <= 256)
        hipLaunchKernelGGL(backtransform_wave_kernel<4>, dim3((unsigned)r), dim3(64), 0, ctx->stream, k, (const double*)vstore, (const double*)taustore, X);
    else if (k <= 512)
        hipLaunchKernelGGL(backtransform_wave_kernel<8>, dim3((unsigned)r), dim3(64), 0, ctx->stream, k, (const double*)vstore, (const double*)taustore, X);
    else if (k <= 1024)
        hipLaunchKernelGGL(backtransform_wave_kernel<16>, dim3((unsigned)r), dim3(64), 0, ctx->stream, k, (const double*)vstore, (const double*)taustore, X);
    else
        hipLaunchKernelGGL(backtransform_kernel, dim3((unsigned)r), dim3(256), 0, ctx->stream, k, (const double*)vstore,
                           (const double*)taustore, X);
    ASER_TRY(aser_check_launch(ctx, "backtransform"));
    for (int phase = 0; phase < 2; ++phase) {
        const int64_t total = phase == 0 ? m * (int64_t)r : (int64_t)r * n;
        hipLaunchKernelGGL(exact_factors_kernel, dim3((unsigned)ceil_div64(total, 256)), dim3(256), 0, ctx->stream, phase, left ? 1 : 0,
                           m, n, k, r, (const double*)X, (const double*)lam, (const double*)A64, A32, T, ldt, LA64, L_A, L_B, sigma,
                           err2_dev);
        ASER_TRY(aser_check_launch(ctx, "exact_factors"));
    }
    return ASER_OK;
}

extern "C" size_t aser_spectrum_workspace_bytes(int64_t m, int64_t n, int32_t with_s) {
    if (m <= 0 || n <= 0) return 0;
    SpecPlan p;
    spectrum_plan(m, n, with_s != 0, &p);
    return p.total + kAserWsTail;
}

extern "C" int aser_singular_values(aser_ctx* ctx, const float* T, int64_t m, int64_t n, int64_t ldt,
                                    const float* S, int64_t lds, double* sigma) {
    if (!ctx) return ASER_ERR_INVALID_ARG;
    if (!T || !sigma) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "singular_values: null pointer");
    if (m <= 0 || n <= 0 || ldt < n || (S && lds < n)) ASER_FAIL(ctx, ASER_ERR_SHAPE, "singular_values: bad shape");
    if (((uintptr_t)T & 3) || (S && ((uintptr_t)S & 3)) || ((uintptr_t)sigma & 7))
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "singular_values: misaligned pointer");
    SpecPlan pl;
    spectrum_plan(m, n, S != nullptr, &pl);
    if (pl.k > 16384) ASER_FAIL(ctx, ASER_ERR_SHAPE, "singular_values: min(m, n) > 16384 is not supported");
    if (!ctx->ws || ctx->ws_bytes < pl.total + kAserWsTail)
        ASER_FAIL(ctx, ASER_ERR_WORKSPACE, "singular_values: workspace too small (%zu needed)", pl.total + kAserWsTail);
    ASER_TRY(aser_prepare_device(ctx));
    char* ws = (char*)ctx->ws;
    float* Tt = (float*)(ws + pl.off_tt);
    float* A = (float*)(ws + pl.off_a);
    float* At = (float*)(ws + pl.off_at);
    double* B = (double*)(ws + pl.off_b);
    const size_t vb = align_up((size_t)pl.k * 8, 256);
    double* vec[8];
    for (int i = 0; i < 8; ++i) vec[i] = (double*)(ws + pl.off_vec + i * vb);
    double *d = vec[4], *e = vec[5];
    const int64_t k = pl.k;

    // the K-major operand of the Gram matrix on the shorter side: Z^T for m <= n, Z for m > n
    const float* P;
    int64_t ldp, K;
    if (S) {
        ASER_TRY(aser_transpose_f32(ctx, T, m, n, ldt, Tt, m));
        GemmArgs g{};
        g.A = Tt; g.lda = m; g.B = S; g.ldb = lds; g.C = A; g.ldc = n; g.Ct = At; g.ldct = m;
        g.M = m; g.N = n; g.K = n; g.alpha = 1.f;
        g.in_type = aser_f32_form(ctx, m * n); g.epi = GEMM_EPI_STORE; g.tiles = GEMM_TILES_ALL; g.krange = GEMM_K_GE_COL;
        g.k_parts = 1;
        g.long_first = 1;
        g.bm = (m > 1024 && n > 1024) ? 256 : 128; g.bn = 128;
        ASER_TRY(aser_gemm_tn(ctx, g));
        if (m <= n) { P = At; ldp = m; K = n; } else { P = A; ldp = n; K = m; }
    } else if (m <= n) {
        ASER_TRY(aser_transpose_f32(ctx, T, m, n, ldt, Tt, m));
        P = Tt; ldp = m; K = n;
    } else {
        P = T; ldp = ldt; K = m;
    }
    ASER_TRY(gram_f64(ctx, P, K, k, ldp, B));
    ASER_TRY(aser_fill_bytes(ctx, vec[0], 8 * vb));
    ASER_TRY(tridiagonalize(ctx, B, k, vec, nullptr, nullptr));
    return tridiag_eigenvalues(ctx, k, d, e, sigma, nullptr);
}

extern "C" int aser_select_rank(aser_ctx* ctx, const double* sigma, int64_t k, double alpha, int32_t* r, double* stats) {
    if (!ctx) return ASER_ERR_INVALID_ARG;
    if (!sigma || !r) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "select_rank: null pointer");
    if (k <= 0) ASER_FAIL(ctx, ASER_ERR_SHAPE, "select_rank: k must be positive");
    if (!(alpha > 0.0 && alpha < 1.0)) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "select_rank: alpha must lie in (0, 1)");
    if ((uintptr_t)sigma & 7) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "select_rank: misaligned pointer");
    if (!ctx->ws || ctx->ws_bytes < kAserWsTail) ASER_FAIL(ctx, ASER_ERR_WORKSPACE, "select_rank: workspace too small");
    ASER_TRY(aser_prepare_device(ctx));
    // results go to the workspace tail, behind the two status words (bytes 64 .. 127)
    char* slot = (char*)ctx->ws + ctx->ws_bytes - kAserWsTail + 64;
    int32_t* r_dev = (int32_t*)slot;
    double* st_dev = (double*)(slot + 8);
    hipLaunchKernelGGL(select_rank_kernel, dim3(1), dim3(64), 0, ctx->stream, sigma, k, alpha, r_dev, st_dev);
    ASER_TRY(aser_check_launch(ctx, "select_rank"));
    int32_t h_r = 0;
    double h_st[3] = {0.0, 0.0, 0.0};
    ASER_HIP(ctx, hipMemcpyAsync(&h_r, r_dev, sizeof(int32_t), hipMemcpyDeviceToHost, ctx->stream));
    ASER_HIP(ctx, hipMemcpyAsync(h_st, st_dev, sizeof(h_st), hipMemcpyDeviceToHost, ctx->stream));
    ASER_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (!(h_st[0] > 0.0)) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "select_rank: the singular values do not have a positive sum");
    *r = h_r;
    if (stats) { stats[0] = h_st[0]; stats[1] = h_st[1]; stats[2] = h_st[2]; }
    return ASER_OK;
}

extern "C" int aser_effective_rank(aser_ctx* ctx, const double* sigma, int64_t k, double eps, double* erank) {
    if (!ctx) return ASER_ERR_INVALID_ARG;
    if (!sigma || !erank) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "effective_rank: null pointer");
    if (k <= 0) ASER_FAIL(ctx, ASER_ERR_SHAPE, "effective_rank: k must be positive");
    if (!(eps >= 0.0)) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "effective_rank: eps must be >= 0");
    if ((uintptr_t)sigma & 7) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "effective_rank: misaligned pointer");
    if (!ctx->ws || ctx->ws_bytes < kAserWsTail) ASER_FAIL(ctx, ASER_ERR_WORKSPACE, "effective_rank: workspace too small");
    ASER_TRY(aser_prepare_device(ctx));
    double* out_dev = (double*)((char*)ctx->ws + ctx->ws_bytes - kAserWsTail + 128);   // bytes 128 .. 135 of the tail
    hipLaunchKernelGGL(effective_rank_kernel, dim3(1), dim3(1024), 0, ctx->stream, sigma, k, eps, out_dev);
    ASER_TRY(aser_check_launch(ctx, "effective_rank"));
    double h = 0.0;
    ASER_HIP(ctx, hipMemcpyAsync(&h, out_dev, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
    ASER_HIP(ctx, hipStreamSynchronize(ctx->stream));
    *erank = h;
    return ASER_OK;
}
