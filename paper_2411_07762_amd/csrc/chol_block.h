// Cholesky factor and its inverse for one diagonal block (b <= 128) of the blocked Cholesky of
// the whitening step (Eq. 5) and of the Cholesky-QR steps of the truncated SVD (Eq. 6).
//
// One workgroup of 8 wavefronts, the block in LDS, blocked again into 32-wide sub-blocks k = 0..3.
// All arithmetic is fp32: the products run on the fp32 MFMA instructions.
//
//   1. one wavefront factors the 32 x 32 diagonal sub-block A_kk = R_kk^T R_kk in registers as 16 x 16 MFMA accumulators, four
//      pivots at a time.  Accumulator register e holds rows 4 e + lane / 16 of the tile (rows and columns are loaded in the order that
//      makes it so), i.e. a group of four pivot rows IS one register and so an operand of the K = 4 instruction as it stands.
//      The 4 x 4 pivot block is spread over all lanes beside an identity and factored with one reciprocal square root, one
//      scaling and one multiply-add per later row and pivot (multipliers are broadcast inside 16 lanes); what the identity has become
//      scales the four rows of a tile in one MFMA, and one more subtracts their products from the tile's later rows.
//   2. everyone, a strip of 16 columns per wavefront: the same groups of four rows, two MFMAs each, applied to the row panel
//      R[k, right] = R_kk^-T A[k, right], to the identity (X_kk = R_kk^-1) and to Z^T (the new block column -Z X_kk of the inverse).
//   3. everyone: trailing update A[right, right] -= R[k, right]^T R[k, right] over the upper
//      triangle of 16 x 16 tiles, and Z = X R[., k + 1].
//
// What bounds it is the chain of 128 pivots on one wavefront, 4.3 k cycles per sub-block: 33 cycles a pivot for the dependent steps alone
// (measured: a dependent multiply-add 7, reciprocal square root 8, broadcast and multiply-add 16, an MFMA that feeds the next 42).  The
// fp32 MFMA takes 31 cycles of a SIMD's matrix core, so the strips (20 each, two wavefronts per SIMD) are 1.9 k and the next
// diagonal tiles 0.8 k cycles; load and store 4.4 k and 1.2 k.  Whole kernel at b = 128: 15.8 us (24.9 with a lane read and a multiply-add per
// pivot and row, rows in registers, the explicit inverse applied to the panel and the results stored at the end; whitening of 4096
// columns 1.70 -> 1.41 ms).
//
// A non-positive pivot at column j is reported as atomicMin(info, pivot_base + j + 1); the factor is meaningless from
// there on (NaN).  Rows and columns beyond b are padded with the identity.
#pragma once
#include "aser_internal.h"

namespace {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kN = 128;       // largest block
// LDS pitches: multiples of four for 16-byte accesses; 12 and 36 modulo 64 banks, so that sixteen rows start at the sixteen multiples of
// four and the MFMA operand reads of four consecutive words of each have no conflicts
constexpr int kP = 140;
constexpr int kPZ = 36;
constexpr int kSub = 32;
constexpr int kCholThreads = 512;
constexpr size_t kCholLdsBytes = (size_t)(2 * kN * kP + 96 * kPZ + kN + 20 * 64) * sizeof(float);

// Trailing update of one 16 x 16 tile behind the sub-block at offset o: A[i][c] -= sum_k P[k][i] P[k][c]
// with the row panel P in rows o .. o + 31, tile (ti <= tc) counted from column o + 32.
__device__ __forceinline__ void trailing_tile(float* As, int o, int ti, int tc, int t_i, int t_q) {
    const float* prow = As + o * kP + o + kSub;
    float* out = As + (o + kSub + 16 * ti + 4 * t_q) * kP + o + kSub + 16 * tc + t_i;
    f4v c;
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] = out[e * kP];
    const float* pa = prow + t_q * kP + 16 * ti + t_i;
    const float* pb = prow + t_q * kP + 16 * tc + t_i;
    float a[8], b[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) { a[s] = pa[4 * s * kP]; b[s] = pb[4 * s * kP]; }
    __builtin_amdgcn_sched_barrier(0);
    f4v d = {0.f, 0.f, 0.f, 0.f};                         // two chains of products
#pragma unroll
    for (int s = 0; s < 8; s += 2) {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(-a[s], b[s], c, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(-a[s + 1], b[s + 1], d, 0, 0, 0);
    }
    c += d;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e * kP] = c[e];
}

// The same for 32 x 32 entries, blocks (bi <= bj) counted from column o + 32: four tiles that share their operands (of a diagonal block
// the tile below the diagonal is not needed, and harmless).
__device__ __forceinline__ void trailing_block(float* As, int o, int bi, int bj, int t_i, int t_q) {
    const float* pa = As + (o + t_q) * kP + o + kSub + 32 * bi + t_i;
    const float* pb = As + (o + t_q) * kP + o + kSub + 32 * bj + t_i;
    float* out = As + (o + kSub + 32 * bi + 4 * t_q) * kP + o + kSub + 32 * bj + t_i;
    f4v c[2][2];
    float a[8][2], b[8][2];
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) c[h >> 1][h & 1][e] = out[(16 * (h >> 1) + e) * kP + 16 * (h & 1)];
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int h = 0; h < 2; ++h) { a[s][h] = pa[4 * s * kP + 16 * h]; b[s][h] = pb[4 * s * kP + 16 * h]; }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int h = 0; h < 4; ++h)
            c[h >> 1][h & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(-a[s][h >> 1], b[s][h & 1], c[h >> 1][h & 1], 0, 0, 0);
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) out[(16 * (h >> 1) + e) * kP + 16 * (h & 1)] = c[h >> 1][h & 1][e];
}

// Rows 16 it .. 16 it + 15 of Z = X R[., o .. o + 31]: Z[i][c] = sum_{t >= i} X[i][t] R[t][o + c], t < o.
__device__ __forceinline__ void z_rows(const float* As, const float* Xs, float* Zs, int o, int it, int t_i, int t_q) {
    const float* pa = Xs + (16 * it + t_i) * kP + 16 * it + t_q;
    const float* pb = As + (16 * it + t_q) * kP + o + t_i;
    f4v z[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    float a[2][4], b[2][4][2];
    const int n = o - 16 * it;                            // a multiple of 16
    auto load = [&](int v, int s) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[v][u] = pa[s + 4 * u];
#pragma unroll
            for (int h = 0; h < 2; ++h) b[v][u][h] = pb[(s + 4 * u) * kP + 16 * h];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](int v) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) z[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][u], b[v][u][h], z[h], 0, 0, 0);
    };
    load(0, 0);
    for (int s = 0; s < n; s += 32) {
        if (s + 16 < n) load(1, s + 16);
        mul(0);
        if (s + 16 >= n) break;
        if (s + 32 < n) load(0, s + 32);
        mul(1);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) Zs[(16 * it + 4 * t_q + e) * kPZ + 16 * h + t_i] = z[h][e];
}

// The value of lane L of every row of 16 lanes.
template <int L>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + L, 0xF, 0xF, true));
}

// x: four pivot rows, row k in lanes 16 k .. 16 k + 15, whose pivot columns 0 .. 3 are the lanes E, 4 + E, 8 + E, 12 + E of a row of 16.
// Returns L^-1 of their 4 x 4 block (L lower triangular) as an MFMA A operand: entry (i, k) in lane 16 k + 4 i + (E + 1) % 4, zeros
// elsewhere, so that the product with x has row i in accumulator register (E + 1) % 4 of lanes 16 i .. 16 i + 15.
// *piv: pivot i in lane 4 i + E (before its square root is taken).  fill(0) .. fill(3): independent work of the caller that is
// issued under the chain of dependent steps.
template <int E, class Fill>
__device__ __forceinline__ float pivots4(float x, int lane, float* piv, Fill fill) {
    typedef unsigned u2v __attribute__((ext_vector_type(2)));
    const unsigned u = __float_as_uint(x);
    const u2v pairs = __builtin_amdgcn_permlane16_swap(u, u, false, false);             // rows 0 0 2 2 | 1 1 3 3
    const u2v even = __builtin_amdgcn_permlane32_swap(pairs[0], pairs[0], false, false);
    const u2v odd = __builtin_amdgcn_permlane32_swap(pairs[1], pairs[1], false, false);
    const unsigned all[4] = {even[0], odd[0], even[1], odd[1]};
    const int grp = lane >> 4, q = (lane >> 2) & 3;
    const bool pivot_col = (lane & 3) == E;
    float X[4], Y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) X[i] = pivot_col ? __uint_as_float(all[i]) : (grp == i ? 1.f : 0.f);
    // v_rsq_f32, 1 ulp: as good as the fp32 data it scales
    float rs = __builtin_amdgcn_rsqf(row_bcast<E>(X[0])), m;
    fill(0);
    Y[0] = X[0] * rs;
    m = -Y[0];
    X[1] = fmaf(row_bcast<4 + E>(m), Y[0], X[1]);
    rs = __builtin_amdgcn_rsqf(row_bcast<4 + E>(X[1]));
    X[2] = fmaf(row_bcast<8 + E>(m), Y[0], X[2]);
    X[3] = fmaf(row_bcast<12 + E>(m), Y[0], X[3]);
    fill(1);
    Y[1] = X[1] * rs;
    m = -Y[1];
    X[2] = fmaf(row_bcast<8 + E>(m), Y[1], X[2]);
    rs = __builtin_amdgcn_rsqf(row_bcast<8 + E>(X[2]));
    X[3] = fmaf(row_bcast<12 + E>(m), Y[1], X[3]);
    fill(2);
    Y[2] = X[2] * rs;
    m = -Y[2];
    X[3] = fmaf(row_bcast<12 + E>(m), Y[2], X[3]);
    rs = __builtin_amdgcn_rsqf(row_bcast<12 + E>(X[3]));
    fill(3);
    Y[3] = X[3] * rs;
    *piv = q < 2 ? (q == 0 ? X[0] : X[1]) : (q == 2 ? X[2] : X[3]);
    const float a = q < 2 ? (q == 0 ? Y[0] : Y[1]) : (q == 2 ? Y[2] : Y[3]);
    return (lane & 3) == ((E + 1) & 3) ? a : 0.f;
}

__device__ __forceinline__ f4v mfma4(float a, float b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// What a group of four pivots leaves for the tile beside it, formed under the next group's chain.
struct PivotRest {
    float linv, np, piv;
};

// Pivot group E of the tile P (HALF 0: with Q right of it and C below Q).  Only P's own product is formed at once; that of Q and C for the group
// before it (`r`) is formed under this one's chain.  ops: see pivots32.
template <int E, int HALF>
__device__ __forceinline__ void pivot_group(f4v& P, f4v& Q, f4v& C, PivotRest& r, float* as, float* ops, float* piv_out, int lane) {
    constexpr int R = (E + 1) & 3, PE = (E + 3) & 3, PR = E;       // the group before and its result register
    const f4v zero = {0.f, 0.f, 0.f, 0.f};
    f4v s;
    float q;
    auto fill = [&](int at) {
        if constexpr (E > 0) {
            __builtin_amdgcn_sched_barrier(0);
            if (at == 0) {
                if (HALF == 0) s = mfma4(r.linv, Q[PE], zero);
                ops[(4 * HALF + PE) * 64 + lane] = r.linv;
            } else if (at == 1) {
                if (HALF == 0) {
                    q = s[PR];
                    Q = mfma4(r.np, q, Q);
                }
                ops[(8 + 4 * HALF + PE) * 64 + lane] = r.np;
            } else if (at == 2) {
                if (HALF == 0) {
                    as[4 * PE * kP + 16] = q;
                    q = -q;
                    C = mfma4(q, -q, C);
                }
                as[4 * PE * kP] = -r.np;
            } else {
                if (HALF == 0) ops[(16 + PE) * 64 + lane] = q;
                if ((lane & 3) == PE && lane < 16) piv_out[4 * PE + (lane >> 2)] = r.piv;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const float linv = pivots4<E>(P[E], lane, &r.piv, fill);
    const float p = mfma4(linv, P[E], zero)[R];
    r.linv = linv;
    r.np = -p;
    if (E < 3) P = mfma4(-p, p, P);
}

// What group 3, which has no later rows in its tile, leaves.
template <int HALF>
__device__ __forceinline__ void pivot_last(const f4v& Q, f4v& C, const PivotRest& r, float* as, float* ops, float* piv_out, int lane) {
    const f4v zero = {0.f, 0.f, 0.f, 0.f};
    if (HALF == 0) {
        const float q = mfma4(r.linv, Q[3], zero)[0];
        C = mfma4(-q, q, C);
        as[12 * kP + 16] = q;
        ops[19 * 64 + lane] = -q;
    }
    ops[(4 * HALF + 3) * 64 + lane] = r.linv;
    ops[(8 + 4 * HALF + 3) * 64 + lane] = r.np;
    as[12 * kP] = -r.np;
    if ((lane & 3) == 3 && lane < 16) piv_out[12 + (lane >> 2)] = r.piv;
}

// The 32 x 32 diagonal sub-block at offset o: R (upper) to As, the pivots to piv.  One wavefront.  Register e, lane l of a
// 16 x 16 tile: row 4 e + l / 16, column 4 (l % 4) + l % 16 / 4: the MFMA's row 4 (l / 16) + e and column l % 16 in an order that puts
// four consecutive rows into one register.  ops: what solve_strip needs, as MFMA A operands of 64 words, per group of four rows L^-1 of its 4 x 4
// block (0 .. 7), minus its rows of the diagonal tile (8 .. 15) and of the tile right of it (16 .. 19).
__device__ __forceinline__ void pivots32(float* As, float* ops, float* piv, int o, int lane) {
    const int g = lane >> 4, col = 4 * (lane & 3) + ((lane & 15) >> 2);
    float* as = As + (o + g) * kP + o + col;
    f4v P, Q, C;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        P[e] = as[4 * e * kP];
        Q[e] = as[4 * e * kP + 16];
        C[e] = as[(16 + 4 * e) * kP + 16];
    }
    piv += o;
    PivotRest r;
    pivot_group<0, 0>(P, Q, C, r, as, ops, piv, lane);
    pivot_group<1, 0>(P, Q, C, r, as, ops, piv, lane);
    pivot_group<2, 0>(P, Q, C, r, as, ops, piv, lane);
    pivot_group<3, 0>(P, Q, C, r, as, ops, piv, lane);
    pivot_last<0>(Q, C, r, as, ops, piv, lane);
    as += 16 * kP + 16;
    piv += 16;
    pivot_group<0, 1>(C, Q, C, r, as, ops, piv, lane);
    pivot_group<1, 1>(C, Q, C, r, as, ops, piv, lane);
    pivot_group<2, 1>(C, Q, C, r, as, ops, piv, lane);
    pivot_group<3, 1>(C, Q, C, r, as, ops, piv, lane);
    pivot_last<1>(Q, C, r, as, ops, piv, lane);
}

// L^-1 times a strip of 16 columns of 32 rows (R = L^T the diagonal sub-block, ops as pivots32 left it), one group of four rows after the other.  Entry
// (k, c) is src[k * sk + c * sc], or minus that of the columns from `unit` on of the identity when src is null; sign times the result goes to
// dst[k * dk + c * dc].
__device__ __forceinline__ void solve_strip(const float* ops, const float* src, int sk, int sc, float sign, int unit, float* dst, int dk, int dc,
                                            int lane) {
    const int g = lane >> 4, c = lane & 15;
    const f4v zero = {0.f, 0.f, 0.f, 0.f};
    f4v top, low;
    float linv[8], np[8], nq[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        linv[e] = ops[e * 64 + lane];
        np[e] = ops[(8 + e) * 64 + lane];
        if (e < 4) nq[e] = ops[(16 + e) * 64 + lane];
    }
    if (src) {
        const float* p = src + g * sk + c * sc;
        const int step = 4 * sk;
#pragma unroll
        for (int e = 0; e < 4; ++e) { top[e] = *p; p += step; }
#pragma unroll
        for (int e = 0; e < 4; ++e) { low[e] = *p; p += step; }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            top[e] = (4 * e + g == unit + c) ? -1.f : 0.f;
            low[e] = (16 + 4 * e + g == unit + c) ? -1.f : 0.f;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    dst += g * dk + c * dc;
    const int step = 4 * dk;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = mfma4(linv[e], top[e], zero)[(e + 1) & 3];
        if (e < 3) top = mfma4(np[e], x, top);
        low = mfma4(nq[e], x, low);
        *dst = sign * x;
        dst += step;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = mfma4(linv[4 + e], low[e], zero)[(e + 1) & 3];
        if (e < 3) low = mfma4(np[4 + e], x, low);
        *dst = sign * x;
        dst += step;
    }
}

// Four words of row i from column k (a multiple of four) on, with zeros below the diagonal.
__device__ __forceinline__ void store_upper4(const float* M, float* out, int i, int k) {
    float4 x = *(const float4*)(M + i * kP + k);
    x.x = k < i ? 0.f : x.x;
    x.y = k + 1 < i ? 0.f : x.y;
    x.z = k + 2 < i ? 0.f : x.z;
    x.w = k + 3 < i ? 0.f : x.w;
    *(float4*)out = x;
}

// The upper triangle of the b x b block D on its way to As, padded with the identity: all global loads of a thread are issued before the first
// LDS store; 16-byte loads when the block allows it (vec).
struct BlockLoad {
    static constexpr int kPer = kN * kN / kCholThreads;
    float4 v[kPer / 4];

    __device__ __forceinline__ void load(const float* D, int64_t ld, int b, bool vec) {
        const int tid = threadIdx.x;
        if (vec) {
#pragma unroll
            for (int u = 0; u < kPer / 4; ++u) {
                const int t = tid + u * kCholThreads, i = t >> 5, k = (t & 31) * 4;
                v[u] = make_float4(k == i ? 1.f : 0.f, k + 1 == i ? 1.f : 0.f, k + 2 == i ? 1.f : 0.f, k + 3 == i ? 1.f : 0.f);
                if (k + 3 >= i && k < b && i < b) v[u] = *(const float4*)(D + (int64_t)i * ld + k);
            }
        } else {
#pragma unroll
            for (int u = 0; u < kPer / 4; ++u) {
                const int t = tid + u * kCholThreads, i = t >> 5, k = (t & 31) * 4;
                float w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    w[q] = (k + q == i) ? 1.f : 0.f;
                    if (k + q >= i && k + q < b && i < b) w[q] = D[(int64_t)i * ld + k + q];
                }
                v[u] = make_float4(w[0], w[1], w[2], w[3]);
            }
        }
    }
    __device__ __forceinline__ void store(float* As) const {
        const int tid = threadIdx.x;
#pragma unroll
        for (int u = 0; u < kPer / 4; ++u) {
            const int t = tid + u * kCholThreads, i = t >> 5, k = (t & 31) * 4;
            if (k + 3 >= i) *(float4*)(As + i * kP + k) = v[u];
        }
    }
};

// A block as it stands.  What chol_block_body asks of its source: load brings it to As (Xs is free until the first strips), first and rest finish the
// 32 x 32 sub-block in the corner (wavefront 0) and everything else (the others, under the first pivot chain).
struct PlainBlock {
    const float* D;
    int64_t ld;
    int b;
    __device__ __forceinline__ void load(float* As, float*, bool vec) const {
        BlockLoad l;
        l.load(D, ld, b, vec);
        l.store(As);
    }
    __device__ __forceinline__ void first(float*, const float*) const {}
    __device__ __forceinline__ void rest(float*, const float*, int) const {}
};

// The whole block; sm: kCholLdsBytes of LDS; see aser_chol_block for the other arguments.
template <class Source>
__device__ __forceinline__ void chol_block_body(const Source& source, float* sm, float* D, int64_t ld, int b, float* Rinv, int32_t* info, int32_t pivot_base,
                                                int clear_d, float* beta_out) {
    float* As = sm;                      // working matrix, upper triangle -> R; what stands below the diagonal is never used
    float* Xs = As + kN * kP;            // R^-1, upper 16 x 16 tiles
    float* Zs = Xs + kN * kP;            // 96 x 32 scratch
    float* piv = Zs + 96 * kPZ;          // the pivots
    float* ops = piv + kN;               // operands of the strips, 20 x 64
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nsub = (b + kSub - 1) / kSub;
    // 16 x 16 tile roles of this lane
    const int t_i = lane & 15, t_q = lane >> 4;

    const bool vec = (((uintptr_t)D | (uintptr_t)Rinv) & 15) == 0 && (ld & 3) == 0 && (b & 3) == 0;
    source.load(As, Xs, vec);
    __syncthreads();

    // Round kb factors diagonal sub-block kb (one wavefront), forms its row panel and its block column of the inverse, and
    // updates what lies behind it.  The pivot chain is the long part and keeps a single wavefront busy,
    // so it runs beside the bulk of the previous round's updates: once the three 16 x 16 tiles of the
    // next diagonal sub-block are updated, wavefront 0 starts on it while the others finish the
    // rest of the trailing update, form Z = X R for the next block column X[:, kb] = -Z X_kk of the inverse and store what is finished.
    for (int kb = 0; kb < nsub; ++kb) {
        const int o = kb * kSub;
        const int ncb = nsub - 1 - kb;             // 32-column blocks to the right

        // ---- 1. diagonal sub-block
        if (wave == 0) {
            __builtin_amdgcn_s_setprio(3);           // the chain shares its SIMD with one wavefront of the updates
            if (kb == 0) source.first(As, Xs);
            pivots32(As, ops, piv, o, lane);
            __builtin_amdgcn_s_setprio(0);
        } else {
            const int op = o - kSub;
            if (kb == 0) source.rest(As, Xs, wave);
            if (kb > 0 && (wave & 3) != 0) {             // six wavefronts: the matrix core of the chain's SIMD is left to it
                // One place per routine: a launch starts with a cold instruction cache.  kb = 1: blocks (0, 1) (0, 2) (1, 1) (1, 2) (2, 2) and
                // both strips of Z; 2: (0, 1) (1, 1) and four strips; 3: six strips, long and short ones paired on a SIMD.
                const int w = wave - 1 - (wave >> 2), ntr = ncb == 2 ? 5 : (ncb == 1 ? 2 : 0), nz = o / 16;
                int it = w - ntr, iend = it + 1;
                if (w < ntr) {
                    const int bi = ncb == 1 ? w : (w < 2 ? 0 : (w < 4 ? 1 : 2));
                    trailing_block(As, op, bi, ncb == 1 ? 1 : (w < 2 ? w + 1 : (w < 4 ? w - 1 : 2)), t_i, t_q);
                    iend = it;
                } else if (ncb == 2) {
                    iend = 2;
                } else if (nz == 6) {
                    it = w < 3 ? w : 8 - w;
                    iend = it + 1;
                }
                for (; it < iend && it < nz; ++it) z_rows(As, Xs, Zs, o, it, t_i, t_q);
            }
            if (vec) {
                const int t0 = tid - 64, i0 = t0 >> 3, k0 = (t0 & 7) * 4;
                if (kb == 0) {                               // the zeros: below the diagonal blocks of R^-1, and D if it is to be cleared
                    for (int i = t0 >> 5, k = (t0 & 31) * 4; i < b; i += 14) {
                        if (clear_d && k < b) *(float4*)(D + (int64_t)i * ld + k) = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (k < (i & ~(kSub - 1))) *(float4*)(Rinv + i * b + k) = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                } else {                                     // rows of R and columns of R^-1 of sub-block kb - 1
                    if (!clear_d)
                        for (int i = op + (t0 >> 5), k = op + (t0 & 31) * 4; i < o; i += 14)
                            if (k < b) store_upper4(As, D + (int64_t)i * ld + k, i, k);
                    for (int i = i0; i < o; i += 56) store_upper4(Xs, Rinv + i * b + op + k0, i, op + k0);
                }
            }
        }
        __syncthreads();

        // ---- 2. strips of 16 columns, one per wavefront (with all four sub-blocks there are eight): the panel L^-1 A[o .., right], the diagonal block
        // X_kk = (L^-1 I)^T of the inverse, and its block column X[above, o ..] = -Z X_kk = -(L^-1 Z^T)^T
        {
            const int npan = 2 * ncb, jx = wave - npan;
            const float* src = nullptr;
            float* dst = As + o * kP + o + kSub + 16 * wave;
            int sk = kP, sc = 1, dk = kP, dc = 1, unit = 0;
            if (jx < 0) {
                src = dst;
            } else {
                dk = 1;
                dc = kP;
                unit = 16 * jx;
                dst = Xs + (o + unit) * kP + o;
                if (jx >= 2) {
                    dst = Xs + (unit - kSub) * kP + o;
                    src = Zs + (unit - kSub) * kPZ;
                    sk = 1;
                    sc = kPZ;
                }
            }
            if (jx < 2 + 2 * kb) solve_strip(ops, src, sk, sc, jx < 0 ? 1.f : -1.f, unit, dst, dk, dc, lane);
        }
        __syncthreads();

        // ---- 3. the three tiles of the next diagonal sub-block
        if (ncb > 0) {
            if (wave < 3) trailing_tile(As, o, wave == 2 ? 1 : 0, wave == 0 ? 0 : 1, t_i, t_q);
            __syncthreads();
        }
    }

    if (info && tid < b && !(piv[tid] > 0.f)) atomicMin(info, pivot_base + tid + 1);
    // write out the rest: the last sub-block
    if (vec) {
        const int o = (nsub - 1) * kSub, k = o + (tid & 7) * 4;
        if (k < b) {
            for (int i = tid >> 3; i < b; i += kCholThreads / 8) {
                if (i >= o && !clear_d) store_upper4(As, D + (int64_t)i * ld + k, i, k);
                store_upper4(Xs, Rinv + i * b + k, i, k);
            }
        }
    } else {
        for (int t = tid; t < b * kN; t += kCholThreads) {
            const int i = t >> 7, k = t & 127;
            if (k < b) {
                D[(int64_t)i * ld + k] = (clear_d || k < i) ? 0.f : As[i * kP + k];
                Rinv[i * b + k] = (k >= i) ? Xs[i * kP + k] : 0.f;
            }
        }
    }
    // ---- optional: the momentum coefficient of the subspace iteration, -(0.9 s^2 / 2)^2 with s the smallest
    // diagonal entry of R, and whether the diagonal of R spans more than a factor of 64
    if (beta_out) {
        float smin = 3.0e38f, smax = 0.f;
        if (tid < b) smin = smax = 1.0f / fabsf(Xs[tid * kP + tid]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            smin = fminf(smin, __shfl_xor(smin, o, 64));
            smax = fmaxf(smax, __shfl_xor(smax, o, 64));
        }
        if (lane == 0 && wave < 2) { Zs[wave] = smin; Zs[2 + wave] = smax; }
        __syncthreads();
        if (tid == 0) {
            const float s = fminf(Zs[0], Zs[1]), hbeta = 0.45f * s * s;
            beta_out[0] = -hbeta * hbeta;
            ((int*)beta_out)[1] = (fmaxf(Zs[2], Zs[3]) > 64.f * s) ? 1 : 0;
        }
    }
}

}  // namespace
