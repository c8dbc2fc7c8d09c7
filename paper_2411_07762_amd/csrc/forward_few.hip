// The compensated layer at inference for a few tokens (decoding: one token, a batch of them, a short prompt):
//     Y[t][o] = s_t c_o sum_i xq[t][i] wq[o][i]  +  sum_k P[t][k] L_A[o][k],   P[t][k] = s_t sum_i xq[t][i] L_B[k][i].
//
// What bounds it: reading the weight codes once (4096 x 14336 int4: 29 MB, 5.7 us at the rate of a large copy) and
// the launches.  The tiles of the prefill kernels give such a call m / 256 workgroups that walk the whole
// contraction one after the other, so here a workgroup owns 16, 32 or 64 outputs and up to 128 tokens, and its wavefronts split
// the contraction: every wavefront streams its own part of the code rows from global memory straight into
// MFMA operands (a lane's 16 bytes are 16 int8 or 32 int4 channels of its row; the order of the channels inside a
// step is free as long as both operands agree), nothing goes through LDS on the way.  The int32 partial sums are exact and meet
// in LDS by integer atomics, so the result does not depend on their order.  The rank-r branch is a kernel in front
// (few_down_kernel: P summed over up to 2048 channels per workgroup) and r / 4 further steps (r / 32 with rounded factors) per output tile in the epilogue, or, with many
// outputs, P in workgroups of the same launch as the codes (neither needs the other) and those steps in a second, short launch;
// all on MFMA instructions, operands straight from global memory.  In the mode that rounds the factors
// to bf16 the same three roundings are made (L_B, P, L_A) as in the prefill kernels; the other one is exact in every product with L_B and keeps fp32 behind it.
#include "aser_internal.h"
#include "bf16_pair.h"

namespace {

typedef int v4i_t __attribute__((ext_vector_type(4)));

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kDownChunk = 2048;      // channels per partial P
constexpr int kDownSum = 256;         // channels per sum inside one
constexpr int kDownSums = kDownChunk / kDownSum;

struct FewArgs {
    const int8_t* xq; const float* xs; int rows; int64_t n;
    const void* wq; const float* ws; int64_t m;
    float* part; int chunks; const float* L_A; const float* L_B; int r, rp, split, vec_a, vec_b;
    int down, tiles;                      // workgroups that form P; output tiles
    float* Y; int64_t ldy;
};

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float below_upper_half(float x) { return x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); }
__device__ __forceinline__ bf16x8_t operand(const uint32_t (&p)[4]) { return __builtin_bit_cast(bf16x8_t, make_uint4(p[0], p[1], p[2], p[3])); }

// The products of eight channels of L_B (b) and of the codes (x) added to acc, v_mfma_f32_16x16x32_bf16.  Codes are bf16 values.  The mode that rounds the factors
// takes b to the nearest bf16; otherwise b is the sum of three bf16 values, each the upper half of what the ones before it leave of its 24 bits, so
// the products are exact either way.  (Of an infinity nothing is left.)  The second is multiplied by 2^7 and the third by 2^15, to the size of the first at
// most, and summed apart: as they are, the bits of a b below 1e-34 would fall under the smallest bf16 value.
struct DownSums { f4v hi = {0.f, 0.f, 0.f, 0.f}, mid = hi, lo = hi; };
__device__ __forceinline__ void down_step(bool split, float4 b0, float4 b1, uint2 x, DownSums& acc) {
    const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    uint32_t c[4], hi[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t w = q < 2 ? x.x : x.y;
        const int s = 16 * (q & 1);
        c[q] = upper_halves((float)(int)(int8_t)(w >> s), (float)(int)(int8_t)(w >> (s + 8)));
    }
    const bf16x8_t codes = operand(c);
    if (!split) {
#pragma unroll
        for (int q = 0; q < 4; ++q) hi[q] = bf16_pair(b[2 * q], b[2 * q + 1]);
        acc.hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(operand(hi), codes, acc.hi, 0, 0, 0);
        return;
    }
    uint32_t mid[4], lo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float m[2], l[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            m[u] = __builtin_isinf(b[2 * q + u]) ? 0.f : below_upper_half(b[2 * q + u]) * 0x1p7f;
            l[u] = below_upper_half(m[u]) * 0x1p8f;
        }
        hi[q] = upper_halves(b[2 * q], b[2 * q + 1]);
        mid[q] = upper_halves(m[0], m[1]);
        lo[q] = upper_halves(l[0], l[1]);
    }
    acc.lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(operand(lo), codes, acc.lo, 0, 0, 0);
    acc.mid = __builtin_amdgcn_mfma_f32_16x16x32_bf16(operand(mid), codes, acc.mid, 0, 0, 0);
    acc.hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(operand(hi), codes, acc.hi, 0, 0, 0);
}

// part[chunk][t][k] = sum over 2048 channels of xq[t][i] L_B[k][i] (without s_t), k up to rp (r rounded up to 16; what stands
// behind r is not read).  A workgroup takes 16 rows of L_B and 16 tokens, a wavefront 2048 / NW channels of them, in fp32 sums of 256 channels
// each, so that P does not depend on NW; lane (l % 16, g = l / 16)
// feeds channels 32 s + 8 g .. + 7 of its row and of its token.  All loads of a round are in flight at once: they are unconditional (addresses clamped into the
// operands), because a load behind a branch is waited for where the branches meet.
// What bounds it: latency, of the launch, of two rounds of loads and of the chain of sums.  One K = 4 fp32 instruction per four channels, each value
// converted and masked by itself, was 3200 cycles per wavefront (us for the whole call; 4096 x 4096 int4, r = 64, 16 tokens: 16.6 -> 14.8; split
// factors, 8192 x 8192, 16 tokens: 27.1 -> 25.6, 3.3e-7 -> 1.8e-7 off the fp64 result; 4096 x 11008 int8, 19 tokens: 29.6 -> 28.1; one token: no faster, no slower).
template <int NW>
__device__ __forceinline__ void few_down(const FewArgs& g, int task, float (*red)[16][17]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int kt = g.rp / 16, chunk = task % g.chunks, ky = (task / g.chunks) % kt, tz = task / (g.chunks * kt);
    const int k = ky * 16 + li, t = tz * 16 + li;
    const float* bp = g.L_B + (int64_t)(k < g.r ? k : 0) * g.n + 8 * lg;
    const int8_t* xp = g.xq + (int64_t)(t < g.rows ? t : 0) * g.n + 8 * lg;
    constexpr int NS = 4;                                 // steps of 32 channels in flight; eight are up to 0.8 us slower
#pragma unroll 1
    for (int w = wave * (kDownSums / NW); w < (wave + 1) * (kDownSums / NW); ++w) {
        DownSums acc;
#pragma unroll 1
        for (int h = 0; h < kDownSum; h += 32 * NS) {
            const int64_t c0 = (int64_t)chunk * kDownChunk + w * kDownSum + h;
            if (c0 >= g.n) break;
            float4 b[NS][2];
            uint2 x[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {                // n % 32 == 0: a step is whole or absent
                const int64_t c = c0 + 32 * s < g.n ? c0 + 32 * s : 0;
                if (g.vec_b) {
                    b[s][0] = *(const float4*)(bp + c);
                    b[s][1] = *(const float4*)(bp + c + 4);
                } else {
                    const float* q = bp + c;
                    b[s][0] = make_float4(q[0], q[1], q[2], q[3]);
                    b[s][1] = make_float4(q[4], q[5], q[6], q[7]);
                }
                x[s] = *(const uint2*)(xp + c);
            }
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (c0 + 32 * s < g.n) down_step(g.split, b[s][0], b[s][1], x[s], acc);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) red[w][li][4 * lg + e] = fmaf(acc.lo[e], 0x1p-15f, fmaf(acc.mid[e], 0x1p-7f, acc.hi[e]));     // (token li, row 4 lg + e)
    }
    __syncthreads();
    if (tid < 256) {
        const int tt = tid >> 4, kk = tid & 15;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kDownSums; ++w) s += red[w][tt][kk];
        if (tz * 16 + tt < g.rows) g.part[((int64_t)chunk * g.rows + tz * 16 + tt) * g.rp + ky * 16 + kk] = s;
    }
}

__global__ __launch_bounds__(512) void few_down_kernel(FewArgs g) {
    __shared__ float red[kDownSums][16][17];
    few_down<8>(g, blockIdx.x, red);
}

// y (outputs O .. O + 15 of 16 tokens, this lane's four outputs of token t) += s_t P L_A^T, on the fp32 MFMA instruction, or, with rounded factors, the
// bf16 one, whose products are exact too and of which two take the place of sixteen at r = 64 (us for the whole call; 4096 x 4096 int4, r = 64, 16 tokens: 14.8 -> 14.4;
// 14336 x 4096, 64 tokens: 41.3 -> 40.0; 4096 x 4096, 200 tokens: 41.1 -> 40.2).
__device__ __forceinline__ f4v few_rank(const FewArgs& g, f4v y, int64_t O, int t, bool tok, float sx, int li, int lg) {
    const int64_t orow = O + li;                             // the row of L_A that this lane feeds
    const float* ap = g.L_A + (orow < g.m ? orow : 0) * g.r;
    const float* pp = g.part + (int64_t)(tok ? t : 0) * g.rp;
    for (int k0 = 0; k0 < g.rp; k0 += 64) {              // two steps of 32 at a time, eight k per lane in each: their loads are in flight together
        float av[4][4];
        float4 pv[4];
        auto col = [&](int q) { return k0 + 32 * (q >> 1) + 8 * lg + 4 * (q & 1); };
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = col(q);
            pv[q] = *(const float4*)(pp + (k < g.rp ? k : 0));
            if (g.vec_a) {
                const float4 v = *(const float4*)(ap + (k < g.r ? k : 0));
                av[q][0] = v.x; av[q][1] = v.y; av[q][2] = v.z; av[q][3] = v.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) av[q][e] = ap[k + e < g.r ? k + e : 0];
            }
        }
#pragma unroll 2
        for (int c = 1; c < g.chunks; ++c) {
            const float* pc = pp + (int64_t)c * g.rows * g.rp;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = col(q);
                const float4 v = *(const float4*)(pc + (k < g.rp ? k : 0));
                pv[q].x += v.x; pv[q].y += v.y; pv[q].z += v.z; pv[q].w += v.w;
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (k0 + 32 * s >= g.rp) break;
            float a[8], p[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int k = col(2 * s + (q >> 2)) + (q & 3);
                const float4 v = pv[2 * s + (q >> 2)];
                const float x[4] = {v.x, v.y, v.z, v.w};
                a[q] = (k < g.r && orow < g.m) ? av[2 * s + (q >> 2)][q & 3] : 0.f;
                p[q] = k < g.r ? x[q & 3] * sx : 0.f;                   // sx is 0 past the last token
            }
            if (g.split) {
#pragma unroll
                for (int q = 0; q < 8; ++q) y = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], p[q], y, 0, 0, 0);
            } else {
                uint32_t ab[4], pb[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    ab[q] = bf16_pair(a[2 * q], a[2 * q + 1]);
                    pb[q] = bf16_pair(p[2 * q], p[2 * q + 1]);
                }
                y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(operand(ab), operand(pb), y, 0, 0, 0);
            }
        }
    }
    return y;
}

// OT: 16-output tiles per workgroup, TG: 16-token tiles, NW: wavefronts that split the contraction.
// v_mfma_i32_16x16x64_i8: a lane feeds 16 bytes of row (output, token) lane % 16, and holds the sums of outputs
// 4 (lane / 16) .. + 3 for token lane % 16.
// BESIDE: the first workgroups form P, and L_A P is left to few_rank_kernel; otherwise P is there already.
template <bool W4, int OT, int TG, int NW, bool BESIDE>
__global__ __launch_bounds__(64 * NW) void few_main_kernel(FewArgs g) {
    constexpr int OUT = 16 * OT, TOK = 16 * TG, NT = 64 * NW;
    constexpr int STEP = W4 ? 128 : 64;                     // channels per step: 16 bytes of codes per lane
    constexpr int U = (TG >= 4) ? 2 : 4;                    // steps in flight
    constexpr int OP = OUT + 4;
    constexpr int kRed = (!BESIDE || TOK * OP > kDownSums * 16 * 17) ? TOK * OP : kDownSums * 16 * 17;
    __shared__ int red[kRed];
    if (BESIDE && (int)blockIdx.x < g.down) {
        few_down<NW>(g, blockIdx.x, (float(*)[16][17])red);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int work = (int)blockIdx.x - (BESIDE ? g.down : 0);
    const int64_t O0 = (int64_t)(work % g.tiles) * OUT;
    const int T0 = work / g.tiles * TOK;
    const int64_t steps = (g.n + STEP - 1) / STEP, per = (steps + NW - 1) / NW;
    const int64_t s0 = wave * per, s1 = (s0 + per < steps) ? s0 + per : steps;

    const char* wp[OT];
#pragma unroll
    for (int i = 0; i < OT; ++i) {
        int64_t o = O0 + 16 * i + li;
        if (o >= g.m) o = g.m - 1;                          // rows past the end repeat the last one; their sums are not stored
        wp[i] = (const char*)g.wq + o * (W4 ? g.n / 2 : g.n) + 16 * lg;
    }
    const char* xp[TG];
    bool xok[TG];
#pragma unroll
    for (int j = 0; j < TG; ++j) {
        const int t = T0 + 16 * j + li;
        xok[j] = t < g.rows;
        xp[j] = (const char*)g.xq + (int64_t)(xok[j] ? t : 0) * g.n + (W4 ? 32 : 16) * lg;
    }
    v4i_t acc[OT][TG];
#pragma unroll
    for (int i = 0; i < OT; ++i)
#pragma unroll
        for (int j = 0; j < TG; ++j) acc[i][j] = v4i_t{0, 0, 0, 0};

    v4i_t wv[U][OT], xv[U][TG][W4 ? 2 : 1];
    auto load = [&](int64_t s, int u) {
        const int64_t k = s * STEP;
        const bool in = s < s1 && k + (W4 ? 32 : 16) * lg < g.n;      // n % 32 == 0: a lane's chunk is whole or absent
#pragma unroll
        for (int i = 0; i < OT; ++i) {
            wv[u][i] = v4i_t{0, 0, 0, 0};
            if (in) wv[u][i] = __builtin_nontemporal_load((const v4i_t*)(wp[i] + (W4 ? k / 2 : k)));
        }
#pragma unroll
        for (int j = 0; j < TG; ++j) {
#pragma unroll
            for (int h = 0; h < (W4 ? 2 : 1); ++h) {
                xv[u][j][h] = v4i_t{0, 0, 0, 0};
                if (in && xok[j]) xv[u][j][h] = *(const v4i_t*)(xp[j] + k + 16 * h);
            }
        }
    };
    auto multiply = [&](int u) {
        if (W4) {
            // a lane's 32 channels as (even ones, odd ones); the codes become 16 q as signed bytes, and the factor 16
            // goes into the scale
            v4i_t xe[TG], xo[TG];
#pragma unroll
            for (int j = 0; j < TG; ++j) {
                const v4i_t a = xv[u][j][0], b = xv[u][j][W4 ? 1 : 0];
                xe[j] = v4i_t{(int)__builtin_amdgcn_perm((uint32_t)a.y, (uint32_t)a.x, 0x06040200u), (int)__builtin_amdgcn_perm((uint32_t)a.w, (uint32_t)a.z, 0x06040200u),
                              (int)__builtin_amdgcn_perm((uint32_t)b.y, (uint32_t)b.x, 0x06040200u), (int)__builtin_amdgcn_perm((uint32_t)b.w, (uint32_t)b.z, 0x06040200u)};
                xo[j] = v4i_t{(int)__builtin_amdgcn_perm((uint32_t)a.y, (uint32_t)a.x, 0x07050301u), (int)__builtin_amdgcn_perm((uint32_t)a.w, (uint32_t)a.z, 0x07050301u),
                              (int)__builtin_amdgcn_perm((uint32_t)b.y, (uint32_t)b.x, 0x07050301u), (int)__builtin_amdgcn_perm((uint32_t)b.w, (uint32_t)b.z, 0x07050301u)};
            }
#pragma unroll
            for (int i = 0; i < OT; ++i) {
                const v4i_t w = wv[u][i];
                const v4i_t we = {(int)(((uint32_t)w.x << 4) & 0xF0F0F0F0u), (int)(((uint32_t)w.y << 4) & 0xF0F0F0F0u),
                                  (int)(((uint32_t)w.z << 4) & 0xF0F0F0F0u), (int)(((uint32_t)w.w << 4) & 0xF0F0F0F0u)};
                const v4i_t wo = {(int)((uint32_t)w.x & 0xF0F0F0F0u), (int)((uint32_t)w.y & 0xF0F0F0F0u),
                                  (int)((uint32_t)w.z & 0xF0F0F0F0u), (int)((uint32_t)w.w & 0xF0F0F0F0u)};
#pragma unroll
                for (int j = 0; j < TG; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(we, xe[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wo, xo[j], acc[i][j], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < OT; ++i)
#pragma unroll
                for (int j = 0; j < TG; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv[u][i], xv[u][j][0], acc[i][j], 0, 0, 0);
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load(s0 + u, u);

    for (int q = tid; q < TOK * OP; q += NT) red[q] = 0;
    __syncthreads();
    for (int64_t s = s0; s < s1; s += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            multiply(u);                                    // steps past s1 were loaded as zeros
            load(s + U + u, u);
        }
    }
#pragma unroll
    for (int i = 0; i < OT; ++i)
#pragma unroll
        for (int j = 0; j < TG; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(red + (16 * j + li) * OP + 16 * i + 4 * lg + e, acc[i][j][e]);
    __syncthreads();

    // a wavefront takes 16 x 16 tiles in turn: the scaled integer sums, then L_A P^T on top of them in the same layout
    const float wfix = W4 ? (1.0f / 16.0f) : 1.0f;
    for (int tile = wave; tile < OT * TG; tile += NW) {
        const int i = tile % OT, j = tile / OT;
        const int t = T0 + 16 * j + li;
        if (T0 + 16 * j >= g.rows) continue;
        const bool tok = t < g.rows;
        const float sx = tok ? g.xs[t] : 0.f;
        const int64_t o4 = O0 + 16 * i + 4 * lg;             // this lane's four outputs
        f4v y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (float)red[(16 * j + li) * OP + 16 * i + 4 * lg + e] * (sx * (o4 + e < g.m ? g.ws[o4 + e] * wfix : 0.f));
        if (!BESIDE) y = few_rank(g, y, O0 + 16 * i, t, tok, sx, li, lg);
        if (!tok) continue;
        float* yr = g.Y + (int64_t)t * g.ldy + o4;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (o4 + e < g.m) yr[e] = y[e];
    }
}

// The second launch where P was formed beside the codes: a 16 x 16 tile per wavefront, 64 outputs of 16 tokens per workgroup.
__global__ __launch_bounds__(256) void few_rank_kernel(FewArgs g) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    const int64_t O = (int64_t)blockIdx.x * 64 + 16 * wave, o4 = O + 4 * lg;
    if (O >= g.m) return;
    const int t = blockIdx.y * 16 + li;
    const bool tok = t < g.rows;
    float* yr = g.Y + (int64_t)(tok ? t : 0) * g.ldy;
    f4v y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = yr[o4 + e < g.m ? o4 + e : g.m - 1];
    y = few_rank(g, y, O, t, tok, tok ? g.xs[t] : 0.f, li, lg);
    if (!tok) return;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (o4 + e < g.m) yr[o4 + e] = y[e];
}

template <bool W4, int OT, int TG, int NW>
int launch_few(aser_ctx* ctx, FewArgs g) {
    g.tiles = (int)ceil_div64(g.m, 16 * OT);
    const int64_t work = g.tiles * ceil_div64(g.rows, 16 * TG);
    // P beside the codes: where the output tiles are small workgroups, one or two per compute unit, and long enough to hide P.  Measured (us, P in front
    // -> beside; channels, outputs, one token / 16 tokens, r = 64, int4): 1536, 14336: 12.9 -> 11.0 / 14.8 -> 13.7; 2048, 8224: 13.6 -> 12.1 / 16.2 -> 14.9; 4096, 10240:
    // 17.0 -> 14.8 / 21.3 -> 19.0; 4096, 14336: 17.0 -> 14.7 / 21.5 -> 19.1; 14336, 8224: 31.3 -> 28.1 / 43.7 -> 38.8; int8, 4096, 14336: 22.4 -> 19.0 / 28.1 -> 24.4;
    // r = 1: 12.6 -> 11.4 / 16.7 -> 15.4.  Either way at 1024 channels (14336 outputs: 11.0 -> 9.8 / 12.7 -> 13.6, split factors 11.4 -> 11.5 / 14.0 -> 13.3) and not at 512
    // (split factors 10.5 -> 11.0 / 11.4 -> 12.4).  From 1536 channels on beside was the faster one in 160 such calls (r 1 to 128).  Not with eight wavefronts
    // per tile or 64 outputs: with P on the fp32 MFMA instruction, up to 2 us longer in front and 1 us beside, 8192, 8192: 17.8 -> 19.2 / 27.0 -> 28.4; 4096, 4096:
    // 12.0 -> 13.8 / 16.5 -> 19.1; 8192, 16384: 25.5 -> 24.9 / 33.9 -> 34.1.
    if constexpr (TG == 1 && NW == 4 && OT == 2) {
        if (g.r > 0 && g.n >= 1536) {
            hipLaunchKernelGGL((few_main_kernel<W4, OT, TG, NW, true>), dim3((unsigned)(g.down + work)), dim3(64 * NW), 0, ctx->stream, g);
            ASER_TRY(aser_check_launch(ctx, "compensated_forward_few"));
            hipLaunchKernelGGL(few_rank_kernel, dim3((unsigned)ceil_div64(g.m, 64), (unsigned)ceil_div64(g.rows, 16)), dim3(256), 0, ctx->stream, g);
            return aser_check_launch(ctx, "compensated_forward_few_rank");
        }
    }
    if (g.r > 0) {
        hipLaunchKernelGGL(few_down_kernel, dim3((unsigned)g.down), dim3(512), 0, ctx->stream, g);
        ASER_TRY(aser_check_launch(ctx, "compensated_forward_few_down"));
    }
    hipLaunchKernelGGL((few_main_kernel<W4, OT, TG, NW, false>), dim3((unsigned)work), dim3(64 * NW), 0, ctx->stream, g);
    return aser_check_launch(ctx, "compensated_forward_few");
}

// Outputs per workgroup: the fewest with which the launch still is one workgroup per compute unit (two for up to 16
// tokens, where the code stream is all there is).  Fewer outputs mean more wavefronts on the code stream, more outputs
// mean fewer passes over the tokens.  Measured without factors (us for 16 / 32 / 64 outputs per workgroup):
// 4096 x 4096 int4, 64 tokens 12.3 / 13.8 / 20.3, 256 tokens 38.8 / 23.5 / 33.4, 512 tokens 74.5 / 45.4 / 34.9;
// 14336 x 4096 int4, 1 token 10.2 / 9.8 / 11.8, 32 tokens 23.6 / 16.3 / 15.5; 4096 x 11008 int8, 1 token 13.1 / 19.0 / 37.2.
template <bool W4, int TG>
int pick_outputs(aser_ctx* ctx, const FewArgs& g) {
    const int64_t groups = ceil_div64(g.rows, 16 * TG), most = TG == 1 ? 512 : 256;
    if (ceil_div64(g.m, 16) * groups <= most) return launch_few<W4, 1, TG, 8>(ctx, g);
    if (ceil_div64(g.m, 32) * groups <= most)
        return TG == 1 ? launch_few<W4, 2, TG, 4>(ctx, g) : launch_few<W4, 2, TG, 8>(ctx, g);
    return launch_few<W4, 4, TG, 4>(ctx, g);
}

template <bool W4>
int dispatch_few(aser_ctx* ctx, const FewArgs& g) {
    const int tg = (g.rows + 15) / 16;
    if (tg <= 1) return pick_outputs<W4, 1>(ctx, g);
    if (tg <= 2) return pick_outputs<W4, 2>(ctx, g);
    if (tg <= 4) return pick_outputs<W4, 4>(ctx, g);
    return pick_outputs<W4, 8>(ctx, g);
}

}  // namespace

// scratch: room for ceil(n / 2048) * rows * (r rounded up to 16) floats when r > 0.
int aser_forward_few(aser_ctx* ctx, const int8_t* xq, const float* xs, int rows, int64_t n, const void* wq, bool w4, const float* ws,
                     int64_t m, const float* L_A, const float* L_B, int r, bool split, float* scratch, float* Y, int64_t ldy) {
    FewArgs g{};
    g.xq = xq; g.xs = xs; g.rows = rows; g.n = n; g.wq = wq; g.ws = ws; g.m = m;
    g.L_A = L_A; g.r = r; g.split = split ? 1 : 0; g.Y = Y; g.ldy = ldy;
    if (r > 0) {
        g.rp = (r + 15) / 16 * 16;
        g.part = scratch;
        g.chunks = (int)ceil_div64(n, kDownChunk);
        g.vec_a = (((uintptr_t)L_A & 15) == 0 && (r & 3) == 0) ? 1 : 0;
        g.L_B = L_B;
        g.vec_b = ((uintptr_t)L_B & 15) == 0 ? 1 : 0;
        g.down = g.chunks * (g.rp / 16) * (int)ceil_div64(rows, 16);
    }
    return w4 ? dispatch_few<true>(ctx, g) : dispatch_few<false>(ctx, g);
}
