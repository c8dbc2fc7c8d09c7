// Remaining layer-output error of the quantized, compensated layer under activation quantization:
//     || X W^T  -  X'_q W~^T ||_F      over a sample of tokens,
// with X' = X M^-1 the smoothed activations (Eq. 10), X'_q their per-token RTN image (Sec. 5.1) and
// W~ = deq(Q(W_s)) + L_A L_B the compensated weight (end of Sec. 4.2).  This is the quantity that the
// paper's error figure plots per layer (Sec. 5.3: ||W X - W_q X_q||_F for RTN, the same norm after
// reconstruction for the other methods), in this library's tokens x channels orientation.
//
// Both outputs are contractions over the channel dimension, which is the contiguous one of every operand (X rows,
// W rows, code rows), and that is how the MFMA wants its operands.  The factors that are not bf16 already become pairs of bf16
// planes, x = hi + lo (about 2^-17 relative): W, fp32 activations.  bf16 activations are exact as they are, so Y = X W^T is two plane
// products instead of the three of a general fp32 product.  The second output needs no planes of W~: the codes of both sides multiply
// exactly on the int8 MFMA, at twice the rate, and the rank-r branch is r / 16 further bf16 steps per tile: L_B, P = x_q L_B^T and L_A as
// three planes each, which hold all of their 24 bits, and six products (with two planes and three products the call took 3 us less, and the result was up to 30 times
// as far from fp64 where factors cancel, and 2 to 5 times elsewhere).  ONE kernel forms both outputs of a tile: the integer sums, then Y on accumulators of its own, ||Y||^2 from
// these, which are then multiplied by -1 / s_t per row and receive c_o times the integer sums and L_A P, and ||s_t (...)||^2:
// neither output is ever stored.
// Without activation quantization (and with r > 128, or where the planes do not fit the workspace) the second output is a product of planes
// as well, of the activations or codes with those of W~ (divided by M when there are no codes), accumulated on top of the first.
// Bound: the MFMA rates; 2048 tokens of the 4096 x 4096 layer are 1.4e11 operations in two bf16 plane products and 0.7e11 in int8: 219 us
// (339 with four plane products; traced now 230), plus 31 for the planes of W and the factors (76 with those of W~) and 17 for P; the whole call 422 -> 289.
#include <math.h>

#include <type_traits>

#include "aser_internal.h"
#include "bf16_pair.h"
#include "rank_planes.h"

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef int i32x16_t __attribute__((ext_vector_type(16)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// eight values as hi = bf16(x) and lo = bf16(x - hi)
__device__ __forceinline__ void split8(const float (&v)[8], uint4& hi, uint4& lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        h[q] = bf16_pair(v[2 * q], v[2 * q + 1]);
        l[q] = bf16_pair(v[2 * q] - __uint_as_float(h[q] << 16), v[2 * q + 1] - __uint_as_float(h[q] & 0xFFFF0000u));
    }
    hi = make_uint4(h[0], h[1], h[2], h[3]);
    lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// Planes of W and of W~ = codes * scale + L_A L_B (divided by mdiag per column when it is given), np columns with zeros
// from n on.  A workgroup takes 64 x 64 entries; the rank-r part runs on the fp32 MFMA (16 x 16 x 4), a wavefront 16 rows of it.
__global__ __launch_bounds__(256) void weight_planes_kernel(const float* __restrict__ W, int64_t m, int64_t n, int64_t ldw, int64_t np,
                                                            const uint8_t* __restrict__ codes, int layout, const float* __restrict__ scales,
                                                            const float* __restrict__ L_A, const float* __restrict__ L_B, int r,
                                                            const float* __restrict__ mdiag, int w_vec, int c_vec,
                                                            uint16_t* __restrict__ w_hi, uint16_t* __restrict__ w_lo,
                                                            uint16_t* __restrict__ v_hi, uint16_t* __restrict__ v_lo) {
    __shared__ __align__(16) float low[64 * 68];                    // L_A L_B, transposed: [column][row]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lg = lane >> 4;
    const int64_t o0 = (int64_t)blockIdx.y * 64, i0 = (int64_t)blockIdx.x * 64;
    if (r > 0) {
        f32x4_t acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        const int64_t o = o0 + 16 * wave + li;
        const float* ap = L_A + (o < m ? o : m - 1) * r;             // rows and columns past the end: clamped here, dropped below
        const float* bp[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) bp[j] = L_B + (i0 + 16 * j + li < n ? i0 + 16 * j + li : n - 1);
        for (int k0 = 0; k0 < r; k0 += 16) {                         // four steps at a time: their loads are in flight together
            float av[4], bv[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 4 * u + lg, kc = k < r ? k : r - 1;
                av[u] = ap[kc];
#pragma unroll
                for (int j = 0; j < 4; ++j) bv[u][j] = bp[j][(int64_t)kc * n];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool ok = k0 + 4 * u + lg < r;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? av[u] : 0.f, ok ? bv[u][j] : 0.f, acc[j], 0, 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) *(f32x4_t*)(low + (16 * j + li) * 68 + 16 * wave + 4 * lg) = acc[j];
    }
    __syncthreads();
    const int64_t o = o0 + (tid >> 2);
    if (o >= m) return;
    const int64_t pitch = (layout == ASER_CODES_INT8) ? n : n / 2;
    const float sc = scales[o];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int cl = 16 * (tid & 3) + 8 * h;
        const int64_t c = i0 + cl;
        if (c >= np) continue;                                      // np is a multiple of 32, so groups of 8 are whole
        float w[8], v[8];
        int q[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) { w[e] = 0.f; q[e] = 0; }
        if (w_vec && c + 8 <= n) {
            const float4 x = *(const float4*)(W + o * ldw + c), y = *(const float4*)(W + o * ldw + c + 4);
            w[0] = x.x; w[1] = x.y; w[2] = x.z; w[3] = x.w; w[4] = y.x; w[5] = y.y; w[6] = y.z; w[7] = y.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (c + e < n) w[e] = W[o * ldw + c + e];
        }
        if (layout == ASER_CODES_INT8) {
            if (c_vec && c + 8 <= n) {
                const uint2 x = *(const uint2*)(codes + o * pitch + c);
#pragma unroll
                for (int e = 0; e < 8; ++e) q[e] = (int)((e < 4 ? x.x : x.y) << (24 - 8 * (e & 3))) >> 24;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (c + e < n) q[e] = (int)(int8_t)codes[o * pitch + c + e];
            }
        } else {                                                    // two's-complement nibbles, even column in the low one
            if (c_vec && c + 8 <= n) {
                const uint32_t x = *(const uint32_t*)(codes + o * pitch + c / 2);
#pragma unroll
                for (int e = 0; e < 8; ++e) q[e] = (int)(x << (28 - 4 * e)) >> 28;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (c + e < n) q[e] = (int)((uint32_t)codes[o * pitch + (c + e) / 2] << (28 - 4 * (e & 1))) >> 28;
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = (float)q[e] * sc;
            if (r > 0) v[e] += low[(cl + e) * 68 + (tid >> 2)];
            if (mdiag && c + e < n) v[e] /= mdiag[c + e];
            if (c + e >= n) v[e] = 0.f;
        }
        uint4 hi, lo;
        split8(w, hi, lo);
        *(uint4*)(w_hi + o * np + c) = hi;
        *(uint4*)(w_lo + o * np + c) = lo;
        split8(v, hi, lo);
        *(uint4*)(v_hi + o * np + c) = hi;
        *(uint4*)(v_lo + o * np + c) = lo;
    }
}

// What the product on codes reads, in one launch: workgroups [0, bx) the activations as bf16 planes of np columns (KIND as below, 3: they are used where
// they are) and their codes in rows of nc bytes, [bx, bx + bw) the planes of W and the weights' codes in such rows, the rest the factors
// (split_factors).  Zeros from channel n on; codes that are used where they are have no destination.  Eight columns per thread.  Bound by HBM, or, for a
// small layer, by the launch (a launch each: 512 x 1000, 17 tokens, r = 64: 95 us for the whole call, 62 now).
struct PrepArgs {
    const void* X; int64_t rows, ldx; uint16_t *x_hi, *x_lo; const int8_t* x_codes; int8_t* x_rows;
    const float* W; int64_t m, ldw; const uint8_t* w_codes; int layout, w_vec, c_vec; uint16_t *w_hi, *w_lo; int8_t* w_rows;
    const float *L_A, *L_B; int r, r_pad; AserRankPlanes rank;
    int64_t n, np, nc;
    int bx, bw;
};

template <int KIND>
__device__ __forceinline__ void act_plane8(const void* __restrict__ X, int64_t row, int64_t c, int64_t n, int64_t ldx, int64_t np, uint16_t* __restrict__ hi,
                                           uint16_t* __restrict__ lo) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {                         // past the end the last one again: a load behind a test is waited for at once
        const int64_t at = row * ldx + (c + e < n ? c + e : n - 1);
        if (KIND == 0) v[e] = __uint_as_float((uint32_t)((const uint16_t*)X)[at] << 16);
        if (KIND == 1) v[e] = ((const float*)X)[at];
        if (KIND == 2) v[e] = (float)((const int8_t*)X)[at];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = c + e < n ? v[e] : 0.f;
    uint4 h, l;
    split8(v, h, l);
    *(uint4*)(hi + row * np + c) = h;
    if (KIND == 1) *(uint4*)(lo + row * np + c) = l;
}

template <int KIND>
__global__ __launch_bounds__(256) void eval_prep_kernel(PrepArgs a) {
    const int64_t n = a.n, np = a.np, nc = a.nc, per_row = nc / 8;
    if ((int)blockIdx.x < a.bx) {
        const int64_t total = a.rows * per_row;
        for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)a.bx * 256) {
            const int64_t row = t / per_row, c = (t % per_row) * 8;
            if constexpr (KIND != 3)
                if (c < np) act_plane8<KIND>(a.X, row, c, n, a.ldx, np, a.x_hi, a.x_lo);
            if (!a.x_rows) continue;
            uint32_t b[2] = {0u, 0u};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (c + e < n) b[e >> 2] |= (uint32_t)(uint8_t)a.x_codes[row * n + c + e] << (8 * (e & 3));
            *(uint2*)(a.x_rows + row * nc + c) = make_uint2(b[0], b[1]);
        }
        return;
    }
    if ((int)blockIdx.x >= a.bx + a.bw) {
        split_factors<3, false>((int64_t)blockIdx.x - a.bx - a.bw, (int64_t)gridDim.x - a.bx - a.bw, a.L_A, a.L_B, a.m, n, a.r, a.r_pad, a.rank);
        return;
    }
    const int64_t block = (int64_t)blockIdx.x - a.bx, blocks = a.bw;
    const float* const W = a.W;
    const uint8_t* const codes = a.w_codes;
    const int64_t m = a.m, ldw = a.ldw;
    const int layout = a.layout;
    uint16_t *const w_hi = a.w_hi, *const w_lo = a.w_lo;
    int8_t* const q = a.w_rows;
    const bool w_vec = a.w_vec, c_vec = a.c_vec;
    const int64_t total = m * per_row, pitch = (layout == ASER_CODES_INT8) ? n : n / 2;
    for (int64_t t = block * 256 + threadIdx.x; t < total; t += blocks * 256) {
        const int64_t o = t / per_row, c = (t % per_row) * 8;
        if (c < np) {
            float w[8];
            if (w_vec && c + 8 <= n) {
                const f32x4_t x = __builtin_nontemporal_load((const f32x4_t*)(W + o * ldw + c)), y = __builtin_nontemporal_load((const f32x4_t*)(W + o * ldw + c + 4));
#pragma unroll
                for (int e = 0; e < 4; ++e) { w[e] = x[e]; w[4 + e] = y[e]; }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = c + e < n ? W[o * ldw + c + e] : 0.f;
            }
            uint4 hi, lo;
            split8(w, hi, lo);
            *(uint4*)(w_hi + o * np + c) = hi;
            *(uint4*)(w_lo + o * np + c) = lo;
        }
        if (!q) continue;
        uint32_t b[2] = {0u, 0u};
        const uint8_t* src = codes + o * pitch;
        if (layout == ASER_CODES_INT8) {
            if (c_vec && c + 8 <= n) {
                const uint2 x = *(const uint2*)(src + c);
                b[0] = x.x; b[1] = x.y;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (c + e < n) b[e >> 2] |= (uint32_t)src[c + e] << (8 * (e & 3));
            }
        } else {                                                    // two's-complement nibbles, even column in the low one
            uint32_t x = 0u;
            if (c_vec && c + 8 <= n) x = *(const uint32_t*)(src + c / 2);
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + 2 * e < n) x |= (uint32_t)src[c / 2 + e] << (8 * e);      // n is even
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e >> 2] |= ((uint32_t)((int)(x << (28 - 4 * e)) >> 28) & 0xFFu) << (8 * (e & 3));
        }
        *(uint2*)(q + o * nc + c) = make_uint2(b[0], b[1]);
    }
}

// Activations as bf16 planes of np columns (zeros from n on): KIND 0 bf16 X copied, 1 fp32 X as hi and lo, 2 int8 codes.
template <int KIND>
__global__ __launch_bounds__(256) void act_planes_kernel(const void* __restrict__ X, int64_t rows, int64_t n, int64_t ldx, int64_t np,
                                                         uint16_t* __restrict__ hi, uint16_t* __restrict__ lo) {
    const int64_t total = rows * (np / 8);
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256)
        act_plane8<KIND>(X, t / (np / 8), (t % (np / 8)) * 8, n, ldx, np, hi, lo);
}

struct EvalArgs {
    const char* a[6]; int64_t pa[6];          // activation planes: address and row pitch in bytes
    const char* b[6]; int64_t pb[6];          // weight planes, likewise (pb: CODED, otherwise 2 np)
    int segs1, segs;                          // plane products up to Y (CODED: the first is of the codes), and of both outputs
    int64_t np, nc, rows, m;                  // channels of a plane row (a multiple of 32), of a code row (of 64)
    const float* xs;                          // per-token scales, or null (1)
    const float* ws;                          // CODED: scales of the outputs, and the rank-r branch as planes of r_pad columns
    AserRankPlanes rank; int r_pad;
    double* out;                              // [0] += ||Y||^2, [1] += ||difference||^2
};

// byte offset of 16-byte chunk c (0..3) of row r inside a [rows][64 bytes] LDS tile
__device__ __forceinline__ int eval_off(int r, int c) { return r * 64 + ((c ^ ((r >> 2) & 3)) << 4); }

// 64 TI tokens x 64 TJ outputs per workgroup (4 wavefronts 2 x 2), 32 channels of one plane product per step.  The
// ring of four stages, the LDS-direct loads in inline assembly, the XOR swizzle and the XCD-aware numbering of the tiles are those of
// the inference kernel's 256 x 256 tiles; operand fragments of the next 16 channels are read under the MFMAs of the
// current ones.  Rows past the end repeat the last one and are left out of the sums.
// CODED: the first product is of int8 codes, 64 channels per step, on integer accumulators.
// No more than two wavefronts per SIMD are asked for where two sets of accumulators fill the registers; for 64 x 64 tiles that bound would keep three of five workgroups
// off a compute unit (500 tokens of 6144 x 6144: 454 -> 552 us).
template <int TI, int TJ, bool CODED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, CODED && TI * TJ > 1 ? 2 : 8))) void eval_kernel(EvalArgs g, int tiles_n, int64_t tiles_total) {
    extern __shared__ __align__(16) char smem[];
    __shared__ float sx[64 * TI], live[64 * TI];          // per row: its scale, 1; 0 past the last row
    constexpr int A_BYTES = 64 * TI * 64, STAGE = A_BYTES + 64 * TJ * 64, NL = TI + TJ;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave >> 1) * 32 * TI, wn0 = (wave & 1) * 32 * TJ;
    const int64_t per_xcd = (tiles_total + 7) / 8;
    const int64_t tile = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= tiles_total) return;
    const int64_t T0 = (tile / tiles_n) * 64 * TI, O0 = (tile % tiles_n) * 64 * TJ;
    for (int t = tid; t < 64 * TI; t += 256) {
        const bool in = T0 + t < g.rows;
        sx[t] = in ? (g.xs ? g.xs[T0 + t] : 1.f) : 0.f;
        live[t] = in ? 1.f : 0.f;
    }

    // ---- fetch roles: instruction t of this wave is tile rows 16 (NT wave + t) + lane / 4, chunk slot lane % 4
    const int chunk = 16 * ((lane & 3) ^ ((lane >> 4) & 3));
    int arow[TI], brow[CODED ? TJ : 1];
    uint32_t aoff[TI], boff[TJ];
#pragma unroll
    for (int t = 0; t < TI; ++t) {
        const int row = 16 * (TI * wave + t) + (lane >> 2);
        arow[t] = (T0 + row < g.rows) ? row : (int)(g.rows - 1 - T0);
    }
#pragma unroll
    for (int t = 0; t < TJ; ++t) {
        const int row = 16 * (TJ * wave + t) + (lane >> 2);
        const int at = O0 + row < g.m ? row : (int)(g.m - 1 - O0);
        if constexpr (CODED) brow[t] = at;
        else boff[t] = (uint32_t)(at * 2 * (int)g.np + chunk);       // every plane of weights has the same rows
    }
    const int64_t segsteps = g.np / 32, steps0 = CODED ? g.nc / 64 : 0;
    const int64_t nsteps = steps0 + segsteps * (g.segs - (CODED ? 1 : 0)), steps1 = CODED ? nsteps : segsteps * g.segs1;
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    int iseg = 0;
    int64_t ikk = 0;                                      // plane product and step inside it of the stage to be fetched
    const char *abase = nullptr, *bbase = nullptr;
    auto seg_start = [&]() {
        const int64_t pa = g.pa[iseg], pb = CODED ? g.pb[iseg] : 2 * g.np;
        abase = g.a[iseg] + T0 * pa;
        bbase = g.b[iseg] + O0 * pb;
#pragma unroll
        for (int t = 0; t < TI; ++t) aoff[t] = (uint32_t)(arow[t] * (int)pa + chunk);
        if constexpr (CODED) {
#pragma unroll
            for (int t = 0; t < TJ; ++t) boff[t] = (uint32_t)(brow[t] * (int)pb + chunk);
        }
    };
    auto issue_one = [&](int64_t step, int q) {           // q: 0 .. TI - 1 activations, TI .. NL - 1 weights
        const uint32_t dst = ring + (uint32_t)(step & 3) * STAGE + (q < TI ? (TI * wave + q) * 1024 : A_BYTES + (TJ * wave + q - TI) * 1024);
        const char* base = q < TI ? abase : bbase;
        const uint32_t off = q < TI ? aoff[q < TI ? q : 0] : boff[q < TI ? 0 : q - TI];
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off), "s"(base) : "memory", "m0");
    };
    auto stage_done = [&]() {                             // all loads of a stage are issued: on to the next one
        abase += 64;
        bbase += 64;
        if (++ikk == (CODED && iseg == 0 ? steps0 : segsteps)) {
            ikk = 0;
            if (++iseg < g.segs) seg_start();
        }
    };
    constexpr int W2 = 0x0F70 | (2 * NL & 15) | ((2 * NL >> 4) << 14), W1 = 0x0F70 | (NL & 15);

    int offa[TI], offb[TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i) offa[i] = eval_off(wm0 + 32 * i + (lane & 31), lane >> 5);
#pragma unroll
    for (int j = 0; j < TJ; ++j) offb[j] = A_BYTES + eval_off(wn0 + 32 * j + (lane & 31), lane >> 5);
    auto read = [&](const char* st, int sl, int off) { return *(const bf16x8_t*)(st + (off ^ (sl ? 32 : 0))); };

    f32x16_t acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    i32x16_t iacc[CODED ? TI : 1][CODED ? TJ : 1];
    if constexpr (CODED) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) iacc[i][j][e] = 0;
    }

    seg_start();
    for (int64_t s = 0; s < 3 && s < nsteps; ++s) {
#pragma unroll
        for (int q = 0; q < NL; ++q) issue_one(s, q);
        stage_done();
    }
    if (nsteps >= 3) __builtin_amdgcn_s_waitcnt(W2);      // stage 0 has landed
    else if (nsteps == 2) __builtin_amdgcn_s_waitcnt(W1);
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    bf16x8_t a0[TI], b0[TJ], a1[TI], b1[TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i) a0[i] = read(smem, 0, offa[i]);
#pragma unroll
    for (int j = 0; j < TJ; ++j) b0[j] = read(smem, 0, offb[j]);

    // the sum of squares, in fp64, of the accumulators times a factor per row (0 past the last row, which those rows repeat)
    auto norm2 = [&](const float* factor) {
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                double part = 0.0;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const double v = (double)acc[i][j][e] * (double)factor[wm0 + 32 * i + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)];
                    part = fma(v, v, part);
                }
                if (O0 + wn0 + 32 * j + (lane & 31) < g.m) sum += part;
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        return sum;
    };
    auto scale_rows = [&]() {                             // Y has its norm: rows times -1 / s_t
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float sc = sx[wm0 + 32 * i + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)];
                const float f = sc >= 1.17549435e-38f ? -1.f / sc : 0.f;      // no reciprocal of a denormal scale (or past the last row)
#pragma unroll
                for (int j = 0; j < TJ; ++j) acc[i][j][e] *= f;
            }
    };
    auto step = [&](int64_t s, auto codes_tag) {
        constexpr bool CODES = decltype(codes_tag)::value;
        const char* st = smem + (int)(s & 3) * STAGE;
        const char* sn = smem + (int)((s + 1) & 3) * STAGE;
        const bool more = s + 1 < nsteps, fetch = s + 3 < nsteps;
        auto multiply = [&](int i, int j, const bf16x8_t& a, const bf16x8_t& b) {
            if constexpr (CODES) iacc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(i32x4_t, a), __builtin_bit_cast(i32x4_t, b), iacc[i][j], 0, 0, 0);
            else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i][j], 0, 0, 0);
        };
        // slice 0 (32 bytes of every row): the operands of slice 1 are read under its MFMAs
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                multiply(i, j, a0[i], b0[j]);
                const int q = i * TJ + j;
                if (q < TI) a1[q < TI ? q : 0] = read(st, 1, offa[q < TI ? q : 0]);
#pragma unroll
                for (int u = q; u < TJ; u += TI * TJ) b1[u] = read(st, 1, offb[u]);
                __builtin_amdgcn_sched_barrier(0);
            }
        // slice 1: behind its first MFMA the wait for the next stage and the barrier, then the loads of stage s + 3 and the
        // reads of the next step's slice 0
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                multiply(i, j, a1[i], b1[j]);
                const int q = i * TJ + j;
                if (q == 0 && more) {
                    if (s + 2 < nsteps) __builtin_amdgcn_s_waitcnt(W1);
                    else __builtin_amdgcn_s_waitcnt(0x0F70);
                    __syncthreads();                      // everyone's share landed; stage s - 1 is free
                }
                if (q == 0) {
                    if (more) {
#pragma unroll
                        for (int u = 0; u < TI; ++u) a0[u] = read(sn, 0, offa[u]);
#pragma unroll
                        for (int u = 0; u < TJ; ++u) b0[u] = read(sn, 0, offb[u]);
                    }
                    if (fetch) {
#pragma unroll
                        for (int u = 0; u < NL; ++u) issue_one(s + 3, u);
                        stage_done();
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    if constexpr (CODED) {
        for (int64_t s = 0; s < steps0; ++s) step(s, std::true_type{});
        for (int64_t s = steps0; s < nsteps; ++s) step(s, std::false_type{});
        const double y2 = norm2(live);
        if (lane == 0) atomicAdd(g.out, y2);
        scale_rows();
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int64_t col = O0 + wn0 + 32 * j + (lane & 31);
            const float c = g.ws[col < g.m ? col : g.m - 1];
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = fmaf((float)iacc[i][j][e], c, acc[i][j][e]);
        }
        for (int kk = 0; kk < g.r_pad; kk += 16) {        // L_A P, 16 columns of either at a time
            const int kq = kk + 8 * (lane >> 5);
            bf16x8_t pv[TI][3];
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int64_t row = T0 + wm0 + 32 * i + (lane & 31), at = (row < g.rows ? row : g.rows - 1) * g.r_pad + kq;
#pragma unroll
                for (int p = 0; p < 3; ++p) pv[i][p] = *(const bf16x8_t*)(g.rank.p[p] + at);
            }
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int64_t col = O0 + wn0 + 32 * j + (lane & 31), at = (col < g.m ? col : g.m - 1) * g.r_pad + kq;
                bf16x8_t lv[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) lv[p] = *(const bf16x8_t*)(g.rank.la[p] + at);
#pragma unroll
                for (int both = 2; both >= 0; --both)        // products down to 2^-16 of the largest, small ones first; the rest is 2^-24
#pragma unroll
                    for (int p = 0; p <= both; ++p)
#pragma unroll
                        for (int i = 0; i < TI; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pv[i][p], lv[both - p], acc[i][j], 0, 0, 0);
            }
        }
    } else {
        for (int64_t s = 0; s < nsteps; ++s) {
            if (s == steps1) {
                const double y2 = norm2(live);
                if (lane == 0) atomicAdd(g.out, y2);
                scale_rows();
            }
            step(s, std::false_type{});
        }
    }
    const double e2 = norm2(sx);
    if (lane == 0) atomicAdd(g.out + 1, e2);
}

template <int TI, int TJ, bool CODED>
int launch_eval(aser_ctx* ctx, const EvalArgs& g) {
    static bool done[16] = {false};
    constexpr int lds = 4 * 64 * (64 * TI + 64 * TJ);
    auto kern = eval_kernel<TI, TJ, CODED>;
    if (ctx->device >= 0 && ctx->device < 16 && !done[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        done[ctx->device] = true;
    }
    const int64_t tn = ceil_div64(g.m, 64 * TJ), total = tn * ceil_div64(g.rows, 64 * TI);
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * ceil_div64(total, 8))), dim3(256), lds, ctx->stream, g, (int)tn, total);
    return aser_check_launch(ctx, "layer_output_error");
}

// The largest tile with which the launch still fills the device
template <bool CODED>
int pick_eval(aser_ctx* ctx, const EvalArgs& g) {
    if (ceil_div64(g.rows, 128) * ceil_div64(g.m, 256) >= 200) return launch_eval<2, 4, CODED>(ctx, g);
    if (ceil_div64(g.rows, 128) * ceil_div64(g.m, 128) >= 200) return launch_eval<2, 2, CODED>(ctx, g);
    return launch_eval<1, 1, CODED>(ctx, g);
}

// The workspace is what the operands, one output and L_A take in fp32 (two m x n, two rows x n, a rows x m and an r x m array), the
// activation codes and scales, and a block of scalars.  The bf16 planes, four of the weights and three of the activations with rows
// padded to np channels, lie in the room of the former.  They fit unless n is short of a multiple of 32 and rows (or n) are few; then the
// outputs, or the tokens, are taken in blocks of m_blk, rows_blk.  One of each always fits: 14 np bytes, np <= n + 31, in
// at least 16 n + 8 bytes of six arrays of 256 bytes or more.
struct EvalPlan {
    int64_t np, m_blk, rows_blk;
    size_t planes, off_codes, off_scales, off_scal, total;
};

void eval_plan(int64_t m, int64_t n, int64_t rows, int r, EvalPlan* p) {
    p->np = (n + 31) / 32 * 32;
    p->planes = 2 * align_up((size_t)m * n * 4, 256) + 2 * align_up((size_t)rows * n * 4, 256) + align_up((size_t)rows * m * 4, 256) +
                align_up((size_t)(r > 0 ? r : 1) * m * 4, 256);
    size_t off = p->planes;
    p->off_codes = off; off += align_up((size_t)rows * n, 256);
    p->off_scales = off; off += align_up((size_t)rows * 4, 256);
    p->off_scal = off; off += 256;
    p->total = off;
    p->m_blk = m;
    p->rows_blk = rows;
    while ((size_t)(8 * p->m_blk + 6 * p->rows_blk) * p->np > p->planes && (p->m_blk > 1 || p->rows_blk > 1)) {
        int64_t& larger = 8 * p->m_blk >= 6 * p->rows_blk && p->m_blk > 1 ? p->m_blk : (p->rows_blk > 1 ? p->rows_blk : p->m_blk);
        larger = (larger + 1) / 2;
    }
}

// Where the operands of the form on codes lie, in the room of the planes; total: what they take.
struct CodedPlan {
    int64_t np, nc;
    int r_pad;
    bool x_direct, xc_direct, wc_direct;
    size_t w_hi, w_lo, wc, x_hi, x_lo, xc, p[3], la[3], lb, total;
};

void coded_plan(int64_t m, int64_t n, int64_t rows, int r, bool bf16, bool x_direct, bool wc_direct, CodedPlan* p) {
    p->np = (n + 31) / 32 * 32;
    p->nc = (n + 63) / 64 * 64;
    p->r_pad = (r + 31) / 32 * 32;
    p->x_direct = x_direct;
    p->xc_direct = p->nc == n;
    p->wc_direct = wc_direct && p->nc == n;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off += align_up(bytes, 256); return at; };
    p->w_hi = take((size_t)m * p->np * 2);
    p->w_lo = take((size_t)m * p->np * 2);
    p->wc = take(p->wc_direct ? 0 : (size_t)m * p->nc);
    p->x_hi = take(x_direct ? 0 : (size_t)rows * p->np * 2);
    p->x_lo = take(x_direct || bf16 ? 0 : (size_t)rows * p->np * 2);
    p->xc = take(p->xc_direct ? 0 : (size_t)rows * p->nc);
    for (size_t& at : p->p) at = take((size_t)rows * p->r_pad * 2);
    for (size_t& at : p->la) at = take((size_t)m * p->r_pad * 2);
    p->lb = take((size_t)p->np * p->r_pad * 6);
    p->total = off;
}

}  // namespace

extern "C" size_t aser_output_error_workspace_bytes(int64_t m, int64_t n, int64_t rows, int32_t r) {
    if (m <= 0 || n <= 0 || rows <= 0 || r < 0) return 0;
    EvalPlan p;
    eval_plan(m, n, rows, r, &p);
    return p.total + kAserWsTail;
}

extern "C" int aser_layer_output_error(aser_ctx* ctx, const float* W, int64_t m, int64_t n, int64_t ldw,
                                       const void* X, int x_dtype, int64_t rows, int64_t ldx, const float* mdiag,
                                       const void* codes, int32_t layout, const float* scales,
                                       const float* L_A, const float* L_B, int32_t r, int32_t act_bits,
                                       double* err, double* ref_norm) {
    if (!ctx) return ASER_ERR_INVALID_ARG;
    if (!W || !X || !codes || !scales || !err) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "layer_output_error: null pointer");
    if (x_dtype != ASER_DTYPE_BF16 && x_dtype != ASER_DTYPE_F32) ASER_FAIL(ctx, ASER_ERR_DTYPE, "layer_output_error: dtype must be bf16 or f32");
    if (m <= 0 || n <= 0 || rows <= 0 || ldw < n || ldx < n) ASER_FAIL(ctx, ASER_ERR_SHAPE, "layer_output_error: bad shape");
    if (r < 0 || (r > 0 && (!L_A || !L_B))) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "layer_output_error: r > 0 needs L_A and L_B");
    if (layout != ASER_CODES_INT8 && layout != ASER_CODES_INT4_PACKED)
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "layer_output_error: unknown code layout");
    if (layout == ASER_CODES_INT4_PACKED && (n & 1)) ASER_FAIL(ctx, ASER_ERR_SHAPE, "layer_output_error: packed int4 needs even n");
    if (act_bits != 0 && (act_bits < 2 || act_bits > 8)) ASER_FAIL(ctx, ASER_ERR_DTYPE, "layer_output_error: act_bits must be 0 or in [2, 8]");
    if (n > 32768) ASER_FAIL(ctx, ASER_ERR_SHAPE, "layer_output_error: n > 32768 is not supported");
    if (((uintptr_t)W & 3) || ((uintptr_t)scales & 3) || ((uintptr_t)X & (x_dtype == ASER_DTYPE_BF16 ? 1 : 3)))
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "layer_output_error: misaligned pointer");
    EvalPlan pl;
    eval_plan(m, n, rows, r, &pl);
    if (!ctx->ws || ctx->ws_bytes < pl.total + kAserWsTail)
        ASER_FAIL(ctx, ASER_ERR_WORKSPACE, "layer_output_error: workspace too small (%zu needed)", pl.total + kAserWsTail);
    ASER_TRY(aser_prepare_device(ctx));
    char* ws = (char*)ctx->ws;
    const int64_t np = pl.np, wn = pl.m_blk * np, xn = pl.rows_blk * np;
    uint16_t* w_hi = (uint16_t*)ws;                       // planes: rows of np entries, 64 bytes or a multiple
    uint16_t *w_lo = w_hi + wn, *v_hi = w_lo + wn, *v_lo = v_hi + wn, *x_hi = v_lo + wn, *x_lo = x_hi + xn, *c_q = x_lo + xn;
    int8_t* acodes = (int8_t*)(ws + pl.off_codes);
    float* ascales = (float*)(ws + pl.off_scales);
    double* scal = (double*)(ws + pl.off_scal);           // [0] = ||Y||^2, [1] = err^2
    const bool bf16 = x_dtype == ASER_DTYPE_BF16;
    const size_t xsz = bf16 ? 2 : 4;
    const int64_t cpitch = layout == ASER_CODES_INT8 ? n : n / 2;
    const int w_vec = (((uintptr_t)W & 15) == 0 && (ldw & 3) == 0) ? 1 : 0;
    const int c_vec = ((uintptr_t)codes & (layout == ASER_CODES_INT8 ? 7 : 3)) == 0 && (n & 7) == 0;
    // bf16 activations whose rows can be fetched 16 bytes at a time are read where they are
    const bool direct = bf16 && ((uintptr_t)X & 15) == 0 && (ldx & 7) == 0 && ldx <= (1 << 22) && np == n;   // 128 rows within 32-bit offsets

    ASER_TRY(aser_fill_bytes(ctx, scal, 256));
    if (act_bits != 0) ASER_TRY(aser_quantize_act_rtn(ctx, X, x_dtype, rows, n, ldx, mdiag, act_bits, acodes, ascales));
    CodedPlan cp;
    coded_plan(m, n, rows, (int)r, bf16, direct, layout == ASER_CODES_INT8 && ((uintptr_t)codes & 15) == 0, &cp);
    const bool coded = act_bits != 0 && r <= 128 && cp.total <= pl.planes;
    if (coded) {
        auto blocks = [](int64_t items) { return (int)(ceil_div64(items, 256) < 4096 ? ceil_div64(items, 256) : 4096); };
        uint16_t *xh = (uint16_t*)(ws + cp.x_hi), *xl = (uint16_t*)(ws + cp.x_lo);
        const int8_t* xc = cp.xc_direct ? acodes : (const int8_t*)(ws + cp.xc);
        const int8_t* wc = cp.wc_direct ? (const int8_t*)codes : (const int8_t*)(ws + cp.wc);
        PrepArgs a{};
        a.X = X; a.rows = rows; a.ldx = ldx; a.x_hi = xh; a.x_lo = xl; a.x_codes = acodes; a.x_rows = cp.xc_direct ? nullptr : (int8_t*)(ws + cp.xc);
        a.W = W; a.m = m; a.ldw = ldw; a.w_codes = (const uint8_t*)codes; a.layout = (int)layout; a.w_vec = w_vec; a.c_vec = c_vec;
        a.w_hi = (uint16_t*)(ws + cp.w_hi); a.w_lo = (uint16_t*)(ws + cp.w_lo); a.w_rows = cp.wc_direct ? nullptr : (int8_t*)(ws + cp.wc);
        a.n = n; a.np = np; a.nc = cp.nc;
        a.bx = direct && cp.xc_direct ? 0 : blocks(rows * (cp.nc / 8));
        a.bw = blocks(m * (cp.nc / 8));
        int64_t total = (int64_t)a.bx + a.bw;
        if (r > 0) {
            for (int i = 0; i < 3; ++i) {
                a.rank.p[i] = (uint16_t*)(ws + cp.p[i]);
                a.rank.la[i] = (uint16_t*)(ws + cp.la[i]);
            }
            a.rank.lb = ws + cp.lb;
            a.L_A = L_A; a.L_B = L_B; a.r = (int)r; a.r_pad = cp.r_pad;
            total += split_factors_blocks(m, n, cp.r_pad);
        }
        auto prep = direct ? eval_prep_kernel<3> : (bf16 ? eval_prep_kernel<0> : eval_prep_kernel<1>);
        hipLaunchKernelGGL(prep, dim3((unsigned)total), dim3(256), 0, ctx->stream, a);
        ASER_TRY(aser_check_launch(ctx, "eval_prep"));
        EvalArgs g{};
        g.np = np; g.nc = cp.nc; g.rows = rows; g.m = m; g.out = scal; g.xs = ascales; g.ws = scales;
        auto add = [&](const void* a, int64_t pa, const void* b, int64_t pb) {
            g.a[g.segs] = (const char*)a; g.pa[g.segs] = pa; g.b[g.segs] = (const char*)b; g.pb[g.segs] = pb; ++g.segs;
        };
        const void* xa = direct ? X : (const void*)xh;
        const int64_t xpitch = direct ? ldx * 2 : np * 2;
        add(xc, cp.nc, wc, cp.nc);
        add(xa, xpitch, ws + cp.w_hi, np * 2);
        add(xa, xpitch, ws + cp.w_lo, np * 2);
        if (!bf16) add(xl, np * 2, ws + cp.w_hi, np * 2);
        if (r > 0) {
            g.rank = a.rank;
            g.r_pad = cp.r_pad;
            ASER_TRY(aser_rank_down(ctx, xc, cp.nc, nullptr, rows, n, nullptr, (int)r, 3, nullptr, m, a.rank));
        }
        ASER_TRY(pick_eval<true>(ctx, g));
    }
    for (int64_t t0 = 0; t0 < rows && !coded; t0 += pl.rows_blk) {
        const int64_t tr = rows - t0 < pl.rows_blk ? rows - t0 : pl.rows_blk;
        const void* Xt = (const char*)X + (size_t)t0 * ldx * xsz;
        const int64_t groups = tr * (np / 8);
        const dim3 xgrid((unsigned)(ceil_div64(groups, 256) < 4096 ? ceil_div64(groups, 256) : 4096));
        if (!direct) {
            if (bf16) hipLaunchKernelGGL(act_planes_kernel<0>, xgrid, dim3(256), 0, ctx->stream, Xt, tr, n, ldx, np, x_hi, x_lo);
            else hipLaunchKernelGGL(act_planes_kernel<1>, xgrid, dim3(256), 0, ctx->stream, Xt, tr, n, ldx, np, x_hi, x_lo);
            ASER_TRY(aser_check_launch(ctx, "act_planes"));
        }
        if (act_bits != 0) {
            hipLaunchKernelGGL(act_planes_kernel<2>, xgrid, dim3(256), 0, ctx->stream, (const void*)(acodes + t0 * n), tr, n, n, np, c_q, c_q);
            ASER_TRY(aser_check_launch(ctx, "code_planes"));
        }
        for (int64_t o0 = 0; o0 < m; o0 += pl.m_blk) {
            const int64_t om = m - o0 < pl.m_blk ? m - o0 : pl.m_blk;
            if (t0 == 0 || pl.m_blk < m) {
                const dim3 grid((unsigned)ceil_div64(np, 64), (unsigned)ceil_div64(om, 64));
                hipLaunchKernelGGL(weight_planes_kernel, grid, dim3(256), 0, ctx->stream, W + o0 * ldw, om, n, ldw, np,
                                   (const uint8_t*)codes + o0 * cpitch, (int)layout, scales + o0, L_A ? L_A + o0 * r : L_A, L_B, (int)r,
                                   act_bits == 0 ? mdiag : (const float*)nullptr, w_vec, c_vec, w_hi, w_lo, v_hi, v_lo);
                ASER_TRY(aser_check_launch(ctx, "weight_planes"));
            }
            EvalArgs g{};
            g.np = np; g.rows = tr; g.m = om; g.out = scal;
            auto add = [&](const void* a, int64_t pa, const void* b) { g.a[g.segs] = (const char*)a; g.pa[g.segs] = pa; g.b[g.segs] = (const char*)b; ++g.segs; };
            const void* xa = direct ? Xt : (const void*)x_hi;
            const int64_t xpitch = direct ? ldx * 2 : np * 2;
            add(xa, xpitch, w_hi);
            add(xa, xpitch, w_lo);
            if (!bf16) add(x_lo, np * 2, w_hi);
            g.segs1 = g.segs;
            if (act_bits == 0) {
                add(xa, xpitch, v_hi);
                add(xa, xpitch, v_lo);
                if (!bf16) add(x_lo, np * 2, v_hi);
            } else {
                add(c_q, np * 2, v_hi);
                add(c_q, np * 2, v_lo);
                g.xs = ascales + t0;
            }
            ASER_TRY(pick_eval<false>(ctx, g));
        }
    }
    double h[2] = {0.0, 0.0};
    ASER_HIP(ctx, hipMemcpyAsync(h, scal, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    ASER_HIP(ctx, hipStreamSynchronize(ctx->stream));
    // finite outputs give finite sums in fp64; an infinite activation may leave an infinite sum instead of a NaN
    if (!isfinite(h[0]) || !isfinite(h[1])) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "layer_output_error: non-finite values in the inputs");
    *err = sqrt(h[1]);
    if (ref_norm) *ref_norm = sqrt(h[0]);
    return ASER_OK;
}
