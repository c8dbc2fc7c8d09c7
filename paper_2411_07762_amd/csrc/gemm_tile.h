// The tile of the MFMA contraction kernels (see gemm_tn.hip for the whole): operand fetch, conversion and LDS layout,
// the products of a K step, the epilogues, and the two bodies that put them together.
#pragma once
#include "aser_internal.h"
#include "bf16_pair.h"

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

namespace {

constexpr int kThreads = 256;

template <int IN> struct InTraits;
template <> struct InTraits<GEMM_IN_BF16> { static constexpr int BK = 64, NP = 1, VEC = 8; };
template <> struct InTraits<GEMM_IN_F32X3> { static constexpr int BK = 32, NP = 2, VEC = 4; };
template <> struct InTraits<GEMM_IN_F32X6> { static constexpr int BK = 32, NP = 3, VEC = 4; };

// LDS position (in 16-byte chunks) of row `mn` inside one k-block.  The XOR pattern makes both
// the transposing stores (8 consecutive rows per lane) and the MFMA operand reads (32
// consecutive rows per half wave) hit distinct bank groups.
__device__ __forceinline__ int swz(int mn) { return (mn ^ ((mn >> 3) & 7)) ^ (((mn >> 6) & 1) << 3); }

// Eight 16-byte rows of one operand block in flight between global memory and LDS.
struct Staged {
    uint4 r[8];
};

// Per-thread fetch state of one operand tile (BMN rows of the tile, BK k-values per step).
// FAST: the operand is 16-byte aligned with leading dimension and extent multiples of the vector
// width, so every column group is whole; loads are branch-free (rows past the K range are read
// from the last valid row and zeroed, column groups past the extent are read from group 0 and
// simply never stored to C).  Otherwise a guarded element-wise path is used.
template <int IN, int BMN, bool FAST>
struct Fetch {
    static constexpr int BK = InTraits<IN>::BK;
    static constexpr int VEC = InTraits<IN>::VEC;       // elements per 16-byte load
    static constexpr int GROUPS = BMN / VEC;            // 16-byte column groups across the tile
    static constexpr int ESZ = (IN == GEMM_IN_BF16) ? 2 : 4;

    const char* p;      // address of (k row of this thread's first load in the next step, first column)
    const char* plast;  // same column group in the last valid k row (FAST)
    int64_t ld_bytes;
    int64_t k;          // k index of this thread's first row in the next step to be loaded
    int cg, kb;         // column group and k-block handled by this thread
    int ncols;          // valid columns at this thread's group (0..VEC)
    bool active, vec_ok;

    __device__ __forceinline__ void init(const void* base, int64_t ld, int64_t mn0, int64_t MN, int64_t k0,
                                         int64_t kEnd, int tid) {
        active = tid < GROUPS * (BK / 8);
        cg = tid % GROUPS;
        kb = tid / GROUPS;
        int64_t col = mn0 + (int64_t)cg * VEC;
        int64_t rem = MN - col;
        ncols = rem >= VEC ? VEC : (rem > 0 ? (int)rem : 0);
        k = k0 + kb * 8;
        ld_bytes = ld * ESZ;
        if (FAST) {
            if (ncols != VEC) col = 0;
            p = (const char*)base + k * ld_bytes + col * ESZ;
            plast = (const char*)base + (kEnd - 1) * ld_bytes + col * ESZ;
            vec_ok = true;
            return;
        }
        p = (const char*)base + k * ld_bytes + col * ESZ;
        plast = p;
        vec_ok = (((uintptr_t)p & 15) == 0) && ((ld_bytes & 15) == 0) && ncols == VEC;
        if (ncols == 0) active = false;
    }

    // Issues the loads of the next step into `st` and moves on by one step.
    __device__ __forceinline__ void load(Staged& st, int64_t kEnd) {
        load_rows(st, kEnd);
        p += (int64_t)BK * ld_bytes;
        k += BK;
    }

    __device__ __forceinline__ void load_rows(Staged& st, int64_t kEnd) {
        uint4* r = st.r;
        if (FAST) {
            if (!active) return;
            if (k + 8 <= kEnd) {
#pragma unroll
                for (int j = 0; j < 8; ++j) r[j] = *(const uint4*)(p + j * ld_bytes);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool ok = k + j < kEnd;
                    const uint4 v = *(const uint4*)(ok ? p + j * ld_bytes : plast);
                    r[j] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
                }
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) r[j] = make_uint4(0u, 0u, 0u, 0u);
        if (!active) return;
        if (vec_ok) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (k + j < kEnd) r[j] = *(const uint4*)(p + j * ld_bytes);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (k + j < kEnd) {
                    const char* q = p + j * ld_bytes;
                    if (IN == GEMM_IN_BF16) {
                        uint32_t w[4] = {0u, 0u, 0u, 0u};
                        for (int e = 0; e < ncols; ++e)
                            w[e >> 1] |= (uint32_t)(*(const uint16_t*)(q + 2 * e)) << (16 * (e & 1));
                        r[j] = make_uint4(w[0], w[1], w[2], w[3]);
                    } else {
                        uint32_t w[4] = {0u, 0u, 0u, 0u};
                        for (int e = 0; e < ncols; ++e) w[e] = *(const uint32_t*)(q + 4 * e);
                        r[j] = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                }
            }
        }
    }

    // Writes a staged block as k-contiguous chunks into the operand's LDS area.
    __device__ __forceinline__ void store(const Staged& st, uint4* lds) const {
        if (!active) return;
        constexpr int KB = BK / 8;
        if (IN == GEMM_IN_BF16) {
            const uint32_t* w = (const uint32_t*)st.r;    // w[4*j + d]: row j, channel pair d
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int d = c >> 1;
                const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
                uint4 o;
                o.x = __builtin_amdgcn_perm(w[4 * 1 + d], w[4 * 0 + d], sel);
                o.y = __builtin_amdgcn_perm(w[4 * 3 + d], w[4 * 2 + d], sel);
                o.z = __builtin_amdgcn_perm(w[4 * 5 + d], w[4 * 4 + d], sel);
                o.w = __builtin_amdgcn_perm(w[4 * 7 + d], w[4 * 6 + d], sel);
                lds[kb * BMN + swz(cg * 8 + c)] = o;
            }
        } else {
            const float* x = (const float*)st.r;          // x[4*j + c]: row j, column c
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                uint32_t hi[4], lo[4], lo2[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float a = x[4 * (2 * q) + c], b = x[4 * (2 * q + 1) + c];
                    const uint32_t h = bf16_pair(a, b);
                    const float ah = __uint_as_float(h << 16), bh = __uint_as_float(h & 0xFFFF0000u);
                    hi[q] = h;
                    const float ar = a - ah, br = b - bh;           // exact: the remainder has at most 16 significant bits
                    lo[q] = bf16_pair(ar, br);
                    if (IN == GEMM_IN_F32X6) {
                        const float am = __uint_as_float(lo[q] << 16), bm = __uint_as_float(lo[q] & 0xFFFF0000u);
                        lo2[q] = bf16_pair(ar - am, br - bm);     // third term: x = hi + mid + lo to 24 bits
                    }
                }
                const int pos = kb * BMN + swz(cg * 4 + c);
                lds[pos] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                lds[KB * BMN + pos] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                if (IN == GEMM_IN_F32X6) lds[2 * KB * BMN + pos] = make_uint4(lo2[0], lo2[1], lo2[2], lo2[3]);
            }
        }
    }
};

template <int IN, int BM, int BN>
struct TileCfg {
    static constexpr int BK = InTraits<IN>::BK;
    static constexpr int NP = InTraits<IN>::NP;
    static constexpr int KB = BK / 8;
    static constexpr int A_CHUNKS = NP * KB * BM;
    static constexpr int B_CHUNKS = NP * KB * BN;
    static constexpr int STAGE_CHUNKS = A_CHUNKS + B_CHUNKS;
    static constexpr size_t LDS_BYTES = (size_t)2 * STAGE_CHUNKS * 16;
    static constexpr int TM = BM / 64, TN = BN / 64;     // 32 x 32 MFMA blocks per wave
};

// Scheduling hint: R groups of (one LDS read, then a share of MF MFMAs).
template <int R, int MF, int T>
struct SchedPattern {
    static __device__ __forceinline__ void emit() {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, (MF * (T + 1)) / R - (MF * T) / R, 0);
        SchedPattern<R, MF, T + 1>::emit();
    }
};
template <int R, int MF>
struct SchedPattern<R, MF, R> {
    static __device__ __forceinline__ void emit() {}
};

// All MFMAs of one K step from LDS stage (sa, sb).  Operand fragments are double buffered: the
// LDS reads of k-slice kk + 1 are in flight while the MFMAs of slice kk execute (one wave per
// SIMD: nothing else hides the LDS latency), and the scheduling hints spread them evenly.
template <int IN, int BM, int BN, int TM, int TN>
__device__ __forceinline__ void mfma_step(f32x16_t (&acc)[TM][TN], const uint4* sa, const uint4* sb,
                                          const int (&offa)[TM], const int (&offb)[TN]) {
    using Cfg = TileCfg<IN, BM, BN>;
    constexpr int NP = Cfg::NP, KB = Cfg::KB, KK = Cfg::BK / 16;
    constexpr int R = NP * (TM + TN);                   // LDS reads per k-slice
    constexpr int MF = TM * TN * (NP == 3 ? 6 : (NP == 2 ? 3 : 1));     // MFMAs per k-slice
    bf16x8_t a[2][NP][TM], b[2][NP][TN];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[0][p][i] = __builtin_bit_cast(bf16x8_t, sa[(p * KB) * BM + offa[i]]);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[0][p][j] = __builtin_bit_cast(bf16x8_t, sb[(p * KB) * BN + offb[j]]);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        const int cur = kk & 1, nxt = cur ^ 1;
        if (kk + 1 < KK) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    a[nxt][p][i] = __builtin_bit_cast(bf16x8_t, sa[(p * KB + 2 * (kk + 1)) * BM + offa[i]]);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    b[nxt][p][j] = __builtin_bit_cast(bf16x8_t, sb[(p * KB + 2 * (kk + 1)) * BN + offb[j]]);
            }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (NP == 3) {
                    // x = hi + mid + lo: all products down to 2^-24 of hi * hi, smallest first
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][NP - 1][i], b[cur][0][j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][0][i], b[cur][NP - 1][j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][1][i], b[cur][1][j], acc[i][j], 0, 0, 0);
                }
                if (NP >= 2) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][1][i], b[cur][0][j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][0][i], b[cur][1][j], acc[i][j], 0, 0, 0);
                }
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][0][i], b[cur][0][j], acc[i][j], 0, 0, 0);
            }
        if (kk + 1 < KK) SchedPattern<R, MF, 0>::emit();
        else __builtin_amdgcn_sched_group_barrier(0x008, MF, 0);
    }
}

// Epilogue of a wavefront's part at (I0, J0).  acc[i][j][e] is C(row, col) with row = 32 i + 8 (e / 4) + 4 (lane / 32) + e % 4,
// col = 32 j + lane % 32.  RESID: the tile can form the residual norm (the large tiles have no registers to spare for it).
template <int TM, int TN, bool RESID>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& g, f32x16_t (&acc)[TM][TN], int64_t I0, int64_t J0, int lane) {
    const float alpha = g.alpha;
    if (RESID && g.epi == GEMM_EPI_RESID) {
        // squared Frobenius norm of C + alpha acc, nothing stored: the loads of one row of 32 x 32
        // blocks are in flight together, squares are summed in fp64, one atomic per wavefront
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int64_t rbase = I0 + 32 * i + 4 * (lane >> 5);
            float old[TN][16];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t col = J0 + 32 * j + (lane & 31);
                const float* cbase = g.C + rbase * g.ldc + col;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int dr = 8 * (e >> 2) + (e & 3);
                    const bool in = col < g.N && rbase + dr < g.M;
                    old[j][e] = in ? cbase[(int64_t)dr * g.ldc] : 0.f;
                    if (!in) acc[i][j][e] = 0.f;
                }
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                float part = 0.f;                          // 16 squares of comparable size in fp32, then fp64
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float d = old[j][e] + alpha * acc[i][j][e];
                    part = fmaf(d, d, part);
                }
                sum += (double)part;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) atomicAdd(g.sumsq, sum);
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = J0 + 32 * j + (lane & 31);
            const int64_t rbase = I0 + 32 * i + 4 * (lane >> 5);
            if (col >= g.N) continue;
            float* cbase = g.C + rbase * g.ldc + col;
            if (g.epi == GEMM_EPI_ATOMIC) {
                // upper_only: entries left of the diagonal are never read by the caller; leaving them
                // out halves the atomic traffic of the small symmetric products
                const int64_t rmax = g.upper_only ? (col + 1 < g.M ? col + 1 : g.M) : g.M;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int dr = 8 * (e >> 2) + (e & 3);
                    if (rbase + dr < rmax) unsafeAtomicAdd(cbase + (int64_t)dr * g.ldc, alpha * acc[i][j][e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int dr = 8 * (e >> 2) + (e & 3);
                    if (rbase + dr < g.M) cbase[(int64_t)dr * g.ldc] = alpha * acc[i][j][e];
                }
                if (g.Ct) {
                    // transposed copy: the 4 consecutive rows of one accumulator group are contiguous in Ct
                    float* tbase = g.Ct + col * g.ldct + rbase;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int dr = 8 * q;
                        if (rbase + dr + 3 < g.M && ((((uintptr_t)(tbase + dr)) & 15) == 0)) {
                            *(float4*)(tbase + dr) = make_float4(alpha * acc[i][j][4 * q], alpha * acc[i][j][4 * q + 1],
                                                                 alpha * acc[i][j][4 * q + 2], alpha * acc[i][j][4 * q + 3]);
                        } else {
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                if (rbase + dr + u < g.M) tbase[dr + u] = alpha * acc[i][j][4 * q + u];
                        }
                    }
                }
            }
        }
}

// One tile of C over the K range [kBeg, kEnd).
//
// Pipeline: while step s is multiplied out of LDS stage s % 2, the operand blocks of step s + 1
// (loaded two steps earlier) are transposed/split into stage (s + 1) % 2 and the global loads of
// step s + 3 are issued into the register set that just became free.  Two register sets per
// operand keep two steps of global loads in flight, which covers an HBM round trip.
template <int IN, int BM, int BN, bool FAST>
__device__ __forceinline__ void tile_body(const GemmArgs& g, int64_t I0, int64_t J0, int64_t kBeg, int64_t kEnd,
                                          uint4* smem) {
    using Cfg = TileCfg<IN, BM, BN>;
    constexpr int BK = Cfg::BK, TM = Cfg::TM, TN = Cfg::TN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);

    // 128 x 128 tiles: an operand's block of a step is 128 threads' work, so threads 0 .. 127 stage A and the others B
    // (with both on the first two wavefronts, their conversion work set the time of a step: mean of a layer's launches 19.0 -> 16.7 us)
    constexpr bool SHARED = BM == 128 && BN == 128;
    const bool second = __builtin_amdgcn_readfirstlane(tid >> 7) != 0;
    Fetch<IN, BM, FAST> fa;
    Fetch<IN, BN, FAST> fb;
    if (SHARED) {
        fa.init(second ? g.B : g.A, second ? g.ldb : g.lda, second ? J0 : I0, second ? g.N : g.M, kBeg, kEnd, tid & 127);
    } else {
        fa.init(g.A, g.lda, I0, g.M, kBeg, kEnd, tid);
        fb.init(g.B, g.ldb, J0, g.N, kBeg, kEnd, tid);
    }
    const int fa_off = (SHARED && second) ? Cfg::A_CHUNKS : 0;

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // LDS chunk offsets of this lane's MFMA operands inside one k-block pair
    int offa[TM], offb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) offa[i] = (lane >> 5) * BM + swz(wm0 + 32 * i + (lane & 31));
#pragma unroll
    for (int j = 0; j < TN; ++j) offb[j] = (lane >> 5) * BN + swz(wn0 + 32 * j + (lane & 31));

    const int64_t steps = (kEnd - kBeg + BK - 1) / BK;
    // Register sets for global loads in flight: the 256 x 256 tile has room for one step only, the
    // smaller tiles keep two steps in flight (four were measured and change nothing: their calls are
    // bound by the operand stream, 6 TB/s summed over the workgroups, not by its latency).
    constexpr int NSETS = (BM == 256 && BN == 256) ? 1 : 2;
    constexpr bool TWO_SETS = NSETS > 1;
    if (TWO_SETS) {
        Staged ra[NSETS], rb[SHARED ? 1 : NSETS];       // set u holds steps u + 1, u + 1 + NSETS, ...
        if (steps > 0) {
            fa.load(ra[0], kEnd);
            if (!SHARED) fb.load(rb[0], kEnd);
            fa.store(ra[0], smem + fa_off);
            if (!SHARED) fb.store(rb[0], smem + Cfg::A_CHUNKS);
#pragma unroll
            for (int u = 0; u < NSETS; ++u)
                if (steps > u + 1) {
                    fa.load(ra[u], kEnd);
                    if (!SHARED) fb.load(rb[SHARED ? 0 : u], kEnd);
                }
        }
        __syncthreads();
        for (int64_t s0 = 0; s0 < steps; s0 += NSETS) {
#pragma unroll
            for (int u = 0; u < NSETS; ++u) {
                const int64_t s = s0 + u;
                if (s < steps) {
                    // NSETS is even, so the LDS stage of step s is u & 1
                    const uint4* sa = smem + (u & 1) * Cfg::STAGE_CHUNKS;
                    uint4* da = smem + ((u + 1) & 1) * Cfg::STAGE_CHUNKS;
                    mfma_step<IN, BM, BN, TM, TN>(acc, sa, sa + Cfg::A_CHUNKS, offa, offb);
                    if (s + 1 < steps) {
                        fa.store(ra[u], da + fa_off);
                        if (!SHARED) fb.store(rb[SHARED ? 0 : u], da + Cfg::A_CHUNKS);
                        if (s + 1 + NSETS < steps) {
                            fa.load(ra[u], kEnd);
                            if (!SHARED) fb.load(rb[SHARED ? 0 : u], kEnd);
                        }
                    }
                    __syncthreads();
                }
            }
        }
    } else {
        Staged a0, b0;
        if (steps > 0) {
            fa.load(a0, kEnd);
            fb.load(b0, kEnd);
            fa.store(a0, smem);
            fb.store(b0, smem + Cfg::A_CHUNKS);
            if (steps > 1) { fa.load(a0, kEnd); fb.load(b0, kEnd); }
        }
        __syncthreads();
        for (int64_t s = 0; s < steps; ++s) {
            const uint4* sa = smem + (s & 1) * Cfg::STAGE_CHUNKS;
            uint4* da = smem + ((s + 1) & 1) * Cfg::STAGE_CHUNKS;
            mfma_step<IN, BM, BN, TM, TN>(acc, sa, sa + Cfg::A_CHUNKS, offa, offb);
            if (s + 1 < steps) {
                fa.store(a0, da);
                fb.store(b0, da + Cfg::A_CHUNKS);
                if (s + 2 < steps) { fa.load(a0, kEnd); fb.load(b0, kEnd); }
            }
            __syncthreads();
        }
    }

    tile_epilogue<TM, TN, BM == 128 && BN == 128>(g, acc, I0 + wm0, J0 + wn0, lane);
}

// ---------------------------------------------------------------------------------------------
// The 256 x 128 tile (or 128 x 256) of the fp32 forms on eight wavefronts (two per SIMD, 64 x 64 each).  A K step is about as much
// conversion (fp32 -> bf16 terms, about six instructions per element) as MFMA work, and with one wavefront per SIMD the two follow
// one another; with two, one converts while the other multiplies.  A thread stages R rows (4 of A, 2 of B, of a k-block of
// 8) x 4 columns of an operand, so a chunk of LDS is filled by 8 / R threads.  Measured on T S (us, four -> eight wavefronts):
// 4096 x 4096 281 -> 223, 14336 x 4096 1101 -> 776, 4096 x 11008 2056 -> 1454.  The 128 x 128 tile keeps four wavefronts:
// its launches are a few K steps long, and more wavefronts only lengthen their start (mean at 4096 channels 16.6 -> 18.8).
template <int IN, int BMN, int R, bool FAST>
struct FetchRows {
    static constexpr int GROUPS = BMN / 4, UNITS = GROUPS * (32 / R), NP = InTraits<IN>::NP;
    const char* p;      // address of (this thread's first row in the next step, first column)
    const char* plast;  // same columns in the last valid row (FAST)
    int64_t ld_bytes, k;
    int cg, kr;         // column group, first row inside a step
    int ncols;
    bool vec_ok;

    __device__ __forceinline__ void init(const void* base, int64_t ld, int64_t mn0, int64_t MN, int64_t k0, int64_t kEnd, int unit) {
        // neighbouring threads fill one chunk, so that a wavefront's stores cover whole chunks of consecutive banks
        constexpr int SUB = 8 / R;
        cg = (unit / SUB) % GROUPS;
        kr = (unit / (SUB * GROUPS)) * 8 + (unit % SUB) * R;
        int64_t col = mn0 + (int64_t)cg * 4;
        const int64_t rem = MN - col;
        ncols = rem >= 4 ? 4 : (rem > 0 ? (int)rem : 0);
        k = k0 + kr;
        ld_bytes = ld * 4;
        if (FAST && ncols != 4) col = 0;                  // never stored to C
        p = (const char*)base + k * ld_bytes + col * 4;
        plast = (const char*)base + (kEnd - 1) * ld_bytes + col * 4;
        vec_ok = FAST || ((((uintptr_t)p & 15) == 0) && ((ld_bytes & 15) == 0) && ncols == 4);
    }

    __device__ __forceinline__ void load(uint4 (&r)[R], int64_t kEnd) {
        if (FAST) {
            if (k + R <= kEnd) {
#pragma unroll
                for (int j = 0; j < R; ++j) r[j] = *(const uint4*)(p + j * ld_bytes);
            } else {
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const bool ok = k + j < kEnd;
                    const uint4 v = *(const uint4*)(ok ? p + j * ld_bytes : plast);
                    r[j] = ok ? v : make_uint4(0u, 0u, 0u, 0u);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                r[j] = make_uint4(0u, 0u, 0u, 0u);
                if (k + j < kEnd) {
                    const char* q = p + j * ld_bytes;
                    if (vec_ok) {
                        r[j] = *(const uint4*)q;
                    } else {
                        uint32_t w[4] = {0u, 0u, 0u, 0u};
                        for (int e = 0; e < ncols; ++e) w[e] = *(const uint32_t*)(q + 4 * e);
                        r[j] = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                }
            }
        }
        p += 32 * ld_bytes;
        k += 32;
    }

    __device__ __forceinline__ void store(const uint4 (&r)[R], uint4* lds) const {
        const float* x = (const float*)r;                 // x[4 j + c]: row j, column c
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint32_t t[NP][R / 2];
#pragma unroll
            for (int q = 0; q < R / 2; ++q) {
                float u = x[4 * (2 * q) + c], v = x[4 * (2 * q + 1) + c];
#pragma unroll
                for (int n = 0; n < NP; ++n) {            // the next term is what the ones before it leave (exact differences)
                    t[n][q] = bf16_pair(u, v);
                    u -= __uint_as_float(t[n][q] << 16);
                    v -= __uint_as_float(t[n][q] & 0xFFFF0000u);
                }
            }
            char* pos = (char*)(lds + (kr >> 3) * BMN + swz(cg * 4 + c)) + (kr & 7) * 2;
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                char* q = pos + n * 4 * BMN * 16;
                if (R == 4) *(uint2*)q = make_uint2(t[n][0], t[n][R / 2 - 1]);
                else *(uint32_t*)q = t[n][0];
            }
        }
    }
};

constexpr int kWideThreads = 512;

// C += alpha * acc for a wavefront's part that nobody else touches.  Parts inside C skip the tests per entry, which cost more than the
// loads and stores (13 -> 7 us for a launch of one 128 x 256 tile and one K step), and a row of blocks is loaded at once.
template <int TM, int TN>
__device__ __forceinline__ void tile_epilogue_add(const GemmArgs& g, f32x16_t (&acc)[TM][TN], int64_t I0, int64_t J0, int lane) {
    float* base = g.C + (I0 + 4 * (lane >> 5)) * g.ldc + J0 + (lane & 31);
    if (I0 + 32 * TM <= g.M && J0 + 32 * TN <= g.N) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float old[TN][16];
#pragma unroll
            for (int e = 0; e < 16; ++e)
#pragma unroll
                for (int j = 0; j < TN; ++j) old[j][e] = base[(int64_t)(8 * (e >> 2) + (e & 3)) * g.ldc + 32 * j];
#pragma unroll
            for (int e = 0; e < 16; ++e)
#pragma unroll
                for (int j = 0; j < TN; ++j) base[(int64_t)(8 * (e >> 2) + (e & 3)) * g.ldc + 32 * j] = old[j][e] + g.alpha * acc[i][j][e];
            base += 32 * g.ldc;
        }
        return;
    }
    // at the edge: loads from the nearest entry inside, so that they still are in flight together
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = J0 + 32 * j + (lane & 31), rbase = I0 + 32 * i + 4 * (lane >> 5);
            float* cbase = g.C + (col < g.N ? col : g.N - 1);
            float old[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t r = rbase + 8 * (e >> 2) + (e & 3);
                old[e] = cbase[(r < g.M ? r : g.M - 1) * g.ldc];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (col >= g.N) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t r = rbase + 8 * (e >> 2) + (e & 3);
                if (r < g.M) cbase[r * g.ldc] = old[e] + g.alpha * acc[i][j][e];
            }
        }
}

template <int IN, int BM, int BN, bool FAST, bool ADD = false>
__device__ __forceinline__ void tile_body_wide(const GemmArgs& g, int64_t I0, int64_t J0, int64_t kBeg, int64_t kEnd, uint4* smem) {
    static_assert(BM * BN == 256 * 128 && BM + BN == 384, "256 x 128 or 128 x 256");
    constexpr int TM = 2, TN = 2, RA = BM / 64, RB = BN / 64;
    using Cfg = TileCfg<IN, BM, BN>;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = wave / (BN / 64) * 64, wn0 = wave % (BN / 64) * 64;
    FetchRows<IN, BM, RA, FAST> fa;
    FetchRows<IN, BN, RB, FAST> fb;
    fa.init(g.A, g.lda, I0, g.M, kBeg, kEnd, tid);
    fb.init(g.B, g.ldb, J0, g.N, kBeg, kEnd, tid);

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    int offa[TM], offb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) offa[i] = (lane >> 5) * BM + swz(wm0 + 32 * i + (lane & 31));
#pragma unroll
    for (int j = 0; j < TN; ++j) offb[j] = (lane >> 5) * BN + swz(wn0 + 32 * j + (lane & 31));

    const int64_t steps = (kEnd - kBeg + Cfg::BK - 1) / Cfg::BK;
    uint4 ra[2][RA], rb[2][RB];                           // set u holds steps u + 1, u + 3, ...
    if (steps > 0) {
        fa.load(ra[0], kEnd);
        fb.load(rb[0], kEnd);
        fa.store(ra[0], smem);
        fb.store(rb[0], smem + Cfg::A_CHUNKS);
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (steps > u + 1) { fa.load(ra[u], kEnd); fb.load(rb[u], kEnd); }
    }
    __syncthreads();
    for (int64_t s0 = 0; s0 < steps; s0 += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t s = s0 + u;
            if (s < steps) {
                const uint4* sa = smem + u * Cfg::STAGE_CHUNKS;
                uint4* da = smem + (u ^ 1) * Cfg::STAGE_CHUNKS;
                auto convert = [&]() {
                    if (s + 1 < steps) {
                        fa.store(ra[u], da);
                        fb.store(rb[u], da + Cfg::A_CHUNKS);
                        if (s + 3 < steps) { fa.load(ra[u], kEnd); fb.load(rb[u], kEnd); }
                    }
                };
                // the two wavefronts of a SIMD start a step with different halves of its work
                const bool convert_first = (wave >> 2) != 0;
                if (convert_first) convert();
                mfma_step<IN, BM, BN, TM, TN>(acc, sa, sa + Cfg::A_CHUNKS, offa, offb);
                if (!convert_first) convert();
                __syncthreads();
            }
        }
    }
    if constexpr (ADD) tile_epilogue_add<TM, TN>(g, acc, I0 + wm0, J0 + wn0, lane);
    else tile_epilogue<TM, TN, false>(g, acc, I0 + wm0, J0 + wn0, lane);
}

}  // namespace
