// Householder tridiagonalisation of a symmetric fp64 matrix of up to 4096 rows with the matrix on the chip, for the middle of the
// chain in spectrum.hip: from a few hundred to 4096 rows left down to the last 256.
//
// One launch per column reads the trailing matrix from the last-level cache (8 (k - j)^2 bytes) and pays a kernel boundary and the
// serial tail of the workgroup that finishes last: 20 us per column at k = 4096.  Here 256 workgroups, one per compute unit, keep
// the matrix in registers and LDS from the first column to the last, and a column costs one exchange between them.
//
// Rows and columns are numbered so that the last one is 4095.  Workgroup w owns the rows 1024 g + 4 w .. + 3 (g = 0 .. 3, sixteen
// slots; four at a time because what it publishes is then 64 bytes in a row, which arrive 1 to 1.7 us earlier than four times 16 bytes
// in lines shared with other workgroups) and its thread t the columns t + 512 q (q = 0 .. 7) of every one of them.  It is done with its
// last row.  The rows that live longest are in registers (nine slots and an eighth, 146 of 256 registers per thread), the next five in
// LDS (156 KB), and the first two slots, which only a matrix of more than 3072 rows has, stay in memory.
// Step j, with the reflector u of row j - 1 not yet normalised and the pair (v, w) of the step before not yet applied:
//   pass      x -= v w^T + w v^T on the own rows, on the way the sums x u of every row and |u|^2;
//   barrier   every row's (x u, x[row, j]) is published; meanwhile alpha, v = u - alpha e_j, tau;
//   exchange  everybody reads all of them: by symmetry x[:, j] is row j, and p = x v = x u - alpha x[:, j];
//   barrier   v^T p, hence w = tau p - (tau^2 / 2)(v^T p) v and the next u = x[j, :] - v_j w - w_j v.
// Everybody computes v, w and u in full, so nothing else has to travel.
//
// The exchange needs no flags: an entry is 16 bytes that hold a NaN of a pattern no computation makes until they are written, and
// readers ask again until the pattern is gone.  Three buffers rotate; an owner of rows that are left restores the pattern in the buffer
// of step j - 1 once it has read all of step j (whose entries their owners wrote after they had read step j - 1), and everybody who
// could read that buffer again, in step j + 2, has first to see the owner's entry of step j + 1, which is written behind it.
//
// All workgroups have to run at the same time.  The cooperative launch only sees to it that they would fit an empty device: work of other
// streams or processes keeps the last ones out until it leaves a compute unit to them.  So the workgroups count themselves in before
// anything is written, and whoever has waited a second or so for the rest calls it off (one word decides, so all agree); the kernel of one
// workgroup behind this one (rescue) then does these columns, in seconds instead of milliseconds, with nothing to wait for.  Past that gate an entry is
// as late as its owner's pass.  A reader that gives up on one all the same, after two million attempts, marks the computation broken, and then
// the last kernel of the chain makes all of d and e NaN, which no caller takes for a spectrum.
// The gate and the second launch: whole spectra of k = 326: 968 -> 976 us, 700 and more within what runs differ.
//
// What bounds it: the exchange, 2.0 us at 1024 columns left and 4.2 at 4096 (every workgroup reads 16 bytes per column past its L2), then
// the pass, 768 fp64 operations per thread at 4096 columns.  A column costs 2.8 us while at most 1024 are left, 5 on average at
// k = 4096.  Whole spectra: k = 700: 5.2 -> 1.9 ms, 1030: 9.2 -> 3.1, 2049: 24.0 -> 7.1, 4096: 82 -> 23.8.
// Callers that overlap wait for each other here, and are still served sooner.  One spectrum on each of 1, 2, 4, 8 streams, ms, a launch per column -> this: k = 700: 5.3, 5.5,
// 6.2, 11.9 -> 2.0, 2.4, 4.6, 9.0; 1000: 8.8, 9.3, 11, 22 -> 2.9, 4.7, 8.6, 17; 2048: 23, 27, 54, 73 -> 7.0, 13, 25, 51.  One-token decode on
// a stream beside spectra of k = 700: median 27 -> 30 us, of k = 4096: 17 -> 2.4 ms (longest 44 -> 22).
#include <math.h>

#include <type_traits>

#include "aser_internal.h"
#include "tridiag_resident.h"
#include "wave_f64.h"

namespace {

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512, kWaves = kThreads / 64, kGroups = 256, kCols = 8, kSlots = 16;
constexpr int kMemSlots = 2, kLdsChunks = 39, kRegSlots = 10;
// where the columns of chunk q of slot s are: a chunk of 512 doubles in LDS, or else, behind the slots in memory, a register
__host__ __device__ constexpr int lds_chunk(int s, int q) { return (s - kMemSlots) * 8 + q; }
__host__ __device__ constexpr bool in_lds(int s, int q) { return s >= kMemSlots && lds_chunk(s, q) < kLdsChunks; }
__host__ __device__ constexpr int row_of(int s, int w) { return 4 * kGroups * (s >> 2) + 4 * w + (s & 3); }
__host__ __device__ constexpr int reg_slot(int s) { return s < 16 - kRegSlots ? 0 : s - (16 - kRegSlots); }
constexpr int kSide = kGroups * kSlots;                   // 4096
constexpr int kTail = kAserTridiagTail;
constexpr int kMaxTries = 1 << 21;                        // a launch argument instead makes 114 registers spill, not 22
constexpr uint64_t kOff = 1ull << 63;                     // in the word of arrivals: called off
constexpr uint64_t kEmpty = 0x7ff8a5e25eed0001ull;        // fp32 inputs widened leave the low 29 bits of a NaN's payload zero
static_assert(!in_lds(8, 0) && !in_lds(7, 0) && kRegSlots == 10, "the dynamic LDS holds slots below 8 only");
static_assert(kSide == kThreads * kCols && kSide == kAserResidentMost && kTail % 4 == 0, "rows and columns");

// The entries of the columns [512 (8 - N), 4096) of this step, N per thread; loads and their wait in one block.
template <int N>
__device__ __forceinline__ void fetch(u32x4_t (&v)[kCols], const uint32_t (&off)[kCols], const uint64_t* buf) {
#define ASER_LD(d, o) "global_load_dwordx4 %" #d ", %" #o ", %"
    if constexpr (N == 1)
        asm volatile(ASER_LD(0, 1) "2 sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v[7]) : "v"(off[7]), "s"(buf) : "memory");
    else if constexpr (N == 2)
        asm volatile(ASER_LD(0, 2) "4 sc1\n\t" ASER_LD(1, 3) "4 sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v[6]), "=&v"(v[7]) : "v"(off[6]), "v"(off[7]), "s"(buf) : "memory");
    else if constexpr (N == 3)
        asm volatile(ASER_LD(0, 3) "6 sc1\n\t" ASER_LD(1, 4) "6 sc1\n\t" ASER_LD(2, 5) "6 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]) : "v"(off[5]), "v"(off[6]), "v"(off[7]), "s"(buf) : "memory");
    else if constexpr (N == 4)
        asm volatile(ASER_LD(0, 4) "8 sc1\n\t" ASER_LD(1, 5) "8 sc1\n\t" ASER_LD(2, 6) "8 sc1\n\t" ASER_LD(3, 7) "8 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]) : "v"(off[4]), "v"(off[5]), "v"(off[6]), "v"(off[7]), "s"(buf) : "memory");
    else if constexpr (N == 5)
        asm volatile(ASER_LD(0, 5) "10 sc1\n\t" ASER_LD(1, 6) "10 sc1\n\t" ASER_LD(2, 7) "10 sc1\n\t" ASER_LD(3, 8) "10 sc1\n\t" ASER_LD(4, 9) "10 sc1\n\t"
                     "s_waitcnt vmcnt(0)"
                     : "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                     : "v"(off[3]), "v"(off[4]), "v"(off[5]), "v"(off[6]), "v"(off[7]), "s"(buf) : "memory");
    else if constexpr (N == 6)
        asm volatile(ASER_LD(0, 6) "12 sc1\n\t" ASER_LD(1, 7) "12 sc1\n\t" ASER_LD(2, 8) "12 sc1\n\t" ASER_LD(3, 9) "12 sc1\n\t" ASER_LD(4, 10) "12 sc1\n\t"
                     ASER_LD(5, 11) "12 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                     : "v"(off[2]), "v"(off[3]), "v"(off[4]), "v"(off[5]), "v"(off[6]), "v"(off[7]), "s"(buf) : "memory");
    else if constexpr (N == 7)
        asm volatile(ASER_LD(0, 7) "14 sc1\n\t" ASER_LD(1, 8) "14 sc1\n\t" ASER_LD(2, 9) "14 sc1\n\t" ASER_LD(3, 10) "14 sc1\n\t" ASER_LD(4, 11) "14 sc1\n\t"
                     ASER_LD(5, 12) "14 sc1\n\t" ASER_LD(6, 13) "14 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                     : "v"(off[1]), "v"(off[2]), "v"(off[3]), "v"(off[4]), "v"(off[5]), "v"(off[6]), "v"(off[7]), "s"(buf) : "memory");
    else
        asm volatile(ASER_LD(0, 8) "16 sc1\n\t" ASER_LD(1, 9) "16 sc1\n\t" ASER_LD(2, 10) "16 sc1\n\t" ASER_LD(3, 11) "16 sc1\n\t" ASER_LD(4, 12) "16 sc1\n\t"
                     ASER_LD(5, 13) "16 sc1\n\t" ASER_LD(6, 14) "16 sc1\n\t" ASER_LD(7, 15) "16 sc1\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                     : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "v"(off[4]), "v"(off[5]), "v"(off[6]), "v"(off[7]), "s"(buf) : "memory");
#undef ASER_LD
}

__device__ __forceinline__ bool is_empty(unsigned lo, unsigned hi) { return lo == (unsigned)kEmpty && hi == (unsigned)(kEmpty >> 32); }

// Asks for the N entries of this thread until all have been written; false after too many attempts.
template <int N>
__device__ __forceinline__ bool wait_for(u32x4_t (&v)[kCols], const uint32_t (&off)[kCols], const uint64_t* buf) {
    for (int tries = 0; tries < kMaxTries; ++tries) {
        fetch<N>(v, off, buf);
        bool there = true;
#pragma unroll
        for (int q = kCols - N; q < kCols; ++q) there = there && !is_empty(v[q][0], v[q][1]) && !is_empty(v[q][2], v[q][3]);
        if (there) return true;
    }
    return false;
}

__device__ __forceinline__ void publish2(uint64_t* at, uint64_t x, uint64_t y) {
    const u32x4_t v = {(unsigned)x, (unsigned)(x >> 32), (unsigned)y, (unsigned)(y >> 32)};
    asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(at), "v"(v) : "memory");
}
__device__ __forceinline__ uint64_t entry_bits(double x) {          // never the pattern of an unwritten entry
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    return b == kEmpty ? 0x7ff8000000000000ull : b;
}
__device__ __forceinline__ double as_double(unsigned lo, unsigned hi) { return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo); }

// Entries of p, of w and of the next u.  Rows and columns each compute their own copy, and the copies have to agree to the last bit: a difference
// between them is a matrix that is no similarity of the old one, and grows by a factor of the size of vj kk - wj per step.
__device__ __forceinline__ double entry_of_p(double alpha, double s, double x) { return fma(-alpha, x, s); }
__device__ __forceinline__ double entry_of_w(double tau, double kk, double p, double v) { return fma(-kk, v, tau * p); }
__device__ __forceinline__ double entry_of_u(double vj, double wj, double x, double w, double v) { return fma(-wj, v, fma(-vj, w, x)); }

// The ring, and behind it the word of arrivals and the mark of a broken computation.
__device__ __forceinline__ uint64_t* arrivals(const AserTridiagResident& a) { return a.ring + 6 * (a.k - a.c0 + 3); }
__global__ void resident_clear_kernel(AserTridiagResident a) {
    const int64_t words = 6 * (a.k - a.c0 + 3);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words + 2; i += (int64_t)gridDim.x * 256) a.ring[i] = i < words ? kEmpty : 0;
}

// Counts this workgroup in and waits for the others: true in all of them, or false in all of them.  (No attempts at all: false.)
__device__ __forceinline__ bool all_here(const AserTridiagResident& a) {
    uint64_t* const word = arrivals(a);
    if (a.gate_attempts == 0) __hip_atomic_fetch_or(word, kOff, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t seen = __hip_atomic_fetch_add(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    for (int tries = 0; seen < kGroups; ++tries) {        // with the mark it is not less
        if (tries < a.gate_attempts) {
            __builtin_amdgcn_s_sleep(1);
            seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (__hip_atomic_compare_exchange_strong(word, &seen, seen | kOff, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            return false;                                 // otherwise `seen` is new: it changes no more than once per workgroup
        }
    }
    return (seen & kOff) == 0;
}

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void tridiag_resident_kernel(AserTridiagResident a) {
    extern __shared__ double low[];                       // [kLdsChunks][kThreads], when the matrix has such rows
    __shared__ double part[kWaves][kSlots], n2part[kWaves], dotpart[kWaves], rowv[kSlots], rowp[kSlots], colj[kSlots], near[6];
    __shared__ int failed, here;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), w = blockIdx.x;
    const int64_t k = a.k, base = k - kSide;              // row i here is row i + base of the matrix
    const int first = (int)(a.c0 - base);
    const int ring0 = first & ~3, turn_words = 2 * (kSide - ring0);
    double* const Bo = a.B + base * k + base;             // only rows and columns from `first` on are looked at
    if (tid == 0) {
        failed = a.broken;
        here = all_here(a);
    }
    lds_barrier();
    if (!here) return;
    double m[kRegSlots][kCols], u[kCols], v[kCols], wv[kCols];
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        const int i = row_of(s, w);
#pragma unroll
        for (int q = 0; q < kCols; ++q) {
            const int l = tid + kThreads * q;
            if (s < kMemSlots) continue;
            if (!in_lds(s, q)) m[reg_slot(s)][q] = (i >= first && l >= first) ? Bo[(int64_t)i * k + l] : 0.0;
            else if (i >= first) low[lds_chunk(s, q) * kThreads + tid] = l >= first ? Bo[(int64_t)i * k + l] : 0.0;
        }
    }
#pragma unroll
    for (int q = 0; q < kCols; ++q) {
        const int l = tid + kThreads * q;
        const bool in = l >= first;
        u[q] = in ? a.vn[base + l] : 0.0;
        v[q] = (in && a.vp) ? a.vp[base + l] : 0.0;
        wv[q] = (in && a.vp) ? a.wp[base + l] : 0.0;
    }
    // lane s of the first wavefront looks after slot s
    const bool owner = tid < kSlots;
    const int row = row_of(lane, w);                      // of an owner
    double ur = 0.0;                                      // u in that row
    if (owner) {
        const bool in = row >= first;
        ur = in ? a.vn[base + row] : 0.0;
        rowv[lane] = (in && a.vp) ? a.vp[base + row] : 0.0;
        rowp[lane] = (in && a.vp) ? a.wp[base + row] : 0.0;
    }
    double tau = 1.0, kk = 0.0;                           // w in a row is tau rowp - kk rowv
    double x0 = lane_value(a.vn[a.c0], 0);                // u in row j
    const double tau_in = lane_value(*a.tau, 0);
    lds_barrier();

    double alpha = 0.0, v0 = 0.0;
    auto norms = [&](auto tag) {                          // |u|^2 of this wavefront's columns
        double n2 = 0.0;
#pragma unroll
        for (int q = decltype(tag)::value; q < kCols; ++q) n2 = fma(u[q], u[q], n2);
        n2 = wave_sum(n2);
        if (lane == 0) n2part[wave] = n2;
    };
    auto reflector = [&](bool given) {                    // the reflector of u as a whole: v0 in row j, alpha, tau
        const double n2 = lane_value(((n2part[0] + n2part[1]) + (n2part[2] + n2part[3])) + ((n2part[4] + n2part[5]) + (n2part[6] + n2part[7])), 0);
        const double root = sqrt(n2);
        alpha = lane_value((x0 > 0.0) ? -root : root, 0);           // lane_value: the same in all threads, kept in scalar registers
        v0 = lane_value(x0 - alpha, 0);
        const double vn2 = n2 - x0 * x0 + v0 * v0;
        tau = lane_value(vn2 > 0.0 ? 2.0 * rcp_f64(vn2) : 0.0, 0);
        if (given) { alpha = 0.0; v0 = x0; tau = tau_in; }
    };

    // The steps whose column lies in chunk Q0: the columns of earlier chunks and the rows of earlier groups of four slots are gone, and
    // the later groups are all there, so the pass is straight-line code but for four slots.
    int j = first;
    bool finished = false;
    auto steps = [&](auto tag) -> bool {
        constexpr int Q0 = decltype(tag)::value, N = kCols - Q0, S0 = 4 * (Q0 / 2);
        constexpr int stop = kThreads * (Q0 + 1) < kSide - kTail ? kThreads * (Q0 + 1) : kSide - kTail;
        for (; j < stop; ++j) {
            norms(tag);
            // ---- pass over the own rows
            const bool mine = tid == j % kThreads;        // the thread of column j
            const double vrow = rowv[lane & (kSlots - 1)], wrow = entry_of_w(tau, kk, rowp[lane & (kSlots - 1)], vrow);   // of slot `lane`
            unsigned t = tid;
            asm volatile("" : "+v"(t));                   // keeps the addresses from being carried along in registers
            auto group = [&](auto from_tag) {             // eight slots
                constexpr int from = decltype(from_tag)::value;
                double acc[8];
#pragma unroll
                for (int s = from; s < from + 8; ++s) {
                    acc[s - from] = 0.0;
                    if (s < S0 || (s < S0 + 4 && row_of(s, w) < j)) continue;
                    const double vr = lane_value(vrow, s), wr = lane_value(wrow, s);
                    auto element = [&](double x, int q) {
                        x = fma(-vr, wv[q], x);
                        x = fma(-wr, v[q], x);
                        acc[s - from] = fma(x, u[q], acc[s - from]);
                        return x;
                    };
                    if (s < kMemSlots) {
                        double* const at = Bo + (int64_t)row_of(s, w) * k;     // the same for all threads
#pragma unroll
                        for (int c = 0; c < kCols; c += 4) {
                            double x[4];
#pragma unroll
                            for (int q = c > Q0 ? c : Q0; q < c + 4; ++q) x[q - c] = (q > Q0 || tid + kThreads * q >= j) ? (at + kThreads * q)[t] : 0.0;
#pragma unroll
                            for (int q = c > Q0 ? c : Q0; q < c + 4; ++q) {
                                x[q - c] = element(x[q - c], q);
                                if (q > Q0 || tid + kThreads * q >= j) (at + kThreads * q)[t] = x[q - c];
                                if (q == Q0 && mine) colj[s] = x[q - c];
                            }
                        }
                    } else {
#pragma unroll
                        for (int c = Q0 & ~3; c < kCols; c += 4) {     // four chunks at a time: the registers have room for no more
                            double x[4];
#pragma unroll
                            for (int q = c > Q0 ? c : Q0; q < c + 4; ++q)
                                if (in_lds(s, q)) x[q - c] = low[lds_chunk(s, q) * kThreads + tid];
#pragma unroll
                            for (int q = c > Q0 ? c : Q0; q < c + 4; ++q) {
                                if (in_lds(s, q)) {
                                    low[lds_chunk(s, q) * kThreads + tid] = element(x[q - c], q);
                                } else {
                                    double& y = m[reg_slot(s)][q];
                                    y = element(y, q);
                                    asm volatile("" : "+v"(y));
                                }
                            }
                            asm volatile("" : "+v"(acc[s - from]));    // these pins keep the compiler from putting rows off, whose operands it then spills
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);    // the registers are full: nothing of another row is begun early
                }
                if (mine) {
#pragma unroll
                    for (int s = from; s < from + 8; ++s)
                        if (s >= S0 && s >= kMemSlots && !in_lds(s, Q0)) colj[s] = m[reg_slot(s)][Q0];
                }
                double s0, s1;
                eight_sums(acc, s0, s1);
                if ((lane & 15) == 0) {
                    part[wave][from + eight_sums_index(lane)] = s0;
                    part[wave][from + eight_sums_index(lane) + 4] = s1;
                }
            };
            if constexpr (S0 < 8) group(std::integral_constant<int, 0>{});
            group(std::integral_constant<int, 8>{});
            lds_barrier();
            // ---- this workgroup's rows of x u and of column j
            const int turn = (j - first) % 3;
            uint64_t* const buf = a.ring + turn * turn_words;
            double sr = 0.0, ar = 0.0;
            const bool have = owner && row >= j;
            if (have) {
                double g[kWaves];
#pragma unroll
                for (int q = 0; q < kWaves; ++q) g[q] = part[q][lane];
                sr = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7]));
                ar = Q0 < 4 && in_lds(lane, Q0) ? low[lds_chunk(lane, Q0) * kThreads + j % kThreads] : colj[lane];
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // the pattern restored in the last step is in place
                publish2(buf + 2 * (row - ring0), entry_bits(sr), entry_bits(ar));
            }
            if (row_of(kSlots - 1, w) <= j) {             // no row is left: nothing of what the others publish matters here
                finished = true;
                return false;
            }
            reflector(j == first);
            if (have) {
                if (row == j) ur = v0;
                rowv[lane] = ur;
                rowp[lane] = entry_of_p(alpha, sr, ar);
            }
#pragma unroll
            for (int q = Q0; q < kCols; ++q) v[q] = (q == Q0 && mine) ? v0 : u[q];
            if (a.vstore && w == kGroups - 1 - (j & 31) && j != first) {
                double* const at = a.vstore + (base + j - 1) * k + base;
                unsigned t = tid;
                asm volatile("" : "+v"(t));
#pragma unroll
                for (int q = Q0; q < kCols; ++q)
                    if (tid + kThreads * q >= j) (at + kThreads * q)[t] = v[q];
                if (tid == 0) a.taustore[base + j - 1] = tau;
            }
            // ---- everybody's
            u32x4_t e[kCols];
            uint32_t off[kCols];
#pragma unroll
            for (int q = Q0; q < kCols; ++q) {
                const int l = tid + kThreads * q;
                off[q] = 16 * (uint32_t)((l > j ? l : j) - ring0);      // a column of the past: any entry that will be written
            }
            if (!wait_for<N>(e, off, buf)) failed = 1;
            double dot = 0.0;
#pragma unroll
            for (int q = Q0; q < kCols; ++q) {
                const int l = tid + kThreads * q;
                const double x = l >= j ? as_double(e[q][2], e[q][3]) : 0.0;
                const double p = entry_of_p(alpha, l >= j ? as_double(e[q][0], e[q][1]) : 0.0, x);
                wv[q] = p;
                u[q] = x;
                dot = fma(v[q], p, dot);
                if (q == Q0 && mine) { near[0] = p; near[1] = v[q]; near[2] = x; }
                if (q <= Q0 + 1 && l == j + 1) { near[3] = p; near[4] = v[q]; near[5] = x; }
            }
            dot = wave_sum(dot);
            if (lane == 0) dotpart[wave] = dot;
            lds_barrier();
            if (failed) return false;
            dot = ((dotpart[0] + dotpart[1]) + (dotpart[2] + dotpart[3])) + ((dotpart[4] + dotpart[5]) + (dotpart[6] + dotpart[7]));
            kk = lane_value(0.5 * tau * tau * dot, 0);
            const double vj = lane_value(near[1], 0), wj = lane_value(entry_of_w(tau, kk, near[0], vj), 0);
            x0 = lane_value(entry_of_u(vj, wj, near[5], entry_of_w(tau, kk, near[3], near[4]), near[4]), 0);
#pragma unroll
            for (int q = Q0; q < kCols; ++q) {
                wv[q] = entry_of_w(tau, kk, wv[q], v[q]);
                const double next = entry_of_u(vj, wj, u[q], wv[q], v[q]);
                u[q] = (q > Q0 || tid + kThreads * q > j) ? next : 0.0;
            }
            if (have) {
                ur = entry_of_u(vj, wj, ar, entry_of_w(tau, kk, entry_of_p(alpha, sr, ar), ur), ur);
                publish2(a.ring + (turn == 0 ? 2 : turn - 1) * turn_words + 2 * (row - ring0), kEmpty, kEmpty);
            }
            if (w == kGroups - 1 && tid == 0) {
                if (j != first) a.e[base + j - 1] = alpha;
                a.d[base + j] = near[2] - 2.0 * vj * wj;
            }
        }
        return true;
    };
    const bool done = steps(std::integral_constant<int, 0>{}) && steps(std::integral_constant<int, 1>{}) && steps(std::integral_constant<int, 2>{}) &&
                      steps(std::integral_constant<int, 3>{}) && steps(std::integral_constant<int, 4>{}) && steps(std::integral_constant<int, 5>{}) &&
                      steps(std::integral_constant<int, 6>{}) && steps(std::integral_constant<int, 7>{});
    if (finished) return;
    if (!done) {                                          // gave up
        if (tid == 0) __hip_atomic_store(aser_tridiag_broken(a), (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    // ---- the last 256 rows, with the reflector that is due and the pair that has not been applied, go back to memory
    norms(std::integral_constant<int, kCols - 1>{});
    lds_barrier();
    reflector(false);
    const int l = tid + kThreads * (kCols - 1);
    if (l >= j) {
        const double vn = l == j ? v0 : u[kCols - 1];
#pragma unroll
        for (int s = kSlots - 4; s < kSlots; ++s) Bo[(int64_t)row_of(s, w) * k + l] = m[reg_slot(s)][kCols - 1];
        if (w == kGroups - 1) {
            a.vn_out[base + l] = vn;
            a.vp_out[base + l] = v[kCols - 1];
            a.wp_out[base + l] = wv[kCols - 1];
            if (a.vstore) a.vstore[(base + j - 1) * k + base + l] = vn;
        }
    }
    if (w == kGroups - 1 && tid == 0) {
        *a.tau_out = tau;
        a.e[base + j - 1] = alpha;
        if (a.vstore) a.taustore[base + j - 1] = tau;
    }
}

// The same columns in one workgroup, where the gate was called off; otherwise it leaves at once.  B in memory, the vectors of a step in LDS; a wavefront
// takes a row at a time.  Bound by what one compute unit reads and writes: whole spectra of k = 326, 700, 1030, 2049, 4096
// in 2.3, 27, 107, 850 and 6700 ms.
constexpr int kRescueThreads = 1024;
__global__ __launch_bounds__(kRescueThreads) void tridiag_rescue_kernel(AserTridiagResident a) {
    extern __shared__ double vecs[];                      // entry i: row and column c0 + i
    __shared__ double red[2][kRescueThreads / 64];
    if ((*arrivals(a) & kOff) == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rest = (int)(a.k - a.c0);
    double *const u = vecs, *const v = u + rest, *const w = v + rest, *const p = w + rest;      // the reflector, the pair B lacks, B u
    double* const Bo = a.B + a.c0 * a.k + a.c0;
    for (int i = tid; i < rest; i += kRescueThreads) {
        u[i] = a.vn[a.c0 + i];
        v[i] = a.vp ? a.vp[a.c0 + i] : 0.0;
        w[i] = a.vp ? a.wp[a.c0 + i] : 0.0;
    }
    double tau = *a.tau;
    auto sum = [&](double x, double* r) {                 // over the workgroup
        x = wave_sum(x);
        if (lane == 0) r[wave] = x;
        __syncthreads();
        double s = 0.0;
        for (int g = 0; g < kRescueThreads / 64; ++g) s += r[g];
        return s;
    };
    __syncthreads();
    for (int j = 0; j < rest - kTail; ++j) {
        for (int i = j + wave; i < rest; i += kRescueThreads / 64) {
            double* const row = Bo + (int64_t)i * a.k;
            const double vi = v[i], wi = w[i];
            double s = 0.0;
            for (int l = j + lane; l < rest; l += 64) {
                const double x = row[l] - (vi * w[l] + wi * v[l]);
                row[l] = x;
                s = fma(x, u[l], s);
            }
            s = wave_sum(s);
            if (lane == 0) p[i] = s;
        }
        __syncthreads();
        double dot = 0.0;
        for (int i = j + tid; i < rest; i += kRescueThreads) dot = fma(u[i], p[i], dot);
        const double kk = 0.5 * tau * tau * sum(dot, red[0]), vj = u[j], wj = tau * p[j] - kk * vj, x0 = Bo[(int64_t)j * a.k + j + 1] - (vj * (tau * p[j + 1] - kk * u[j + 1]) + wj * u[j + 1]);
        __syncthreads();                                  // u and p of rows j and j + 1 have been read
        double n2 = 0.0;
        for (int i = j + tid; i < rest; i += kRescueThreads) {
            const double ui = u[i], wi = tau * p[i] - kk * ui, x = Bo[(int64_t)j * a.k + i] - (vj * wi + wj * ui);
            v[i] = ui;
            w[i] = wi;
            if (i == j) a.d[a.c0 + j] = x;
            u[i] = i == j ? 0.0 : x;
            n2 += i == j ? 0.0 : x * x;
        }
        n2 = sum(n2, red[1]);
        const double alpha = x0 > 0.0 ? -sqrt(n2) : sqrt(n2), v0 = x0 - alpha, vn2 = n2 - x0 * x0 + v0 * v0;
        tau = vn2 > 0.0 ? 2.0 / vn2 : 0.0;
        if (tid == 0) {
            u[j + 1] = v0;
            a.e[a.c0 + j] = alpha;
            if (a.vstore) a.taustore[a.c0 + j] = tau;
        }
        __syncthreads();
        if (a.vstore)
            for (int i = j + 1 + tid; i < rest; i += kRescueThreads) a.vstore[(a.c0 + j) * a.k + a.c0 + i] = u[i];
    }
    for (int i = rest - kTail + tid; i < rest; i += kRescueThreads) {
        a.vn_out[a.c0 + i] = u[i];
        a.vp_out[a.c0 + i] = v[i];
        a.wp_out[a.c0 + i] = w[i];
    }
    if (tid == 0) *a.tau_out = tau;
}

}  // namespace

void aser_set_exchange(aser_ctx* ctx, int gate_attempts, bool broken) {
    ctx->gate_attempts = gate_attempts;
    ctx->exchange_broken = broken;
}

int aser_tridiag_resident(aser_ctx* ctx, const AserTridiagResident& a, bool* done) {
    *done = false;
    const int64_t rest = a.k - a.c0;
    if (rest <= kTail || rest > kSide) return ASER_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (ctx->stream && (hipStreamIsCapturing(ctx->stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)) {
        (void)hipGetLastError();
        return ASER_OK;
    }
    int cus = 0, coop = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, ctx->device) != hipSuccess || cus < kGroups || !coop) {
        (void)hipGetLastError();
        return ASER_OK;
    }
    const int first = (int)(kSide - rest);
    constexpr int most_lds = kLdsChunks * kThreads * (int)sizeof(double);
    const size_t lds = first < kGroups * 8 ? (size_t)most_lds : 0;
    constexpr int row_bytes = 4 * (int)sizeof(double);
    if (hipFuncSetAttribute((const void*)tridiag_resident_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most_lds) != hipSuccess ||
        hipFuncSetAttribute((const void*)tridiag_rescue_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, row_bytes * kSide) != hipSuccess) {
        (void)hipGetLastError();
        return ASER_OK;
    }
    hipLaunchKernelGGL(resident_clear_kernel, dim3(96), dim3(256), 0, ctx->stream, a);
    AserTridiagResident args = a;
    void* params[] = {&args};
    if (hipGetLastError() != hipSuccess ||
        hipLaunchCooperativeKernel((const void*)tridiag_resident_kernel, dim3(kGroups), dim3(kThreads), params, (unsigned)lds, ctx->stream) != hipSuccess) {
        (void)hipGetLastError();
        return ASER_OK;
    }
    hipLaunchKernelGGL(tridiag_rescue_kernel, dim3(1), dim3(kRescueThreads), (size_t)row_bytes * rest, ctx->stream, a);
    *done = true;
    return aser_check_launch(ctx, "tridiag_rescue");
}
