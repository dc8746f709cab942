// Persistent FP32 and mixed sweeps for networks between the register-resident kernels of
// fpi_mixed.hip (128 PQ buses) and kMaxMidBuses, where one workgroup still holds a batch of
// columns: their injections in LDS, their drops U = V - w and last injections in
// registers, and the operator streamed from L2 in fragment order by every sweep.
//
// As kernels of their own per sweep (fpi_large.hip) these networks moved their state,
// injections and operands through HBM four times a sweep, waited on three launches per
// sweep, and queued launches up to max_iter (300 buses, mixed FP16: 8.26 ms for 210,240
// columns and 0.50 ms for 1,000; here 3.20 and 0.11 ms).  Here S is read and V written once.  The
// iterates, the per-column schedule and the results are those of that path bit for bit
// (mixed_steps.h); columns of a batch may be at different stages, so a sweep runs the
// 16-bit product for the 16-column groups that have a column wanting it and the FP32 product
// likewise.
//
// Bound: the FP32 product by the matrix cores (a column needs about one; 57,000 cycles of a
// batch's 195,000 at 299 buses), the 16-bit products by the operator's way from L2 (0.73 MB
// per batch and sweep, 11,000 cycles), the injections by vector instructions (8,000 per
// sweep; cycles of a build that took 3.55 ms).  Two workgroups of 16 columns per CU (128
// registers, spills) took 3.76 ms instead of those.
#include <type_traits>

#include "mixed_steps.h"

namespace tpf {

namespace {

constexpr int kMidWaves = 8, kMidTiles = 5;  // 16-row tiles per wave: n <= 8 * 40
static_assert(kMaxMidBuses <= 8 * kMidWaves * kMidTiles, "a wave's tiles");

// Odd multiples of four dwords between columns: the fragments' reads touch every LDS bank.
__host__ __device__ constexpr int mid_stride32(int n) { return 4 * (((2 * n + 15) / 16 * 4) | 1); }
__host__ __device__ constexpr int mid_stride16(int n) { return 8 * (((2 * n + 31) / 32 * 4) | 1); }

struct MidColumn {
    long long col;  // -1: none
    int live;       // still sweeping
    MixState m;
};

// Columns set aside.  A batch sweeps until its slowest column ends, and every sweep streams the
// whole operator for it, so once at most half of its columns have been left over for kFewSweeps
// sweeps (columns of alike loads end within two of each other), they are written to the
// workgroup's own pool in the workspace and the next columns are taken; a pool that holds a
// batch's worth is swept as a batch of its own, as is what is left at the end.  A column resumes
// where it stopped: drops, last injections and schedule state.  60,000 columns of 199 buses of
// which 0, 1, 3, 10 and 30 % are infeasible (100 sweeps each), mixed FP16: 0.68, 3.1, 3.2, 4.3
// and 8.2 ms, against 0.70, 4.9, 8.6, 14.2 and 16.7 when every batch waits for its slowest and
// 1.9, 7.6, 7.9, 8.7 and 12.7 as kernels per sweep; with an eighth of the batch for a half 4.9 and
// 13.5 ms at 10 and 30 %.
constexpr int kFewLive = 16, kFewSweeps = 3, kPoolColumns = 32 + kFewLive;

// A workgroup's pool: [kPoolColumns][2][16 MT] drops and last injections, [kPoolColumns] MidColumn.
__host__ __device__ constexpr size_t mid_pool_bytes(int n) {
    return ((size_t)kPoolColumns * (2 * ((2 * n + 15) / 16 * 16) * 4 + sizeof(MidColumn)) + 255) / 256 * 256;
}
// Workgroups that have one: at most one workgroup is resident per CU (for its registers), and
// without a second batch there is nothing to take instead.
constexpr int kPools = 256;
inline int mid_pools(int64_t tau) { return (int)std::min<int64_t>(kPools, (tau + 63) / 64); }
constexpr size_t kMidQueueBytes = 256;

template <int MODE, int CG, bool ZIP, typename IO>
__global__ __launch_bounds__(kMidWaves * 64) __attribute__((amdgpu_waves_per_eu(2))) void fpi_mid_kernel(
    const IO *__restrict__ S, IO *__restrict__ Vout, int32_t *__restrict__ iters_out, int8_t *__restrict__ status_out,
    const IO *__restrict__ V0, const f4x *__restrict__ A32, const uint4 *__restrict__ A16,
    const double *__restrict__ w, int n, int sZ, float zscale, const ZipShares zs_, long long tau, double tol,
    int max_iter, unsigned long long *__restrict__ queue, unsigned char *__restrict__ pools, int pool_count) {
    constexpr bool kMixed = MODE != TPF_MODE_FP32;
    constexpr int LM = kMixed ? MODE : TPF_MODE_MIXED_BF16;  // (unused for FP32)
    constexpr int NC = 16 * CG, NT = kMidWaves * 64, TPW = kMidTiles;
    const ZipShares zs = ZIP ? zs_ : ZipShares{nullptr, nullptr, nullptr};
    const int MT = (2 * n + 15) / 16;             // 16-row tiles
    const int K4 = MT;                            // groups of four FP32 k-steps (16 k values)
    const int KS = (2 * n + 31) / 32;             // 16-bit k-steps
    const int st32 = mid_stride32(n), st16 = mid_stride16(n);

    const __amdgpu_buffer_rsrc_t R32 =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<f4x *>(A32), 0, MT * K4 * 1024, 0x00027000);
    const __amdgpu_buffer_rsrc_t R16 =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(A16), 0, MT * KS * 1024, 0x00027000);

    extern __shared__ __align__(16) unsigned char smem[];
    float *B32 = reinterpret_cast<float *>(smem);                               // [NC][st32] last injections
    uint32_t *B16 = reinterpret_cast<uint32_t *>(B32 + NC * st32);              // [NC][st16 / 2] (mixed)
    f4x *wf = reinterpret_cast<f4x *>(B16 + (kMixed ? NC * st16 / 2 : 0));      // [MT][4] w in FP32, per tile and lane group
    MidColumn *cs = reinterpret_cast<MidColumn *>(wf + 4 * MT);                 // [NC]
    unsigned long long *mx = reinterpret_cast<unsigned long long *>(cs + NC);   // [NC] max step^2 as double bits
    unsigned *um = reinterpret_cast<unsigned *>(mx + NC);                       // [NC] max |U|
    int *bd = reinterpret_cast<int *>(um + NC);                                 // [NC] non-finite step / loads / start
    float *sm = reinterpret_cast<float *>(bd + 2 * NC);                         // [NC] max |S|
    unsigned long long *qb = reinterpret_cast<unsigned long long *>(sm + NC);   // [1]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;

    if constexpr (kMixed)
        for (int e = tid; e < NC * st16 / 2; e += NT) B16[e] = 0u;
    for (int e = tid; e < 16 * MT; e += NT) reinterpret_cast<float *>(wf)[e] = e < 2 * n ? (float)w[e] : (e & 1 ? 0.0f : 1.0f);

    // The lane's place, made anew by each phase: the compiler would keep the addresses that
    // every phase derives from it in registers through the products, and spill the state.
    struct Place {
        int g, j;
    };
    auto place = [&]() __attribute__((always_inline)) {
        Place p{lane >> 4, lane & 15};
        asm volatile("" : "+v"(p.g), "+v"(p.j));
        return p;
    };
    // w read where it is used: hoisted out of the sweep loop it would take 40 registers
    auto w_now = [&]() __attribute__((always_inline)) {
        const double *p = w;
        asm volatile("" : "+s"(p));
        return p;
    };
    // the mixed forms read the loads in FP32, the FP32 form as given
    typedef std::conditional_t<kMixed, float, IO> SX;
    typedef SX s4 __attribute__((ext_vector_type(4)));
    f4x U[CG][TPW];
    s4 Sx[CG][TPW];
    bool first = true;
    // pool of this workgroup (CG = 2: with 16 columns it has one batch only)
    const bool pooled = CG == 2 && (int)blockIdx.x < pool_count;
    float *pool = reinterpret_cast<float *>(pools + (size_t)blockIdx.x * mid_pool_bytes(n));
    MidColumn *pool_cs = reinterpret_cast<MidColumn *>(pool + (size_t)kPoolColumns * 2 * 16 * MT);
    int held = 0;         // columns in it
    bool packed = false;  // the batch came from it
    bool drained = false; // no new batch is left

    // Forms the injections of every live column from the current drops and writes the operand
    // of its next sweep.
    auto prepare = [&]() __attribute__((always_inline)) {
        const double *w = w_now();
        const auto [g, j] = place();
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            const MidColumn *k = cs + 16 * c + j;
            const bool live = k->live, low = kMixed && live && !k->m.want;
            const int ph = k->m.ph;
            const float ks = k->m.ks;
            const bool any_low = __ballot(low) != 0;
            if (__ballot(live) == 0) continue;
            // No branch per bus or tile (past the last bus loads and drops are zero and w is 1,
            // which gives a zero injection): the chains of a lane's buses overlap.
            f4x in[TPW];
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                const int t = min(wave + kMidWaves * q, MT - 1);
                const f4x wq = wf[4 * t + g];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int b = min(8 * t + 2 * g + h, n - 1);
                    float2 iz;
                    if constexpr (kMixed)
                        iz = mixed_injection(Sx[c][q][2 * h], Sx[c][q][2 * h + 1], wq[2 * h], wq[2 * h + 1],
                                             U[c][q][2 * h], U[c][q][2 * h + 1], zs, b);
                    else
                        iz = full_injection((double)Sx[c][q][2 * h], (double)Sx[c][q][2 * h + 1], w[2 * b],
                                            w[2 * b + 1], U[c][q][2 * h], U[c][q][2 * h + 1], zs, b);
                    in[q][2 * h] = iz.x;
                    in[q][2 * h + 1] = iz.y;
                }
            }
            if constexpr (kMixed) {
                if (any_low) {
                    f4x was[TPW];
#pragma unroll
                    for (int q = 0; q < TPW; ++q)
                        was[q] = *reinterpret_cast<const f4x *>(B32 + (16 * c + j) * st32 +
                                                                16 * min(wave + kMidWaves * q, MT - 1) + 4 * g);
                    uint2 o[TPW];
#pragma unroll
                    for (int q = 0; q < TPW; ++q) {
                        f4x d;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float diff = rounded_difference(in[q][e], was[q][e]);
                            d[e] = ph ? diff : in[q][e];
                        }
                        o[q].x = Low16<LM>::enc2(d[0] * ks, d[1] * ks);
                        o[q].y = Low16<LM>::enc2(d[2] * ks, d[3] * ks);
                    }
                    if (low) {
#pragma unroll
                        for (int q = 0; q < TPW; ++q)
                            if (wave + kMidWaves * q < MT)
                                *reinterpret_cast<uint2 *>(
                                    B16 + ((16 * c + j) * st16 + 16 * (wave + kMidWaves * q) + 4 * g) / 2) = o[q];
                    }
                }
            }
            if (live) {
#pragma unroll
                for (int q = 0; q < TPW; ++q)
                    if (wave + kMidWaves * q < MT)
                        *reinterpret_cast<f4x *>(B32 + (16 * c + j) * st32 + 16 * (wave + kMidWaves * q) + 4 * g) = in[q];
            }
        }
    };

    // A batch's rows of S, V0 and V are contiguous in memory but scattered over the lanes: they
    // pass through the FP32 operand's place (free between batches) with whole-line accesses,
    // all columns at once in complex64, half of them at a time in complex128.  (Loads of each
    // lane's buses from the rows themselves, 64-byte pieces, took 75,000 cycles per batch and
    // 24,000 per sweep against 12,000 for a 16-bit product.)
    typedef IO pair __attribute__((ext_vector_type(2)));
    constexpr int kParts = sizeof(IO) / 4, CP = NC / kParts;
    pair *stage = reinterpret_cast<pair *>(B32);  // [CP][n]
    auto rows_here = [&](long long base, int p) {
        const long long left = tau - base - (long long)CP * p;
        return (int)(left < 0 ? 0 : left < CP ? left : CP);
    };
    auto fetch_rows = [&](const IO *src, long long base, auto use) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            const int count = rows_here(base, p) * n;
            const pair *from = reinterpret_cast<const pair *>(src) + (base + CP * p) * n;
            __syncthreads();
            for (int e0 = tid; e0 < count; e0 += 8 * NT) {
                pair v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (e0 + u * NT < count) v[u] = __builtin_nontemporal_load(from + e0 + u * NT);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (e0 + u * NT < count) stage[e0 + u * NT] = v[u];
            }
            __syncthreads();
            const auto [g, j] = place();
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                const int k = 16 * c + j - CP * p;  // row of the stage
                if (k < 0 || k >= CP || base + 16 * c + j >= tau) continue;
#pragma unroll
                for (int q = 0; q < TPW; ++q)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int b = 8 * (wave + kMidWaves * q) + 2 * g + h;
                        if (b < n) use(c, q, h, b, stage[k * n + b]);
                    }
            }
        }
        __syncthreads();
    };
    auto store_rows = [&](long long base) __attribute__((always_inline)) {
        const double *w = w_now();
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            __syncthreads();
            const auto [g, j] = place();
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                const int k = 16 * c + j - CP * p;
                if (k < 0 || k >= CP) continue;
#pragma unroll
                for (int q = 0; q < TPW; ++q)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int b = 8 * (wave + kMidWaves * q) + 2 * g + h;
                        if (b < n)
                            stage[k * n + b] = pair{(IO)(w[2 * b] + (double)U[c][q][2 * h]),
                                                    (IO)(w[2 * b + 1] + (double)U[c][q][2 * h + 1])};
                    }
            }
            __syncthreads();
            const int count = rows_here(base, p) * n;
            pair *to = reinterpret_cast<pair *>(Vout) + (base + CP * p) * n;
            for (int e = tid; e < count; e += NT) __builtin_nontemporal_store(stage[e], to + e);
        }
        __syncthreads();
    };

    // The same for the columns in cs, wherever their rows are (batches of set-aside columns and
    // batches that set some aside).
    auto store_columns = [&]() __attribute__((always_inline)) {
        const double *w = w_now();
        const auto [g, j] = place();
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            const long long col = cs[16 * c + j].col;
            if (col < 0) continue;
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int b = 8 * (wave + kMidWaves * q) + 2 * g + h;
                    if (b < n)
                        reinterpret_cast<pair *>(Vout)[col * n + b] = pair{(IO)(w[2 * b] + (double)U[c][q][2 * h]),
                                                                           (IO)(w[2 * b + 1] + (double)U[c][q][2 * h + 1])};
                }
        }
    };
    // bit k: column k of the batch is live (uniform)
    auto live_mask = [&]() __attribute__((always_inline)) {
        unsigned m = 0;
#pragma unroll
        for (int c = 0; c < CG; ++c) m |= (unsigned)(__ballot(cs[16 * c + j].live) & 0xffff) << (16 * c);
        return m;
    };
    // Sets the live columns aside, as they are between a sweep and the forming of its injections.
    auto set_aside = [&](unsigned mask) __attribute__((always_inline)) {
        const auto [g, j] = place();
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            const int k = 16 * c + j;
            if (!(mask >> k & 1)) continue;
            float *to = pool + (size_t)(held + __popc(mask & ((1u << k) - 1u))) * 2 * 16 * MT;
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                const int t = wave + kMidWaves * q;
                if (t >= MT) continue;
                *reinterpret_cast<f4x *>(to + 16 * t + 4 * g) = U[c][q];
                if constexpr (kMixed)
                    *reinterpret_cast<f4x *>(to + 16 * MT + 16 * t + 4 * g) =
                        *reinterpret_cast<const f4x *>(B32 + k * st32 + 16 * t + 4 * g);
            }
        }
        if (tid < NC && (mask >> tid & 1)) pool_cs[held + __popc(mask & ((1u << tid) - 1u))] = cs[tid];
        held += __popc(mask);
        __syncthreads();
        if (tid < NC && (mask >> tid & 1)) cs[tid].col = -1, cs[tid].live = 0;
        __syncthreads();
    };
    // The last columns set aside, up to a batch of them.
    auto resume = [&]() __attribute__((always_inline)) {
        const int count = held < NC ? held : NC;
        held -= count;
        if (tid < NC) {
            mx[tid] = 0ull;
            um[tid] = 0u;
            bd[tid] = 0;
            cs[tid].col = -1;
            cs[tid].live = 0;
            if (tid < count) cs[tid] = pool_cs[held + tid];
        }
        __syncthreads();
        const auto [g, j] = place();
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            const int k = 16 * c + j;
            const long long col = cs[k].col;
            const float *from = pool + (size_t)(held + k) * 2 * 16 * MT;
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                const int t = wave + kMidWaves * q;
                U[c][q] = f4x{0, 0, 0, 0};
                Sx[c][q] = s4{0, 0, 0, 0};
                if (k >= count || t >= MT) continue;
                U[c][q] = *reinterpret_cast<const f4x *>(from + 16 * t + 4 * g);
                if constexpr (kMixed)
                    *reinterpret_cast<f4x *>(B32 + k * st32 + 16 * t + 4 * g) =
                        *reinterpret_cast<const f4x *>(from + 16 * MT + 16 * t + 4 * g);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int b = 8 * t + 2 * g + h;
                    if (b >= n) continue;
                    const pair v = reinterpret_cast<const pair *>(S)[col * n + b];
                    Sx[c][q][2 * h] = (SX)v.x;
                    Sx[c][q][2 * h + 1] = (SX)v.y;
                }
            }
        }
        packed = true;
        prepare();
        __syncthreads();
    };

    // Loads the next batch (loads, start voltages, schedule state); false when none is left.
    long long base = 0;
    auto refill = [&]() -> bool {
        const double *w = w_now();
        if (tid < NC) {
            mx[tid] = 0ull;
            um[tid] = 0u;
            bd[tid] = bd[NC + tid] = 0;
            sm[tid] = 0.0f;
        }
        // the first batches are dealt by block; when they are all, the queue is not touched
        // (nor cleared by the launch)
        const unsigned long long dealt = (unsigned long long)NC * gridDim.x;
        if (tid == 0)
            *qb = first                                 ? (unsigned long long)NC * blockIdx.x
                  : dealt >= (unsigned long long)tau ? (unsigned long long)tau
                                                      : dealt + atomicAdd(queue, (unsigned long long)NC);
        first = false;
        __syncthreads();
        base = (long long)*qb;
        if (base >= tau) return false;
        packed = false;
        const auto [g, j] = place();
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int b = 8 * (wave + kMidWaves * q) + 2 * g + h;
                    Sx[c][q][2 * h] = Sx[c][q][2 * h + 1] = 0;
                    U[c][q][2 * h] = U[c][q][2 * h + 1] = 0.0f;
                    if (b < n) {
                        U[c][q][2 * h] = (float)(1.0 - w[2 * b]);
                        U[c][q][2 * h + 1] = (float)(0.0 - w[2 * b + 1]);
                    }
                }
        float smax[CG];
        int sbad[CG];
#pragma unroll
        for (int c = 0; c < CG; ++c) smax[c] = 0.0f, sbad[c] = 0;
        fetch_rows(S, base, [&](int c, int q, int h, int, const pair &v) __attribute__((always_inline)) {
            const double sr = fabs((double)v.x), si = fabs((double)v.y);
            sbad[c] |= !(sr + si < HUGE_VAL);
            smax[c] = fmaxf(smax[c], (float)fmax(sr, si));
            Sx[c][q][2 * h] = (SX)v.x;
            Sx[c][q][2 * h + 1] = (SX)v.y;
        });
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            // (non-negative floats order like their bit patterns)
            atomicMax(reinterpret_cast<int *>(sm) + 16 * c + j, __float_as_int(smax[c]));
            if (sbad[c]) bd[16 * c + j] = 1;
        }
        if (V0) {
            int vbad[CG];
#pragma unroll
            for (int c = 0; c < CG; ++c) vbad[c] = 0;
            fetch_rows(V0, base, [&](int c, int q, int h, int b, const pair &v) __attribute__((always_inline)) {
                const double vr = (double)v.x, vi = (double)v.y, m2 = vr * vr + vi * vi;
                vbad[c] |= (m2 >= 0.25 && m2 <= 2.25) ? 0 : 1;
                U[c][q][2 * h] = (float)(vr - w[2 * b]);
                U[c][q][2 * h + 1] = (float)(vi - w[2 * b + 1]);
            });
#pragma unroll
            for (int c = 0; c < CG; ++c)
                if (vbad[c]) bd[NC + 16 * c + j] = 1;
            __syncthreads();
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                if (bd[NC + 16 * c + j]) {  // the guard failed somewhere in the column: flat start
#pragma unroll
                    for (int q = 0; q < TPW; ++q)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int b = 8 * (wave + kMidWaves * q) + 2 * g + h;
                            if (b < n) {
                                U[c][q][2 * h] = (float)(1.0 - w[2 * b]);
                                U[c][q][2 * h + 1] = (float)(0.0 - w[2 * b + 1]);
                            }
                        }
                }
            }
        }
        __syncthreads();
        if (tid < NC) {
            MidColumn k;
            k.col = base + tid < tau ? base + tid : -1;
            k.live = k.col >= 0;
            float s = sm[tid];
            s *= zscale;
            k.m = mixed_start<LM>(s, bd[tid], sZ);
            cs[tid] = k;
            bd[tid] = 0;  // from here on: a step that is not finite
        }
        __syncthreads();
        prepare();
        __syncthreads();
        return true;
    };

    // Products of the column groups [G0, G0 + GN) for the wave's tiles.
    auto product32 = [&](auto G0, auto GN, f4x(&acc)[CG][TPW]) __attribute__((always_inline)) {
        constexpr int g0 = decltype(G0)::value, gn = decltype(GN)::value;
        const auto [g, j] = place();
#pragma unroll
        for (int q = 0; q < TPW; ++q)
#pragma unroll
            for (int c = g0; c < g0 + gn; ++c) acc[c][q] = f4x{0, 0, 0, 0};
        // tile q of the wave (past the last tile: the last one again, unused)
        auto fetch = [&](int q, int k) __attribute__((always_inline)) {
            const int t = min(wave + kMidWaves * q, MT - 1);
            return __builtin_bit_cast(f4x,
                                      __builtin_amdgcn_raw_buffer_load_b128(R32, 16 * lane, (t * K4 + k) * 1024, 0));
        };
        f4x a[2][TPW];
#pragma unroll
        for (int q = 0; q < TPW; ++q) a[0][q] = fetch(q, 0);
        const float *Bp = B32 + j * st32 + g;
        for (int k = 0; k < K4; k += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (k + u < K4) {
                    const int nx = k + u + 1 < K4 ? k + u + 1 : k + u;
#pragma unroll
                    for (int q = 0; q < TPW; ++q) a[u ^ 1][q] = fetch(q, nx);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
#pragma unroll
                        for (int c = g0; c < g0 + gn; ++c) {
                            const float b = Bp[16 * c * st32 + 16 * (k + u) + 4 * e];
#pragma unroll
                            for (int q = 0; q < TPW; ++q)
                                acc[c][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][q][e], b, acc[c][q], 0, 0, 0);
                        }
                    }
                }
            }
        }
    };
    auto product16 = [&](auto G0, auto GN, f4x(&acc)[CG][TPW]) __attribute__((always_inline)) {
        constexpr int g0 = decltype(G0)::value, gn = decltype(GN)::value;
        const auto [g, j] = place();
#pragma unroll
        for (int q = 0; q < TPW; ++q)
#pragma unroll
            for (int c = g0; c < g0 + gn; ++c) acc[c][q] = f4x{0, 0, 0, 0};
        auto fetch = [&](int q, int s) __attribute__((always_inline)) {
            const int t = min(wave + kMidWaves * q, MT - 1);
            return __builtin_bit_cast(uint4,
                                      __builtin_amdgcn_raw_buffer_load_b128(R16, 16 * lane, (t * KS + s) * 1024, 0));
        };
        uint4 a[2][TPW];
#pragma unroll
        for (int q = 0; q < TPW; ++q) a[0][q] = fetch(q, 0);
        const uint32_t *Bp = B16 + (j * st16 + 8 * g) / 2;
        for (int s = 0; s < KS; s += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (s + u < KS) {
                    const int nx = s + u + 1 < KS ? s + u + 1 : KS - 1;
#pragma unroll
                    for (int q = 0; q < TPW; ++q) a[u ^ 1][q] = fetch(q, nx);
#pragma unroll
                    for (int c = g0; c < g0 + gn; ++c) {
                        const uint4 b = *reinterpret_cast<const uint4 *>(Bp + (16 * c * st16 + 32 * (s + u)) / 2);
#pragma unroll
                        for (int q = 0; q < TPW; ++q) acc[c][q] = Low16<LM>::mma(a[u][q], b, acc[c][q]);
                    }
                }
            }
        }
    };

    if (!refill()) return;
    int few = 0;  // sweeps since few columns are left of the batch
    while (true) {
        // which products the groups need (uniform: every wave holds all columns in its lanes)
        bool low[CG], full[CG];
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            const MidColumn *k = cs + 16 * c + j;
            const bool live = k->live, want = !kMixed || k->m.want;
            low[c] = kMixed && __ballot(live && !want) != 0;
            full[c] = __ballot(live && want) != 0;
        }
        std::integral_constant<int, 0> i0;
        std::integral_constant<int, 1> i1;
        std::integral_constant<int, CG> ic;
        if constexpr (kMixed) {
            f4x acc[CG][TPW];
            auto update = [&](int c) __attribute__((always_inline)) {
                const MidColumn *k = cs + 16 * c + j;
                if (!k->live || k->m.want) return;
                const int ph = k->m.ph;
                const float inv = k->m.inv;
                float emax = 0.f, umx = 0.f;
                int bad = 0;
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    if (wave + kMidWaves * q >= MT) continue;  // (rows past the last bus are zero)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float2 nu = low_update(acc[c][q][2 * h], acc[c][q][2 * h + 1],
                                                     make_float2(U[c][q][2 * h], U[c][q][2 * h + 1]), ph, inv, emax, umx,
                                                     bad);
                        U[c][q][2 * h] = nu.x;
                        U[c][q][2 * h + 1] = nu.y;
                    }
                }
                atomicMax(mx + 16 * c + j, (unsigned long long)__double_as_longlong((double)emax));
                atomicMax(um + 16 * c + j, __float_as_uint(umx));
                if (bad) bd[16 * c + j] = 1;
            };
            if (CG == 2 && low[0] && low[CG - 1]) {
                product16(i0, ic, acc);
                update(0);
                update(CG - 1);
            } else if (low[0]) {
                product16(i0, i1, acc);
                update(0);
            } else if (CG == 2 && low[CG - 1]) {
                product16(std::integral_constant<int, CG - 1>{}, i1, acc);
                update(CG - 1);
            }
        }
        {
            f4x acc[CG][TPW];
            auto update = [&](int c) __attribute__((always_inline)) {
                const MidColumn *k = cs + 16 * c + j;
                if (!k->live || (kMixed && !k->m.want)) return;
                double emax = 0.0;
                int bad = 0;
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    if (wave + kMidWaves * q >= MT) continue;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float2 nu = full_update(acc[c][q][2 * h], acc[c][q][2 * h + 1],
                                                      make_float2(U[c][q][2 * h], U[c][q][2 * h + 1]), emax, bad);
                        U[c][q][2 * h] = nu.x;
                        U[c][q][2 * h + 1] = nu.y;
                    }
                }
                atomicMax(mx + 16 * c + j, (unsigned long long)__double_as_longlong(emax));
                if (bad) bd[16 * c + j] = 1;
            };
            if (CG == 2 && full[0] && full[CG - 1]) {
                product32(i0, ic, acc);
                update(0);
                update(CG - 1);
            } else if (full[0]) {
                product32(i0, i1, acc);
                update(0);
            } else if (CG == 2 && full[CG - 1]) {
                product32(std::integral_constant<int, CG - 1>{}, i1, acc);
                update(CG - 1);
            }
        }
        __syncthreads();  // maxima complete; every wave is done with the operands
        if (tid < NC && cs[tid].live) {
            MidColumn k = cs[tid];
            const double e = __longlong_as_double((long long)mx[tid]);
            bool conv;
            if constexpr (kMixed) {
                conv = mixed_schedule<LM>(k.m, k.m.want != 0, (float)sqrt(e), __uint_as_float(um[tid]), (float)tol);
            } else {
                k.m.it += 1;
                conv = sqrt(e) < tol;
            }
            const int bad = bd[tid];
            if (bad || conv || k.m.it >= max_iter) {
                iters_out[k.col] = k.m.it;
                status_out[k.col] = bad ? TPF_ST_NONFINITE : (conv ? TPF_ST_CONVERGED : TPF_ST_MAX_ITER);
                k.live = 0;  // its drops stay as they are until the batch is stored
            }
            cs[tid] = k;
            mx[tid] = 0ull;
            um[tid] = 0u;
            bd[tid] = 0;
        }
        __syncthreads();
        const unsigned mask = live_mask();
        if (mask && __popc(mask) <= kFewLive) ++few;
        const bool aside = pooled && mask && few >= kFewSweeps && !drained && base + NC < tau;
        if (mask && !aside) {
            prepare();
            __syncthreads();
            continue;
        }
        // the batch is done, or left to its last few
        if (aside) set_aside(mask);
        if (packed || aside)
            store_columns();
        else
            store_rows(base);
        __syncthreads();
        few = 0;
        if (held < NC && !drained) {
            if (refill()) continue;
            drained = true;
        }
        if (held == 0) break;
        resume();
    }
}

size_t mid_lds(int n, int CG, bool mixed) {
    const int NC = 16 * CG, MT = (2 * n + 15) / 16;
    return (size_t)NC * mid_stride32(n) * 4 + (mixed ? (size_t)NC * mid_stride16(n) * 2 : 0) + (size_t)MT * 64 +
           NC * (sizeof(MidColumn) + 8 + 4 + 8 + 4) + 16;
}

template <int MODE, int CG, bool ZIP, typename IO>
int launch_as(const tpf_network_s &net, const DeviceNet &dn, const void *S, int64_t tau, double tol, int max_iter,
              const void *V0, void *V, int32_t *iters, int8_t *status, void *workspace, hipStream_t st) {
    auto *queue = static_cast<unsigned long long *>(workspace);
    const size_t lds = mid_lds(net.n, CG, MODE != TPF_MODE_FP32);
    auto k = fpi_mid_kernel<MODE, CG, ZIP, IO>;
    if (hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return fail(TPF_ERR_DEVICE, "hipFuncSetAttribute failed");
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kMidWaves * 64, lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    const int64_t blocks = std::min<int64_t>((int64_t)num_cus() * per_cu, (tau + 16 * CG - 1) / (16 * CG));
    if (16 * CG * blocks < tau) {  // the batches past the first come from the queue
        const int rc = launch_zero_u64(queue, 1, st);
        if (rc != TPF_OK) return rc;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kMidWaves * 64), lds, st, (const IO *)S, (IO *)V, iters, status,
                       (const IO *)V0, reinterpret_cast<const f4x *>(dn.AM32),
                       reinterpret_cast<const uint4 *>(MODE == TPF_MODE_MIXED_BF16 ? dn.AMbf : dn.AMh), dn.wl, net.n,
                       dn.sZ, dn.aP ? dn.zscale : 1.0f, ZipShares{dn.aP, dn.aI, dn.aZ}, (long long)tau, tol, max_iter,
                       queue, static_cast<unsigned char *>(workspace) + kMidQueueBytes, mid_pools(tau));
    return TPF_OK;
}

// Batches of 32 columns share a product's way through the operator (300 buses, 210,240
// columns: mixed FP16 3.20 ms against 4.01 with 16, FP32 6.61 and 7.02); 16 go to more CUs when the columns do not fill
// the chip anyway.
template <int MODE, typename IO>
int launch_io(const tpf_network_s &net, const DeviceNet &dn, const void *S, int64_t tau, double tol, int max_iter,
              const void *V0, void *V, int32_t *iters, int8_t *status, void *workspace, hipStream_t st) {
    const bool one = tau <= 16 * (int64_t)num_cus();
    if (dn.aP)
        return one ? launch_as<MODE, 1, true, IO>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, workspace, st)
                   : launch_as<MODE, 2, true, IO>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, workspace, st);
    return one ? launch_as<MODE, 1, false, IO>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, workspace, st)
               : launch_as<MODE, 2, false, IO>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, workspace, st);
}

}  // namespace

size_t mid_workspace_bytes(int n, int64_t tau) { return kMidQueueBytes + (size_t)mid_pools(tau) * mid_pool_bytes(n); }

int launch_fpi_mid(const tpf_network_s &net, const DeviceNet &dn, int mode, const void *S, int dtype, int64_t tau,
                   double tol, int max_iter, const void *V0, void *V, int32_t *iters, int8_t *status,
                   void *workspace, hipStream_t st) {
    if (!dn.AM32) return fail(TPF_ERR_UNSUPPORTED, "mid-size operator not staged");
#define TPF_MODE_CASE(M)                                                                                       \
    if (mode == M)                                                                                             \
        return dtype == TPF_C128                                                                               \
                   ? launch_io<M, double>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, workspace, st)     \
                   : launch_io<M, float>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, workspace, st);
    TPF_MODE_CASE(TPF_MODE_FP32)
    TPF_MODE_CASE(TPF_MODE_MIXED_BF16)
    TPF_MODE_CASE(TPF_MODE_MIXED_FP16)
#undef TPF_MODE_CASE
    return fail(TPF_ERR_INVALID_ARG, "unknown mode");
}

}  // namespace tpf
