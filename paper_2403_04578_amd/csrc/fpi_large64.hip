// FP64 sweeps of networks too large for the register-resident kernel (the dense operator no
// longer fits one workgroup): each sweep of Algorithm 1 is one product kernel, whose
// epilogue updates the state and forms the next sweep's injection, and one kernel that
// applies the stopping rule and rebuilds the list of active columns.  Every sweep is queued
// without waiting on the device: the active counts stay there.
#include <type_traits>

#include "device_math.h"
#include "large_common.h"

namespace tpf {

typedef double d4x __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ d4x mma64(double a, double b, const d4x &c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---- FP64 sweeps
//
// The complex product V' = Z I + w in separate sums m1 = Zr Ir, m2 = Zi Ii and m3, with THREE as
// three real products,
//     m3 = (Zr - Zi)(Ir - Ii);  Re = m1 - m2, Im = m1 + m2 - m3,
// else m3 = Zr Ii + Zi Ir = Im (as in the register-resident kernel: a quarter fewer FP64 matrix
// products, for the networks of three_products), and the next sweep's injection formed by the
// lane that holds the new voltage, so that between two products only the lists of active
// columns are rebuilt.  The operand B[column][KB] is kept
// per column, not per place in the list, in two copies used in turn: a sweep writes one
// while other tiles still read the other.  The state x is V itself, and for complex128 it
// is the caller's output array where that can be: a column that retires is in place already.

typedef double d2x __attribute__((ext_vector_type(2)));

// I = conj(S./V) (or the ZIP form) from the new voltage of bus b.  The fused operations are
// written out here and in update64: left to the compiler, kernels that inline these may fuse
// differently, and a column's bits would depend on the kernel its call picks.
__device__ __forceinline__ d2x injection64(double sr, double si, double vr, double vi, int b, const ZipShares &zs) {
#pragma clang fp contract(off)
    const double inv = 1.0 / __builtin_fma(vr, vr, vi * vi);
    const double pr = __builtin_fma(sr, vr, si * vi), pi = __builtin_fma(sr, vi, -(si * vr));
    double jr = pr * inv, ji = pi * inv;
    if (zs.aP) {
        const double ap = zs.aP[b], ai = zs.aI[b];
        jr = __builtin_fma(ap, jr, ai * sr);
        ji = __builtin_fma(ap, ji, -(ai * si));
        if (zs.aZ) {
            const double az = zs.aZ[b];
            jr = __builtin_fma(az, pr, jr);
            ji = __builtin_fma(az, pi, ji);
        }
    }
    return d2x{jr, ji};
}

// Start voltages (guarded V0 or flat) into x and the first injections into B0; zeroes the
// K padding of the copies of B (B1 may be NULL), the column maxima and the sweep counts.  One wave
// per column.  x may be V0.
template <typename IO>
__global__ void start64_kernel(const IO *__restrict__ S, const IO *V0, int n, int KB, long long tau,
                               const ZipShares zs, double *x, d2x *__restrict__ B0,
                               d2x *__restrict__ B1, int32_t *__restrict__ iters, long long *__restrict__ act,
                               int *__restrict__ cnt, unsigned long long *__restrict__ dmax) {
    const long long c = blockIdx.x * 4LL + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= tau) return;
    int ok = V0 != nullptr;
    if (V0)
        for (int b = lane; b < n; b += 64) {
            const double vr = (double)V0[2 * (c * n + b)], vi = (double)V0[2 * (c * n + b) + 1];
            const double m2 = vr * vr + vi * vi;
            ok &= (m2 >= 0.25 && m2 <= 2.25) ? 1 : 0;
        }
    for (int off = 32; off > 0; off >>= 1) ok &= __shfl_xor(ok, off);
    for (int b = lane; b < KB; b += 64) {
        d2x inj = d2x{0.0, 0.0};
        if (b < n) {
            double vr = 1.0, vi = 0.0;
            if (ok) vr = (double)V0[2 * (c * n + b)], vi = (double)V0[2 * (c * n + b) + 1];
            reinterpret_cast<d2x *>(x)[c * n + b] = d2x{vr, vi};
            inj = injection64((double)S[2 * (c * n + b)], (double)S[2 * (c * n + b) + 1], vr, vi, b, zs);
        } else if (B1) {
            B1[c * KB + b] = inj;
        }
        B0[c * KB + b] = inj;
    }
    if (lane == 0) {
        iters[c] = 0;
        act[c] = c;
        dmax[c] = 0ull;
        if (c < 3) cnt[c] = c == 0 ? (int)tau : 0;
        if (c == 0 && tau < 3)
            for (int k = (int)tau; k < 3; ++k) cnt[k] = 0;
    }
}

// The products of entry (z, i) added to m3; zd = z.x - z.y, id = i.x - i.y.
template <bool THREE>
__device__ __forceinline__ d4x third(const d2x &z, const d2x &i, double zd, double id, const d4x &m3) {
    if constexpr (THREE) return mma64(zd, id, m3);
    return mma64(z.y, i.x, mma64(z.x, i.y, m3));
}

// Im(Z I) from the three sums.
template <bool THREE>
__device__ __forceinline__ double imaginary(double m1, double m2, double m3) {
    return THREE ? m1 + m2 - m3 : m3;
}

// One bus of one active column: V' = p + w, the step |V' - V|^2 into `dmax` (and NaN into
// `poison` when it is not finite), V' into x and the next injection into Bn (unless NULL).
template <typename IO>
__device__ __forceinline__ void update64(double pr, double pi, d2x w, long long c, int bus, int n, int KB,
                                         const IO *__restrict__ S, const ZipShares &zs, d2x old, double sr, double si,
                                         double *__restrict__ x, d2x *__restrict__ Bn, double &dmax, double &poison) {
#pragma clang fp contract(off)
    const double nr = pr + w.x, ni = pi + w.y;
    const double dr = nr - old.x, di = ni - old.y;
    const double e = __builtin_fma(dr, dr, di * di);
    poison = __builtin_fma(e, 0.0, poison);
    dmax = fmax(dmax, e);
    reinterpret_cast<d2x *>(x)[c * n + bus] = d2x{nr, ni};
    if (Bn) Bn[c * KB + bus] = injection64(sr, si, nr, ni, bus, zs);
}

// Tiles of 64 buses x 64 active columns, four waves of 32 x 32 (2 x 2 MFMA tiles, three
// accumulators each).  A: fragments [tile of 16 buses][KT k-steps of 4 buses][64 lanes]
// (Re, Im); k-slabs of two k-steps of both operands go through LDS in fragment order, two
// buffers.  Bound by the FP64 matrix cores: 24 products (1,536 cycles) per wave and slab
// against 8 KB of LDS reads; the epilogue's traffic (x, S in, x, B out) hides behind them.
template <bool THREE, typename IO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void gemm64_kernel(
    const d2x *__restrict__ A, int KT, const d2x *__restrict__ B, d2x *__restrict__ Bn, int KB,
    const long long *__restrict__ act, const int *__restrict__ na, int row_blocks, const d2x *__restrict__ w, int n,
    const IO *__restrict__ S, const ZipShares zs, double *__restrict__ x, unsigned long long *__restrict__ dmax) {
    const int nact = *na;
    const int ct = (nact + 63) / 64;
    __shared__ d2x As[2][4][128], Bs[2][4][128];  // [buffer][16-row or 16-column group][k-step, lane]
    __shared__ unsigned long long red[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, j = lane & 15;
    const int wr = (wave >> 1) * 2, wc = (wave & 1) * 2;  // first row group, first column group
    for (int t = blockIdx.x; t < ct * row_blocks; t += gridDim.x) {
        const int c0 = (t % ct) * 64, rb = t / ct;
        d4x m1[2][2], m2[2][2], m3[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) m1[a][b] = m2[a][b] = m3[a][b] = d4x{0, 0, 0, 0};
        if (tid < 64) red[tid] = 0ull;
        // A: thread copies fragments tid and tid + 256 of the slab's 512; B: two buses of one column
        const d2x *Ap = A + ((size_t)(4 * rb + (tid >> 7)) * KT) * 64 + (tid & 127);
        const size_t a2 = (size_t)2 * KT * 64;
        const int bc = tid >> 2, bk = 2 * (tid & 3);
        const int slot = c0 + bc < nact ? c0 + bc : nact - 1;
        const d2x *Bp = B + act[slot] * KB + bk;
        d2x *bdst = &Bs[0][bc >> 4][64 * (bk >> 2) + 16 * (bk & 3) + (bc & 15)];
        d2x *adst = &As[0][tid >> 7][tid & 127];
        d2x pa0 = Ap[0], pa1 = Ap[a2], pb0 = Bp[0], pb1 = Bp[1];
        adst[0] = pa0, adst[256] = pa1, bdst[0] = pb0, bdst[16] = pb1;
        __syncthreads();
        int buf = 0;
        for (int s = 0; s < KT / 2; ++s) {
            const bool more = 2 * s + 2 < KT;
            if (more) {
                Ap += 128;
                Bp += 8;
                pa0 = Ap[0], pa1 = Ap[a2], pb0 = Bp[0], pb1 = Bp[1];
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                d2x af[2], bf[2];
                double as[2], bs[2];
#pragma unroll
                for (int a = 0; a < 2; ++a) af[a] = As[buf][wr + a][64 * k + lane], as[a] = af[a].x - af[a].y;
#pragma unroll
                for (int b = 0; b < 2; ++b) bf[b] = Bs[buf][wc + b][64 * k + lane], bs[b] = bf[b].x - bf[b].y;
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        m1[a][b] = mma64(af[a].x, bf[b].x, m1[a][b]);
                        m2[a][b] = mma64(af[a].y, bf[b].y, m2[a][b]);
                        m3[a][b] = third<THREE>(af[a], bf[b], as[a], bs[b], m3[a][b]);
                    }
            }
            if (more) {  // the other buffer: its last readers passed the previous barrier
                const int o = (buf ^ 1) * 512;
                adst[o] = pa0, adst[o + 256] = pa1, bdst[o] = pb0, bdst[o + 16] = pb1;
            }
            __syncthreads();
            buf ^= 1;
        }
        // lane (g, j) holds buses g + 4 r of the row groups, column j of the column groups
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int ac = c0 + 16 * (wc + b) + j;
            const bool live = ac < nact;
            const long long c = act[live ? ac : nact - 1];
            double e = 0.0, poison = 0.0;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int bus0 = 64 * rb + 16 * (wr + a) + g;
                d2x old[4];
                double sr[4], si[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (live && bus0 + 4 * r < n) {
                        old[r] = reinterpret_cast<const d2x *>(x)[c * n + bus0 + 4 * r];
                        sr[r] = (double)S[2 * (c * n + bus0 + 4 * r)];
                        si[r] = (double)S[2 * (c * n + bus0 + 4 * r) + 1];
                    }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (live && bus0 + 4 * r < n)
                        update64<IO>(m1[a][b][r] - m2[a][b][r],
                                     imaginary<THREE>(m1[a][b][r], m2[a][b][r], m3[a][b][r]), w[bus0 + 4 * r], c,
                                     bus0 + 4 * r, n, KB, S, zs, old[r], sr[r], si[r], x, Bn, e, poison);
            }
            // non-negative doubles order like their bit patterns; ~0 marks a step that is not finite
            if (live)
                atomicMax(red + 16 * (wc + b) + j, poison == 0.0 ? (unsigned long long)__double_as_longlong(e) : ~0ull);
        }
        __syncthreads();
        if (tid < 64 && c0 + tid < nact) atomicMax(dmax + act[c0 + tid], red[tid]);
        __syncthreads();  // red is reused
    }
}

// The same sweep for batches that leave a CU fewer than six such workgroups, as 32 x 32, 64 x 32
// or 64 x 64 blocks: the operands straight from L2 through a register ring (no LDS and no barrier
// in the loop).  Every element's three sums run over the k-steps in the order of gemm64_kernel, so
// a column has the same bits whichever kernel its batch picks; splitting the k-steps among
// wavefronts is faster for a few columns (197 against 235 us for one at 999 buses) but adds the
// terms in another order.  Four wavefronts, 2 x 2, with TR x TC tiles each; 1 x 1 is bound by the
// operands' way through L1 (43 bytes per cycle and CU), 2 x 1 takes three quarters of it and 2 x 2
// half.
template <bool THREE, int TR, int TC, typename IO>
__global__ __launch_bounds__(256) void gemm64_direct_kernel(
    const d2x *__restrict__ A, int KT, const d2x *__restrict__ B, d2x *__restrict__ Bn, int KB,
    const long long *__restrict__ act, const int *__restrict__ na, int row_blocks, const d2x *__restrict__ w, int n,
    const IO *__restrict__ S, const ZipShares zs, double *__restrict__ x, unsigned long long *__restrict__ dmax) {
    constexpr int kCols = 32 * TC;  // of a workgroup's block
    constexpr int kRing = TR + TC == 2 ? 6 : TR + TC == 3 ? 4 : 3;
    const int nact = *na;
    const int ct = (nact + kCols - 1) / kCols;
    __shared__ unsigned long long red[kCols];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;
    for (int t = blockIdx.x; t < ct * row_blocks; t += gridDim.x) {
        const int cb = t / row_blocks * kCols;                      // the block's first column,
        const int c0 = cb + 16 * TC * (wave & 1);                   // the wavefront's,
        const int rt = t % row_blocks * 2 * TR + TR * (wave >> 1);  // and its first row tile
        if (tid < kCols) red[tid] = 0ull;
        const d2x *Ap[TR], *Bp[TC];
#pragma unroll
        for (int a = 0; a < TR; ++a) Ap[a] = A + (size_t)(rt + a) * KT * 64 + lane;
#pragma unroll
        for (int b = 0; b < TC; ++b) {
            const int slot = c0 + 16 * b + j;
            Bp[b] = B + act[slot < nact ? slot : nact - 1] * KB + g;
        }
        d4x m1[TR][TC], m2[TR][TC], m3[TR][TC];
#pragma unroll
        for (int a = 0; a < TR; ++a)
#pragma unroll
            for (int b = 0; b < TC; ++b) m1[a][b] = m2[a][b] = m3[a][b] = d4x{0, 0, 0, 0};
        d2x ra[kRing][TR], rb[kRing][TC];
        auto fetch = [&](int u, int kt) __attribute__((always_inline)) {
            const int k = kt < KT ? kt : KT - 1;  // past the end: a step already read
#pragma unroll
            for (int a = 0; a < TR; ++a) ra[u][a] = Ap[a][(size_t)k * 64];
#pragma unroll
            for (int b = 0; b < TC; ++b) rb[u][b] = Bp[b][4 * k];
        };
        auto step = [&](int u) __attribute__((always_inline)) {
#pragma unroll
            for (int a = 0; a < TR; ++a)
#pragma unroll
                for (int b = 0; b < TC; ++b) {
                    const d2x z = ra[u][a], i = rb[u][b];
                    m1[a][b] = mma64(z.x, i.x, m1[a][b]);
                    m2[a][b] = mma64(z.y, i.y, m2[a][b]);
                    m3[a][b] = third<THREE>(z, i, z.x - z.y, i.x - i.y, m3[a][b]);
                }
        };
#pragma unroll
        for (int u = 0; u < kRing; ++u) {
            fetch(u, u);
            __builtin_amdgcn_sched_barrier(0);  // (in the order they are used)
        }
        // whole turns of the ring without a branch, which would wait for every load in flight
        int kt = 0;
        for (; kt + kRing <= KT; kt += kRing) {
#pragma unroll
            for (int u = 0; u < kRing; ++u) {
                step(u);
                fetch(u, kt + u + kRing);
                __builtin_amdgcn_sched_barrier(0);  // (the loads stay spread over the turn)
            }
        }
#pragma unroll
        for (int u = 0; u < kRing; ++u)
            if (kt + u < KT) step(u);
        __syncthreads();  // red clear
#pragma unroll
        for (int b = 0; b < TC; ++b) {
            const int slot = c0 + 16 * b + j;
            const bool live = slot < nact;
            const long long c = act[live ? slot : nact - 1];
            double e = 0.0, poison = 0.0;
#pragma unroll
            for (int a = 0; a < TR; ++a) {
                const int bus0 = 16 * (rt + a) + g;
                d2x old[4];
                double sr[4], si[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (live && bus0 + 4 * r < n) {
                        old[r] = reinterpret_cast<const d2x *>(x)[c * n + bus0 + 4 * r];
                        sr[r] = (double)S[2 * (c * n + bus0 + 4 * r)];
                        si[r] = (double)S[2 * (c * n + bus0 + 4 * r) + 1];
                    }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (live && bus0 + 4 * r < n)
                        update64<IO>(m1[a][b][r] - m2[a][b][r],
                                     imaginary<THREE>(m1[a][b][r], m2[a][b][r], m3[a][b][r]), w[bus0 + 4 * r], c,
                                     bus0 + 4 * r, n, KB, S, zs, old[r], sr[r], si[r], x, Bn, e, poison);
            }
            if (live)
                atomicMax(red + slot - cb, poison == 0.0 ? (unsigned long long)__double_as_longlong(e) : ~0ull);
        }
        __syncthreads();
        if (tid < kCols && cb + tid < nact) atomicMax(dmax + act[cb + tid], red[tid]);
        __syncthreads();  // red is reused
    }
}

// The same for few columns: a workgroup per 16 x 16 tile, a wavefront for each of the
// three sums, so that a sweep takes about one chain of KT products (64 cycles each), and
// kLoaders more that bring the operands: they request them kSets chunks of kChunk k-steps before
// they write them to LDS, real and imaginary parts and what the third product takes in planes
// of their own, so that a product reads the 1 KB it uses.  Three buffers: while the sums are at
// chunk c and read on into c + 1, chunk c + 2 is written.  A sweep of one column at 999 buses:
// 22 us with the three wavefronts bringing the operands themselves, as with one loader; 17 with
// four (LDS writes and sums each take about as long as the chain, 6.7 us); 8 loaders 20, chunks of 12
// and more chunks requested ahead 17.
constexpr int kChunk = 8, kLoaders = 4, kSets = 2;

template <bool THREE, typename IO>
__global__ __launch_bounds__(64 * (3 + kLoaders)) void gemm64_sums_kernel(
    const d2x *__restrict__ A, int KT, const d2x *__restrict__ B, d2x *__restrict__ Bn, int KB,
    const long long *__restrict__ act, const int *__restrict__ na, int row_blocks, const d2x *__restrict__ w, int n,
    const IO *__restrict__ S, const ZipShares zs, double *__restrict__ x, unsigned long long *__restrict__ dmax) {
    constexpr int kPlanes = THREE ? 6 : 4;  // Zr, Zi, Ir, Ii (and Zr - Zi, Ir - Ii)
    constexpr int kAhead = 4;               // k-steps between a read from LDS and its product
    constexpr int kOwn = kChunk / kLoaders;  // k-steps of a chunk that a loader brings
    const int nact = *na;
    const int ct = (nact + 15) / 16;
    const int chunks = (KT + kChunk - 1) / kChunk;
    const int turns = (chunks + 2 + kSets - 1) / kSets * kSets;  // chunks written: two are ahead
    __shared__ double stage[3][kChunk][kPlanes][64];  // [buffer][k-step][plane][lane]
    __shared__ double part[3][4][64];
    __shared__ unsigned long long red[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;
    for (int t = blockIdx.x; t < ct * row_blocks; t += gridDim.x) {
        const int c0 = t / row_blocks * 16, rt = t % row_blocks;
        if (tid < 16) red[tid] = 0ull;
        const bool live = c0 + j < nact;
        const long long c = act[live ? c0 + j : nact - 1];
        auto bring = [&] {
            const int own = kOwn * (wave - 3);
            const d2x *Ap = A + (size_t)rt * KT * 64 + lane;
            const d2x *Bp = B + c * KB + g;
            d2x ra[kSets][kOwn], rb[kSets][kOwn];
            auto fetch = [&](int u, int chunk) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < kOwn; ++i) {
                    const int kt = chunk * kChunk + own + i, k = kt < KT ? kt : KT - 1;
                    ra[u][i] = Ap[(size_t)k * 64];
                    rb[u][i] = Bp[4 * k];
                }
            };
            auto put = [&](int u, int chunk, int buffer) __attribute__((always_inline)) {
                if ((chunk + 1) * kChunk > KT)  // products past the end add nothing
#pragma unroll
                    for (int i = 0; i < kOwn; ++i)
                        if (chunk * kChunk + own + i >= KT) ra[u][i] = rb[u][i] = d2x{0.0, 0.0};
#pragma unroll
                for (int i = 0; i < kOwn; ++i) {
                    const d2x z = ra[u][i], q = rb[u][i];
                    double(*s)[64] = stage[buffer][own + i];
                    s[0][lane] = z.x, s[1][lane] = z.y;
                    s[2][lane] = q.x, s[3][lane] = q.y;
                    if constexpr (THREE) s[4][lane] = z.x - z.y, s[5][lane] = q.x - q.y;
                }
            };
#pragma unroll
            for (int u = 0; u < kSets; ++u) {
                fetch(u, u);
                __builtin_amdgcn_sched_barrier(0);
            }
            int buffer = 0;  // of chunk k + u
            for (int k = 0; k < turns; k += kSets) {
#pragma unroll
                for (int u = 0; u < kSets; ++u) {
                    put(u, k + u, buffer);
                    __builtin_amdgcn_sched_barrier(0);
                    fetch(u, k + u + kSets);
                    __builtin_amdgcn_sched_barrier(0);
                    lds_barrier();
                    buffer = buffer == 2 ? 0 : buffer + 1;
                }
            }
        };
        auto sum = [&](auto which) __attribute__((always_inline)) {
            constexpr int P = decltype(which)::value;
            constexpr bool kBoth = P == 2 && !THREE;  // the third sum of four products
            constexpr int kZ = P == 2 ? (THREE ? 4 : 0) : P, kI = P == 2 ? (THREE ? 5 : 3) : 2 + P;
            d4x m = d4x{0, 0, 0, 0};
            double z[kChunk], i[kChunk], z2[kChunk], i2[kChunk];
            auto read = [&](int buffer, int k) __attribute__((always_inline)) {
                z[k] = stage[buffer][k][kZ][lane];
                i[k] = stage[buffer][k][kI][lane];
                if constexpr (kBoth) z2[k] = stage[buffer][k][1][lane], i2[k] = stage[buffer][k][2][lane];
            };
            lds_barrier();
            lds_barrier();  // chunks 0 and 1 are there
#pragma unroll
            for (int k = 0; k < kAhead; ++k) read(0, k);
            int buffer = 0;
            for (int chunk = 0; chunk < chunks; ++chunk) {
                const int next = buffer == 2 ? 0 : buffer + 1;
#pragma unroll
                for (int k = 0; k < kChunk; ++k) {
                    if (k + kAhead < kChunk)
                        read(buffer, k + kAhead);
                    else
                        read(next, k + kAhead - kChunk);
                    __builtin_amdgcn_sched_barrier(0);
                    m = mma64(z[k], i[k], m);
                    if constexpr (kBoth) m = mma64(z2[k], i2[k], m);
                }
                lds_barrier();
                buffer = next;
            }
            for (int k = chunks + 2; k < turns; ++k) lds_barrier();
#pragma unroll
            for (int r = 0; r < 4; ++r) part[P][r][lane] = m[r];
        };
        if (wave >= 3) bring();
        if (wave == 0) sum(std::integral_constant<int, 0>{});
        if (wave == 1) sum(std::integral_constant<int, 1>{});
        if (wave == 2) sum(std::integral_constant<int, 2>{});
        __syncthreads();  // the sums visible, red clear
        double e = 0.0, poison = 0.0;
        if (wave < 4) {
            const int r = wave, bus = 16 * rt + g + 4 * r;
            if (live && bus < n) {
                const double p1 = part[0][r][lane], p2 = part[1][r][lane], p3 = part[2][r][lane];
                update64<IO>(p1 - p2, imaginary<THREE>(p1, p2, p3), w[bus], c, bus, n, KB, S, zs,
                             reinterpret_cast<const d2x *>(x)[c * n + bus], (double)S[2 * (c * n + bus)],
                             (double)S[2 * (c * n + bus) + 1], x, Bn, e, poison);
            }
        }
        if (live) atomicMax(red + j, poison == 0.0 ? (unsigned long long)__double_as_longlong(e) : ~0ull);
        __syncthreads();
        if (tid < 16 && c0 + tid < nact) atomicMax(dmax + act[c0 + tid], red[tid]);
        __syncthreads();  // red and part are reused
    }
}

constexpr int kXcds = 8;  // workgroups are dealt to the chip's eight dies in turn

// The same for a handful of columns: a wavefront per 16 buses x 4 columns, whose 4 x 4 x 4 products
// (four blocks of four buses, the operator's fragments as they are) take 24 cycles instead of 64
// and round alike: both are chains of FMAs over their k values.  No LDS and no barrier in the
// loop.  Bound by issue, three products per k-step (72 cycles), with a ring deep enough for the
// way to L2.  One column of 999 buses: 14.6 us a sweep, 17 by the kernel above.  A tile's column
// groups go to one die.
template <bool THREE, typename IO>
__global__ __launch_bounds__(64) void gemm64_few_kernel(
    const d2x *__restrict__ A, int KT, const d2x *__restrict__ B, d2x *__restrict__ Bn, int KB,
    const long long *__restrict__ act, const int *__restrict__ na, int row_blocks, const d2x *__restrict__ w, int n,
    const IO *__restrict__ S, const ZipShares zs, double *__restrict__ x, unsigned long long *__restrict__ dmax) {
    constexpr int kRing = 20;
    const int nact = *na;
    const int lane = threadIdx.x, j = lane & 3;
    const int spread = (row_blocks + kXcds - 1) / kXcds * kXcds;
    __shared__ unsigned long long red[4];
    for (int t = blockIdx.x; t < (nact + 3) / 4 * spread; t += gridDim.x) {
        const int c0 = t / spread * 4, rt = t % spread;
        if (rt >= row_blocks) continue;
        if (lane < 4) red[lane] = 0ull;
        const bool live = c0 + j < nact;
        const long long c = act[live ? c0 + j : nact - 1];
        const int bus = 16 * rt + 4 * (lane >> 2 & 3) + (lane >> 4);  // of the lane's result
        const bool mine = live && bus < n;
        d2x wv = d2x{0.0, 0.0}, old = wv;
        double sr = 0.0, si = 0.0;
        if (mine) {
            wv = w[bus];
            old = reinterpret_cast<const d2x *>(x)[c * n + bus];
            sr = (double)S[2 * (c * n + bus)], si = (double)S[2 * (c * n + bus) + 1];
        }
        const d2x *Ap = A + (size_t)rt * KT * 64 + lane;
        const d2x *Bp = B + c * KB + (lane >> 4);
        double m1 = 0.0, m2 = 0.0, m3 = 0.0;
        d2x ra[kRing], rb[kRing];
        auto fetch = [&](int u, int kt) __attribute__((always_inline)) {
            const int k = kt < KT ? kt : KT - 1;  // past the end: a step already read
            ra[u] = Ap[(size_t)k * 64];
            rb[u] = Bp[4 * k];
        };
        auto step = [&](int u) __attribute__((always_inline)) {
            const d2x z = ra[u], i = rb[u];
            m1 = __builtin_amdgcn_mfma_f64_4x4x4f64(z.x, i.x, m1, 0, 0, 0);
            m2 = __builtin_amdgcn_mfma_f64_4x4x4f64(z.y, i.y, m2, 0, 0, 0);
            if constexpr (THREE) {
                m3 = __builtin_amdgcn_mfma_f64_4x4x4f64(z.x - z.y, i.x - i.y, m3, 0, 0, 0);
            } else {
                m3 = __builtin_amdgcn_mfma_f64_4x4x4f64(z.x, i.y, m3, 0, 0, 0);
                m3 = __builtin_amdgcn_mfma_f64_4x4x4f64(z.y, i.x, m3, 0, 0, 0);
            }
        };
#pragma unroll
        for (int u = 0; u < kRing; ++u) {
            fetch(u, u);
            __builtin_amdgcn_sched_barrier(0);
        }
        int kt = 0;
        for (; kt + kRing <= KT; kt += kRing) {
#pragma unroll
            for (int u = 0; u < kRing; ++u) {
                step(u);
                fetch(u, kt + u + kRing);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int u = 0; u < kRing; ++u)
            if (kt + u < KT) step(u);
        double e = 0.0, poison = 0.0;
        if (mine)
            update64<IO>(m1 - m2, imaginary<THREE>(m1, m2, m3), wv, c, bus, n, KB, S, zs, old, sr, si, x, Bn, e,
                         poison);
        __syncthreads();  // red clear
        if (live) atomicMax(red + j, poison == 0.0 ? (unsigned long long)__double_as_longlong(e) : ~0ull);
        __syncthreads();
        if (lane < 4 && c0 + lane < nact) atomicMax(dmax + act[c0 + lane], red[lane]);
        __syncthreads();  // red is reused
    }
}

// Chunks of cpb <= 256 active columns, one thread each: sweep count, stopping rule (thr: the bit
// pattern of the smallest |dV|^2 whose root is not below the tolerance), retirement and the
// staying columns' places in the next list.  Where the state is kept `apart` from the
// results (and B has no second copy) one wave per column then copies a retired one and forms
// a staying one's next injection.  `cnt_next` was cleared a sweep earlier; `cnt_clear` (the count
// two sweeps back, read by no kernel still to run) is cleared for the sweep after next.
template <typename IO>
__global__ __launch_bounds__(256) void finish64_kernel(const long long *__restrict__ act, const int *__restrict__ cnt,
                                                       int *cnt_clear, const double *x, int n,
                                                       const IO *S, const ZipShares zs, int KB, d2x *B,
                                                       unsigned long long thr, int max_iter,
                                                       unsigned long long *__restrict__ dmax, int32_t *iters,
                                                       int8_t *status, IO *V, bool apart, int cpb,
                                                       long long *__restrict__ act_next, int *cnt_next,
                                                       int *done_flag, int seq) {
    __shared__ long long cols[256];  // column + 1, negative when retired; 0: none
    __shared__ int wsum[4], base_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nact = *cnt;
    if (blockIdx.x == 0 && tid == 0) {
        *cnt_clear = 0;
        if (nact == 0) post_done(done_flag, seq);
    }
    for (long long c0 = blockIdx.x * (long long)cpb; c0 < nact; c0 += (long long)gridDim.x * cpb) {  // block-uniform
        long long c = -1;
        bool stay = false;
        if (tid < cpb && c0 + tid < nact) {
            c = act[c0 + tid];
            const unsigned long long d = dmax[c];
            const bool bad = d == ~0ull, conv = d < thr;
            const int it = iters[c] + 1;
            stay = !(bad || conv || it >= max_iter);
            iters[c] = it;
            dmax[c] = 0ull;
            if (!stay) status[c] = bad ? TPF_ST_NONFINITE : (conv ? TPF_ST_CONVERGED : TPF_ST_MAX_ITER);
        }
        const int slot = chunk_slot(stay, cnt_next, wsum, &base_s);
        if (stay) act_next[slot] = c;
        if (apart) {
            cols[tid] = c < 0 ? 0 : stay ? c + 1 : -c - 1;
            __syncthreads();
            for (int k = wave; k < cpb; k += 4) {
                if (cols[k] == 0) break;  // past the active columns (wave-uniform)
                const bool on = cols[k] > 0;
                const long long cc = (on ? cols[k] : -cols[k]) - 1;
                for (int b = lane; b < n; b += 64) {
                    const d2x v = reinterpret_cast<const d2x *>(x)[cc * n + b];
                    if (on) {
                        B[cc * KB + b] = injection64((double)S[2 * (cc * n + b)], (double)S[2 * (cc * n + b) + 1], v.x,
                                                     v.y, b, zs);
                    } else {
                        V[2 * (cc * n + b)] = (IO)v.x;
                        V[2 * (cc * n + b) + 1] = (IO)v.y;
                    }
                }
            }
        }
        __syncthreads();  // the chunk's tables are reused
    }
}

}  // namespace

// Workspace of the FP64 sweeps: two copies of B [tau][KB] (complex), the column maxima
// [tau], two active lists [tau], three counts.  Where the state cannot live in the output
// array it takes the second copy's place.
struct Large64 {
    int KT, KB;
    size_t bB, bD, bA;
    Large64(int n, int64_t tau) {
        auto al = [](size_t b) { return (b + 255) / 256 * 256; };
        KT = large64_ksteps(n);
        KB = 4 * KT;
        bB = al((size_t)tau * KB * 16);
        bD = al((size_t)tau * 8);
        bA = al((size_t)tau * 8);
    }
    size_t total() const { return 2 * bB + bD + 2 * bA + 256; }
};

size_t large64_workspace(int n, int64_t tau) { return Large64(n, tau).total(); }

template <bool THREE, typename IO>
static int run_large64(const tpf_network_s &net, const DeviceNet &dn, const void *S, int64_t tau, double tol,
                       int max_iter, const void *V0, void *V, int32_t *iters, int8_t *status, void *ws,
                       hipStream_t st) {
    const int n = net.n;
    const Large64 L(n, tau);
    char *p = static_cast<char *>(ws);
    d2x *B[2];
    B[0] = reinterpret_cast<d2x *>(p), p += L.bB;
    B[1] = reinterpret_cast<d2x *>(p), p += L.bB;
    auto *dmax = reinterpret_cast<unsigned long long *>(p);
    p += L.bD;
    long long *act[2];
    act[0] = reinterpret_cast<long long *>(p), p += L.bA;
    act[1] = reinterpret_cast<long long *>(p), p += L.bA;
    int *cnt = reinterpret_cast<int *>(p);  // three active counts in rotation
    // the state lives in a complex128 result, unless the caller solves in place (S is read
    // by every sweep) or the result begins inside the start voltages (a column's first state would
    // overwrite another's start; the very same array is fine)
    const size_t bytes = (size_t)tau * n * 2 * sizeof(IO);
    const bool apart = sizeof(IO) == 4 || overlap(S, V, bytes) || (V0 != V && overlap(V0, V, bytes));
    double *x = static_cast<double *>(V);
    if (apart) {
        x = reinterpret_cast<double *>(B[1]);
        B[1] = nullptr;
    }
    const ZipShares zs{dn.aP, dn.aI, dn.aZ};
    const auto *A = reinterpret_cast<const d2x *>(dn.AL64);
    const auto *w = reinterpret_cast<const d2x *>(dn.wl);
    hipLaunchKernelGGL((start64_kernel<IO>), dim3((unsigned)((tau + 3) / 4)), dim3(256), 0, st, (const IO *)S,
                       (const IO *)V0, n, L.KB, (long long)tau, zs, x, B[0], B[1], iters, act[0], cnt, dmax);
    // Every sweep is queued without waiting, with grids fixed from tau: the active counts
    // stay on the device (three of them in rotation: read, appended, cleared) and the
    // kernels of a sweep with no active column exit at once.  Queueing stops early when
    // the device has already posted that none is left (all_retired).
    // Shape by the tiles a batch has (the results do not depend on it).  16 buses x 4 columns up to
    // one per CU, 16 x 16 up to two, 32 x 32 up to one, staged 64 x 64 from six; between them 64 x 32
    // straight from L2, or 64 x 64 where those do not save half a turn of the chip and the turns
    // are three or more (a turn of 64 x 32 at 999 buses takes 445 us and 445 more per solve, of
    // 64 x 64 840 and 560), and 64 x 64 when an operator beyond the 256 MB cache would be streamed more
    // than three times (4,999 buses, 500 columns: 11.1 ms by 64 x 32, 10.0).
    // Per solve, us, at 999 buses (16 x 4 / 16 x 16 / 32 x 32 / 64 x 32 / 64 x 64 / staged): 1 column
    // 235 / 269 / 447 / - / 1,206 / 1,525; 16: 242 / 282; 32: 348 / 300 / 597; 128: 1,075 / 451 / 601 / - /
    // 1,383 / 1,745; 256: - / 845 / 659 / 885 / 1,390; 500: - / 1,325 / 1,094 / 915 / 1,402 / 1,763; 1,000: -
    // / - / 1,740 / 1,356 / 1,426 / 1,795; 2,000: - / - / 3,043 / 2,238 / 2,250 / 2,575; 4,000: - / - / 5,733 /
    // 4,166 / 4,137 / 4,356; 8,192: 7,899 / 7,769 (64 x 64, staged).  At 349 buses: 32: 92 / 104 / 176;
    // 64: 117 / 111 / 169; 256: - / 155 / 184 / 238 / 399; 1,000: - / - / 308 / 260 / 415; 3,000: - / - /
    // 647 / 576 / 704; 5,000: - / - / 881 / 746 / 721 / 882.
    const int64_t cus = num_cus();
    auto tiles = [&](int rows, int columns) {
        return (int64_t)((n + rows - 1) / rows) * ((tau + columns - 1) / columns);
    };
    const int64_t turns = (tiles(64, 32) + cus - 1) / cus, twice = (tiles(64, 64) + cus - 1) / cus * 2;
    const bool cached = (size_t)16 * n * n <= ((size_t)192 << 20);
    const int shape = tiles(64, 64) >= 6 * cus                                         ? 5
                      : tiles(16, 4) <= cus                                            ? 0
                      : tiles(16, 16) <= 2 * cus                                       ? 1
                      : tiles(32, 32) <= cus                                           ? 2
                      : (turns < twice || twice < 6) && (turns <= 3 || cached)         ? 3
                                                                                       : 4;
    const int rows = shape >= 3 ? 64 : shape == 2 ? 32 : 16;
    const int columns = shape >= 4 ? 64 : shape >= 2 ? 32 : shape == 1 ? 16 : 4;
    const int row_blocks = (n + rows - 1) / rows;
    const auto gemm = shape == 5   ? gemm64_kernel<THREE, IO>
                      : shape == 4 ? gemm64_direct_kernel<THREE, 2, 2, IO>
                      : shape == 3 ? gemm64_direct_kernel<THREE, 2, 1, IO>
                      : shape == 2 ? gemm64_direct_kernel<THREE, 1, 1, IO>
                      : shape == 1 ? gemm64_sums_kernel<THREE, IO>
                                   : gemm64_few_kernel<THREE, IO>;
    const int threads = shape == 0 ? 64 : shape == 1 ? 64 * (3 + kLoaders) : 256;
    const int64_t blocks =
        shape == 0 ? (row_blocks + kXcds - 1) / kXcds * kXcds * ((tau + 3) / 4) : tiles(rows, columns);
    const unsigned g_mm = (unsigned)gemm_grid((const void *)gemm, threads, blocks);
    const int cpb = apart ? finish_chunk(n) : 256;
    const unsigned g_fin = (unsigned)std::min<int64_t>(kFinishGrid, (tau + cpb - 1) / cpb);
    const unsigned long long thr = square_bound(tol);
    const int seq = ++dn.solve_seq;
    for (int sweep = 0; sweep < max_iter; ++sweep) {
        if (all_retired(dn, seq)) break;
        const int cur = sweep & 1;
        int *cr = cnt + sweep % 3, *cn = cnt + (sweep + 1) % 3, *cz = cnt + (sweep + 2) % 3;
        hipLaunchKernelGGL(gemm, dim3(g_mm), dim3(threads), 0, st, A, L.KT, apart ? B[0] : B[cur],
                           apart ? nullptr : B[cur ^ 1], L.KB, act[cur], cr, row_blocks, w, n, (const IO *)S, zs, x,
                           dmax);
        hipLaunchKernelGGL((finish64_kernel<IO>), dim3(g_fin), dim3(256), 0, st, act[cur], cr, cz, x, n,
                           (const IO *)S, zs, L.KB, B[0], thr, max_iter, dmax, iters, status, (IO *)V, apart, cpb,
                           act[cur ^ 1], cn, dn.done_dev, seq);
    }
    return TPF_OK;
}

int launch_fpi_large64(const tpf_network_s &net, const DeviceNet &dn, const void *S, int dtype, int64_t tau, double tol,
                       int max_iter, const void *V0, void *V, int32_t *iters, int8_t *status, void *ws,
                       hipStream_t st) {
    if (!dn.AL64) return fail(TPF_ERR_UNSUPPORTED, "large-network operator not staged");
#define TPF_GO(M, IO) return run_large64<M, IO>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, ws, st)
    if (dtype == TPF_C128) {
        if (dn.three) TPF_GO(true, double);
        TPF_GO(false, double);
    }
    if (dn.three) TPF_GO(true, float);
    TPF_GO(false, float);
#undef TPF_GO
}

}  // namespace tpf
