// Persistent FP64 sweep kernel for networks with up to 320 PQ buses.
//
// Algorithm 1 (Sec. IV-A) evaluates V <- Z conj(S ./ V) + w for every power flow
// (column) of the reshaped load matrix until the voltage step of that column
// falls below the tolerance.  Here a workgroup owns 16 column slots, and each of its
// wavefronts some tiles of 16 buses of all of them.  Per sweep it
//   1. multiplies the injections (MFMA B operand, in LDS, never stored to memory) by Z on the
//      16x16x4 FP64 matrix cores, the complex product as three or four real ones, with Z
//      streamed from L2 in fragment order,
//   2. adds w, measures max_i |V'_i - V_i| per column with atomics on LDS, and forms the next
//      injections conj(S./V) = conj(S) V / |V|^2 (Eq. (3)) into the operand's other copy,
//   3. retires converged columns (writes V, sweep count and status) and refills
//      their slots from a global atomic column queue, so the 16-wide MFMA tiles
//      stay full while columns finish after different numbers of sweeps.
//
// Register layout.  A tile is 16 buses; the real and imaginary parts of Z are separate
// operands.  The FP64 MFMA leaves tile row g + 4r of output column j in lane 16g + j,
// register r, for each of the products, so a lane combines Re and Im of buses
// 16t + g + 4r of its column by itself.  For k-step 4t + r lane 16g + j must supply
// I[16t + 4r + g][j], which is exactly the bus it holds in register r of tile t: the
// epilogue lane writes the operand entry that the same lane position reads.
#include <cmath>
#include <cstring>

#include "device_math.h"
#include "tpf_internal.h"

namespace tpf {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

template <typename IO>
__device__ __forceinline__ void ld_c(const IO *p, double &re, double &im) {
    re = (double)p[0];
    im = (double)p[1];
}

template <typename IO>
__device__ __forceinline__ void st_c(IO *p, double re, double im) {
    p[0] = (IO)re;
    p[1] = (IO)im;
}

// One workgroup of NW waves owns 16 column slots; wave w computes the 16-bus tiles
// t = w + NW q of all 16 columns.  Per lane and owned tile the slot's
// voltages and loads of buses 16t + g + 4r, r = 0..3, in registers; the injections
// conj(S./V) of all buses live in LDS as Ib[bus][16 columns] complex values: the lane that
// holds bus 16t + g + 4r of column j writes row 16t + 4r + g, and k-step kt reads rows
// 4kt .. 4kt + 3, so both access patterns are contiguous 1 KB spans.
template <int TPW>
struct SlotState {
    d4 vr[TPW], vi[TPW], sr[TPW], si[TPW];
};

// a - b of the rounded terms, whatever products they came from: the third product's operand
// has to be the difference of the values the other two use.
__device__ __forceinline__ double plain_difference(double a, double b) {
#pragma clang fp contract(off)
    return a - b;
}

// Injections in LDS: complex values, and with SUM their Re - Im as a plane of its own.
template <bool SUM>
struct Inj {
    d2 *c;      // [rows][16]
    double *s;  // [rows][16] (SUM)
};

// Writes the injection conj(S./V) of the lane's four buses of tile t (rows below `rows`); for
// ZIP loads (Eq. (2)) alpha_P conj(S./V) + alpha_I conj(S) + alpha_Z conj(S) V, with the
// shares staged in LDS as zl[3][16 MT] (alpha_P, alpha_I, alpha_Z).
template <bool SUM, bool ZIP>
__device__ __forceinline__ void put_injection(const Inj<SUM> &I, int t, int lane, const d4 &vr, const d4 &vi,
                                              const d4 &sr, const d4 &si, const double *zl, int MT, int rows) {
    const int g = lane >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int b = 16 * t + 4 * r + g;
        const double inv = reciprocal(vr[r] * vr[r] + vi[r] * vi[r]);
        const double pr = sr[r] * vr[r] + si[r] * vi[r], pi = sr[r] * vi[r] - si[r] * vr[r];  // conj(S) V
        double ir = pr * inv, ii = pi * inv;                                                  // conj(S/V)
        if constexpr (ZIP) {
            const double ap = zl[b], ai = zl[16 * MT + b], az = zl[32 * MT + b];
            ir = ap * ir + ai * sr[r] + az * pr;
            ii = ap * ii - ai * si[r] + az * pi;
        }
        if (b < rows) {
            I.c[64 * (4 * t + r) + lane] = d2{ir, ii};
            if constexpr (SUM) I.s[64 * (4 * t + r) + lane] = plain_difference(ir, ii);
        }
    }
}

typedef int i4 __attribute__((ext_vector_type(4)));

// The complex product Z I in separate sums m1 = Zr Ir, m2 = Zi Ii and m3.  THREE: three real
// products instead of four,
//     m3 = (Zr - Zi)(Ir - Ii);  Re = m1 - m2, Im = m1 + m2 - m3;
// else m3 = Zr Ii + Zi Ir = Im.
// The sweep is bound by the FP64 units (64 cycles per 16x16x4 product, and the vector
// instructions beside it do not overlap with the matrix ones: their busy shares add up to
// the same 85 % in every form of this kernel), so a quarter fewer products is a quarter
// less time there.  Every term stays in FP64, but with three products Im is the difference of
// sums of the size of Re's: the voltage angles of a resistive feeder would lose digits (rms error
// of Im V against 80-bit arithmetic 3 to 40 times the four products' at x = 0.3 r).  Networks
// whose reactances allow it take three (three_products in network.cpp: rms error of V there 0.7
// to 1.0 times the four products', of its imaginary part 0.8 to 0.9 times for loads at power
// factors from 0.9), the others four.  Fragments of Z (Re and Im of a lane's entry as
// one 16-byte load) stream from L2 through a 4-deep register ring, issued three k-steps
// ahead of their products.
//
// NV tiles into slots Q0 .. Q0 + NV - 1 over the k-steps [k0, k1); the first one's fragments
// [KT + pad][64] start at fragment group `a0` (of 64) of the buffer, the others `stride`
// groups further each.
template <bool THREE, int TPW, int Q0, int NV, bool SUM>
__device__ __forceinline__ void sweep_product(d4 (&m1)[TPW], d4 (&m2)[TPW], d4 (&m3)[TPW],
                                              __amdgpu_buffer_rsrc_t A, int a0, int stride, const Inj<SUM> &I, int k0,
                                              int k1, int lane) {
    d2 r0[NV], r1[NV], r2[NV], r3[NV];
    const int voff = lane * 16;
    // buffer loads: the k-step is a scalar offset, no vector address arithmetic
    auto fetch = [&](d2(&r)[NV], int kt) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NV; ++q)
            r[q] = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(A, voff, (a0 + q * stride + kt) * 1024, 0));
    };
    const d2 *Bl = I.c + lane;
    const double *Sl = I.s + lane;
    d2 nb = Bl[k0 * 64];  // the next k-step's injections, read ahead of its products
    double ns = 0.0;
    if constexpr (SUM) ns = Sl[k0 * 64];
    auto step = [&](const d2(&r)[NV], int kt) __attribute__((always_inline)) {
        const d2 b = nb;
        double bs = ns;
        nb = Bl[(kt + 1) * 64];  // one row group past the last is read, not used
        if constexpr (SUM)
            ns = Sl[(kt + 1) * 64];
        else
            bs = b.x - b.y;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const double as = r[q].x - r[q].y;
            m1[Q0 + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(r[q].x, b.x, m1[Q0 + q], 0, 0, 0);
            m2[Q0 + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(r[q].y, b.y, m2[Q0 + q], 0, 0, 0);
            if constexpr (THREE) {
                m3[Q0 + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(as, bs, m3[Q0 + q], 0, 0, 0);
            } else {
                m3[Q0 + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(r[q].x, b.y, m3[Q0 + q], 0, 0, 0);
                m3[Q0 + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(r[q].y, b.x, m3[Q0 + q], 0, 0, 0);
            }
        }
    };
    fetch(r0, k0);
    fetch(r1, k0 + 1);
    fetch(r2, k0 + 2);
    int kt = k0;
#pragma unroll 1
    for (; kt + 4 <= k1; kt += 4) {  // a tile's fragments are padded with zero k-steps: no bounds branch
        fetch(r3, kt + 3);
        step(r0, kt);
        fetch(r0, kt + 4);
        step(r1, kt + 1);
        fetch(r1, kt + 5);
        step(r2, kt + 2);
        fetch(r2, kt + 6);
        step(r3, kt + 3);
    }
    if (kt < k1) step(r0, kt);
    if (kt + 1 < k1) step(r1, kt + 1);
    if (kt + 2 < k1) step(r2, kt + 2);
}

// Waves w and w + 4 of a workgroup share a SIMD, so the tiles left over by whole rounds of
// four, MT % 4 = r of them, would leave 4 - r SIMDs idle for a tile's time.  With SHARE their
// k-steps are shared out among wave roles 4 .. 7: roles 4 .. 3 + r own one such tile each and
// do its first r / 4, the other 4 - r do the rest and hand their partial sums over in LDS.
//
// The injections are kept in `bufs` copies used in turn: with two (and no shared tiles), a
// wave that ends its part of the product writes the next injections at once, without
// waiting for the others.
//
// `thr` is the bit pattern of the smallest double whose square root is not below the
// tolerance: non-negative doubles order like their bit patterns, so the stopping rule and
// the column maxima (|dV|^2 by LDS atomics) are integer work.
template <int TPW, int NW, bool SHARE, bool ZIP, bool THREE, typename IO>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(TPW == 1 ? 4 : 2))) void fpi_f64_kernel(
    const IO *__restrict__ S, IO *__restrict__ Vout, int32_t *__restrict__ iters_out,
    int8_t *__restrict__ status_out, const IO *__restrict__ V0, const double *__restrict__ A,
    const double *__restrict__ wv, int n, int MT, long long tau, unsigned long long thr, int max_iter, int bufs,
    unsigned long long *__restrict__ queue, const double *__restrict__ aP, const double *__restrict__ aI,
    const double *__restrict__ aZ) {
    constexpr bool SUM = THREE && TPW == 1;
    extern __shared__ __align__(16) double lds[];
    const int KT = (n + 3) / 4, rows = 4 * KT;
    d2 *Ibuf = reinterpret_cast<d2 *>(lds);                      // [bufs][rows][16]
    double *Isum = reinterpret_cast<double *>(Ibuf + (size_t)bufs * rows * 16);  // [bufs][rows][16] (SUM)
    d2 *wl = reinterpret_cast<d2 *>(Isum + (SUM ? (size_t)bufs * rows * 16 : 0));  // [16 MT] w staged once
    unsigned long long *mx = reinterpret_cast<unsigned long long *>(wl + 16 * MT);  // [3][16] max |dV|^2 in turn
    unsigned long long *qb = mx + 48;
    int *flag = reinterpret_cast<int *>(qb + 2);                 // [16] start voltages refused
    d2 *hand = reinterpret_cast<d2 *>(flag + 16);                // [3][4][64] partial sums handed over (extra > 0)
    const int extra = SHARE ? MT & 3 : 0;                        // tiles whose k-steps are shared out
    double *zl = reinterpret_cast<double *>(hand + (extra ? 768 : 0));  // [3][16 MT] ZIP shares (ZIP only)

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    const int g = lane >> 4, j = lane & 15;
    // tiles tw + NW q: the first `nf` (TPW or TPW - 1) over all k-steps, and for owners of a
    // shared tile one more over the first `ks`
    const int tw = wave;
    const int whole = MT - extra;
    const int nf = (whole - tw + NW - 1) / NW;
    const bool owner = extra > 0 && tw >= 4 && tw < 4 + extra, helper = extra > 0 && tw >= 4 + extra;
    const int nv = nf + (owner ? 1 : 0);
    const int ks = (extra * KT + 3) / 4;
    const int tstride = KT + kFragPadSteps;  // fragment groups of a tile
    const __amdgpu_buffer_rsrc_t Az =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(A), 0, MT * tstride * 1024, 0x00027000);
    // tile of slot q (whole tiles go round the roles; the shared ones come last)
    auto tile_of = [&](int q) { return q < nf ? tw + NW * q : whole + tw - 4; };

    SlotState<TPW> st;
    Inj<SUM> I{Ibuf, Isum};
    int turn = 0;  // mx[turn]: this sweep's column maxima
    long long col = -1;
    int it = 0;
    bool exhausted = false;

    // Loads column c into the lanes of the slots with `take` (c < 0: empty slot),
    // writes their injections, and applies the warm-start guard across the workgroup.
    auto load_slots = [&](bool take, long long c) {
        int bad = 0;
        const bool real = take && c >= 0;
        if (take) {
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                if (q < nv) {
                    const int b0 = 16 * tile_of(q) + g;
                    const IO *Sp = S + 2 * (c * n + b0), *Vp = V0 + 2 * (c * n + b0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double sr = 0.0, si = 0.0, vr = 1.0, vi = 0.0;
                        if (real && b0 + 4 * r < n) {
                            ld_c(Sp + 8 * r, sr, si);
                            if (V0) {
                                ld_c(Vp + 8 * r, vr, vi);
                                const double m2 = vr * vr + vi * vi;
                                bad |= (m2 >= 0.25 && m2 <= 2.25) ? 0 : 1;
                            }
                        }
                        st.sr[q][r] = sr;
                        st.si[q][r] = si;
                        st.vr[q][r] = vr;
                        st.vi[q][r] = vi;
                    }
                }
            }
        }
        if (V0) {  // uniform: a warm start is kept only if every bus of the column passes
            if (threadIdx.x < 16) flag[threadIdx.x] = 0;
            __syncthreads();
            if (bad) flag[j] = 1;
            __syncthreads();
            if (real && flag[j]) {
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    st.vr[q] = d4{1.0, 1.0, 1.0, 1.0};
                    st.vi[q] = d4{0.0, 0.0, 0.0, 0.0};
                }
            }
        }
        if (take) {
            col = c;
            it = 0;
#pragma unroll
            for (int q = 0; q < TPW; ++q)
                if (q < nv)
                    put_injection<SUM, ZIP>(I, tile_of(q), lane, st.vr[q], st.vi[q], st.sr[q], st.si[q], zl, MT, rows);
        }
    };

    for (int e = threadIdx.x; e < 16 * MT; e += NW * 64) wl[e] = d2{wv[e], wv[16 * MT + e]};
    if (threadIdx.x < 48) mx[threadIdx.x] = 0ull;
    if constexpr (ZIP) {  // padding buses: no load, share 0
        for (int e = threadIdx.x; e < 16 * MT; e += NW * 64) {
            zl[e] = e < n ? aP[e] : 0.0;
            zl[16 * MT + e] = e < n ? aI[e] : 0.0;
            zl[32 * MT + e] = e < n && aZ ? aZ[e] : 0.0;
        }
        __syncthreads();
    }
    // Initial fill: 16 consecutive columns per workgroup; the queue deals out those past
    // the first 16 gridDim.x (it is not touched when there are none).
    const unsigned long long dealt = 16ull * gridDim.x;
    {
        const long long base = 16ll * blockIdx.x;
        if (dealt >= (unsigned long long)tau) exhausted = true;
        const long long c = base + j;
        load_slots(true, c < tau ? c : -1);
    }
    __syncthreads();

    while (__ballot(col >= 0)) {
        // ---- complex product Z I for the owned tiles
        d4 m1[TPW], m2[TPW], m3[TPW];
#pragma unroll
        for (int q = 0; q < TPW; ++q) m1[q] = m2[q] = m3[q] = d4{0.0, 0.0, 0.0, 0.0};
        if constexpr (!SHARE) {
            if (nf == TPW)
                sweep_product<THREE, TPW, 0, TPW>(m1, m2, m3, Az, tw * tstride, NW * tstride, I, 0, KT, lane);
            else if constexpr (TPW > 1)
                sweep_product<THREE, TPW, 0, TPW - 1>(m1, m2, m3, Az, tw * tstride, NW * tstride, I, 0, KT, lane);
        } else {
            if constexpr (TPW > 1)
                sweep_product<THREE, TPW, 0, TPW - 1>(m1, m2, m3, Az, tw * tstride, NW * tstride, I, 0, KT, lane);
            // the last slot: a whole tile, an owner's part of a shared one, or a helper's parts.
            // extra = 3: role 7 does the rest of each of the three tiles; 2: roles 6 and 7 of one
            // each; 1: roles 5, 6 and 7 a third of it each
            const int h = tw - 4 - extra, third = (KT - ks + 2) / 3;
            const int e1 = helper ? (extra == 3 ? 3 : h + 1) : nv == TPW ? 1 : 0;
            for (int e = helper && extra != 3 ? h : 0; e < e1; ++e) {
                const int t = helper ? whole + (extra == 1 ? 0 : e) : tile_of(TPW - 1);
                const int k0 = !helper ? 0 : extra == 1 ? min(KT, ks + e * third) : ks;
                const int k1 = owner ? ks : helper && extra == 1 ? min(KT, k0 + third) : KT;
                m1[TPW - 1] = m2[TPW - 1] = m3[TPW - 1] = d4{0.0, 0.0, 0.0, 0.0};
                sweep_product<THREE, TPW, TPW - 1, 1>(m1, m2, m3, Az, t * tstride, 0, I, k0, k1, lane);
                if (helper) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        hand[256 * e + 64 * r + lane] =
                            d2{m1[TPW - 1][r] - m2[TPW - 1][r],
                               THREE ? m1[TPW - 1][r] + m2[TPW - 1][r] - m3[TPW - 1][r] : m3[TPW - 1][r]};
                }
            }
        }
        if (bufs == 1) {
            __syncthreads();  // every wave has read the injections; partial sums visible
        } else {
            I.s = I.c == Ibuf ? Isum + 16 * rows : Isum;
            I.c = I.c == Ibuf ? Ibuf + 16 * rows : Ibuf;
        }
        // ---- epilogue: V' = Z I + w, partial max |V' - V|^2, next injections
        double dmax = 0.0, poison = 0.0;
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            if (q < nv) {
                const int t = tile_of(q);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const d2 w = wl[16 * t + g + 4 * r];
                    double pr = m1[q][r] - m2[q][r], pi = THREE ? m1[q][r] + m2[q][r] - m3[q][r] : m3[q][r];
                    if (SHARE && q == TPW - 1 && owner) {
                        const int e1 = extra == 1 ? 3 : tw - 3;
                        for (int e = extra == 1 ? 0 : tw - 4; e < e1; ++e) {
                            const d2 p = hand[256 * e + 64 * r + lane];
                            pr += p.x;
                            pi += p.y;
                        }
                    }
                    const double nr = pr + w.x, ni = pi + w.y;
                    const double dr = nr - st.vr[q][r], di = ni - st.vi[q][r];
                    const double e = dr * dr + di * di;
                    poison = __builtin_fma(e, 0.0, poison);  // NaN once a step is not finite
                    dmax = fmax(dmax, e);
                    st.vr[q][r] = nr;
                    st.vi[q][r] = ni;
                }
                put_injection<SUM, ZIP>(I, t, lane, st.vr[q], st.vi[q], st.sr[q], st.si[q], zl, MT, rows);
            }
        }
        // three sets of maxima in turn: this sweep's, the next one's (a wave may already
        // write it while another still reads these), and the last one's, cleared below
        unsigned long long *m = mx + 16 * turn;
        if (nv > 0) atomicMax(m + j, poison == 0.0 ? (unsigned long long)__double_as_longlong(dmax) : ~0ull);
        __syncthreads();
        const unsigned long long dm2 = m[j];
        turn = turn == 2 ? 0 : turn + 1;
        if (threadIdx.x < 16) mx[16 * (turn == 2 ? 0 : turn + 1) + threadIdx.x] = 0ull;
        ++it;
        const bool bad = dm2 == ~0ull, conv = dm2 < thr;
        const bool done = col >= 0 && (bad || conv || it >= max_iter);
        const unsigned long long dm = __ballot(done && g == 0);  // same in every wave
        if (dm) {
            const int cnt = __popcll(dm);
            if (threadIdx.x == 0)
                *qb = exhausted ? (unsigned long long)tau : dealt + atomicAdd(queue, (unsigned long long)cnt);
            if (done) {
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    if (q < nv) {
                        const int b0 = 16 * tile_of(q) + g;
                        IO *Vp = Vout + 2 * (col * n + b0);
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (b0 + 4 * r < n) st_c(Vp + 8 * r, st.vr[q][r], st.vi[q][r]);
                    }
                }
                if (wave == 0 && g == 0) {
                    iters_out[col] = it;
                    status_out[col] = bad ? TPF_ST_NONFINITE : (conv ? TPF_ST_CONVERGED : TPF_ST_MAX_ITER);
                }
            }
            __syncthreads();
            const unsigned long long base = *qb;
            if (base + cnt >= (unsigned long long)tau) exhausted = true;
            const int rank = __popcll(dm & ((1ull << j) - 1ull));
            const long long c = (long long)base + rank;
            load_slots(done, c < tau ? c : -1);
            __syncthreads();  // refilled injections visible; qb free again
        }
    }
}

// max_iter == 0: return the start voltages (guarded warm start or flat).
template <typename IO>
__global__ void start_only_kernel(int n, const IO *__restrict__ V0, long long tau, IO *__restrict__ V,
                                  int32_t *__restrict__ iters, int8_t *__restrict__ status) {
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < tau;
         c += (long long)gridDim.x * blockDim.x) {
        bool ok = V0 != nullptr;
        if (V0)
            for (int b = 0; b < n; ++b) {
                const double vr = (double)V0[2 * (c * n + b)], vi = (double)V0[2 * (c * n + b) + 1];
                const double m2 = vr * vr + vi * vi;
                ok = ok && (m2 >= 0.25 && m2 <= 2.25);
            }
        for (int b = 0; b < n; ++b) {
            V[2 * (c * n + b)] = ok ? V0[2 * (c * n + b)] : (IO)1;
            V[2 * (c * n + b) + 1] = ok ? V0[2 * (c * n + b) + 1] : (IO)0;
        }
        iters[c] = 0;
        status[c] = TPF_ST_MAX_ITER;
    }
}

__global__ void zero_u64_kernel(unsigned long long *p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0ull;
}

// One workgroup copies chunk after chunk from the end that the destination does not reach first: a
// chunk is read whole before any of it is written.
constexpr int kMoveThreads = 1024, kMoveEach = 4;

template <typename T>
__global__ __launch_bounds__(kMoveThreads) void move_kernel(const T *src, T *dst, long long count, bool up) {
    constexpr long long kChunk = (long long)kMoveThreads * kMoveEach;
    for (long long done = 0; done < count; done += kChunk) {
        const long long base = (up ? done : count - done - kChunk) + threadIdx.x;  // (below 0: not there)
        T v[kMoveEach];
#pragma unroll
        for (int u = 0; u < kMoveEach; ++u) {
            const long long e = base + u * kMoveThreads;
            if (e >= 0 && e < count) v[u] = src[e];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kMoveEach; ++u) {
            const long long e = base + u * kMoveThreads;
            if (e >= 0 && e < count) dst[e] = v[u];
        }
        __syncthreads();
    }
}

int num_cus() {
    static int cached[64] = {0};
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 64) dev = 0;
    if (!cached[dev]) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 1;
        cached[dev] = v;
    }
    return cached[dev];
}

unsigned long long square_bound(double tol) {
    double x = tol * tol;
    while (std::sqrt(x) >= tol && x > 0.0) x = std::nextafter(x, 0.0);
    while (std::sqrt(x) < tol) x = std::nextafter(x, HUGE_VAL);
    unsigned long long bits;
    std::memcpy(&bits, &x, 8);
    return bits;
}

template <int TPW, int NW, bool SHARE, bool ZIP, bool THREE, typename IO>
static int launch_rows_as(const tpf_network_s &net, const DeviceNet &dn, const void *S, int64_t tau, double tol,
                          int max_iter, const void *V0, void *V, int32_t *iters, int8_t *status,
                          unsigned long long *queue, hipStream_t stream) {
    const int n = net.n, MT = dn.MT64;
    const size_t ib = (size_t)(n + 3) / 4 * 4 * (THREE && TPW == 1 ? 384 : 256);  // one copy of the injections
    size_t rest = (size_t)16 * MT * 16 + 48 * 8 + 16 + 64 + (SHARE ? 768 * 16 : 0) + (size_t)(ZIP ? 48 : 0) * MT * 8;
    auto kern = fpi_f64_kernel<TPW, NW, SHARE, ZIP, THREE, IO>;
    rest = std::max(rest, (size_t)1024);  // the product reads one row group past the last
    // Two copies of the injections where they do not cost a resident workgroup (half of the
    // barriers against fewer workgroups to fill the waits of the others).
    auto resident = [&](int bufs) {
        const size_t lds = bufs * ib + rest;
        int per_cu = 0;
        if (lds > (size_t)160 * 1024 ||
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, NW * 64, lds) != hipSuccess)
            per_cu = 0;
        return per_cu;
    };
    const int one = resident(1), two = SHARE ? 0 : resident(2);
    const int bufs = two > 0 && two >= one ? 2 : 1;
    const size_t lds = bufs * ib + rest;
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return fail(TPF_ERR_DEVICE, "hipFuncSetAttribute failed");
    const int per_cu = std::max(1, bufs == 2 ? two : one);
    const long long blocks = std::min<long long>((long long)num_cus() * per_cu, (tau + 15) / 16);
    if (16 * blocks < tau) {  // the columns past the first fill come from the queue
        const int rc = launch_zero_u64(queue, 1, stream);
        if (rc != TPF_OK) return rc;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(NW * 64), lds, stream, (const IO *)S, (IO *)V, iters,
                       status, (const IO *)V0, dn.A64, dn.w64, n, MT, (long long)tau, square_bound(tol), max_iter, bufs, queue,
                       (const double *)dn.aP, (const double *)dn.aI, (const double *)dn.aZ);
    return TPF_OK;
}

template <int TPW, int NW, bool SHARE, typename IO>
static int launch_rows(const tpf_network_s &net, const DeviceNet &dn, const void *S, int64_t tau, double tol,
                       int max_iter, const void *V0, void *V, int32_t *iters, int8_t *status,
                       unsigned long long *queue, hipStream_t stream) {
#define TPF_GO(Z, M) \
    return launch_rows_as<TPW, NW, SHARE, Z, M, IO>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, queue, stream)
    if (dn.aP) {
        if (dn.three) TPF_GO(true, true);
        TPF_GO(true, false);
    }
    if (dn.three) TPF_GO(false, true);
    TPF_GO(false, false);
#undef TPF_GO
}

// Leftover tiles are shared out among the waves wherever there are some, as long as a wave
// owns at most two (with three the registers are full).  Against whole tiles: 145 against
// 164 us for 43,200 columns of 86 buses (6 tiles), 1,168 against 1,236 us for 100,000 of 149
// (10 tiles), 1,046 against 1,126 us for 50,000 of 209 (14 tiles); no difference for the
// 99-bus year (7 tiles, one idle wave of eight).
static bool shares_tiles(int MT) { return MT > 4 && MT <= 16 && MT % 4 != 0; }

template <typename IO>
static int dispatch_rows(const tpf_network_s &net, const DeviceNet &dn, const void *S, int64_t tau, double tol,
                         int max_iter, const void *V0, void *V, int32_t *iters, int8_t *status,
                         unsigned long long *queue, hipStream_t stream) {
    int NW = 0, TPW = 0;
    f64_config(dn.MT64, NW, TPW);
    const bool share = shares_tiles(dn.MT64);
#define TPF_GO(T, W, SH)                                                                                       \
    if (TPW == T && NW == W && share == SH)                                                                    \
        return launch_rows<T, W, SH, IO>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, queue, stream);
    TPF_GO(1, 1, false) TPF_GO(1, 2, false) TPF_GO(1, 3, false) TPF_GO(1, 4, false) TPF_GO(1, 8, false)
    TPF_GO(2, 8, false) TPF_GO(3, 8, false) TPF_GO(1, 8, true) TPF_GO(2, 8, true)
#undef TPF_GO
    return fail(TPF_ERR_UNSUPPORTED, "register-resident sweep kernel: no instance for this network size");
}

int launch_fpi_small_f64(const tpf_network_s &net, const DeviceNet &dn, const void *S, int dtype, int64_t tau,
                         double tol, int max_iter, const void *V0, void *V, int32_t *iters, int8_t *status,
                         unsigned long long *queue, hipStream_t stream) {
    if (dtype == TPF_C128)
        return dispatch_rows<double>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, queue, stream);
    return dispatch_rows<float>(net, dn, S, tau, tol, max_iter, V0, V, iters, status, queue, stream);
}

int launch_start_only(int n, const void *V0, int dtype, int64_t tau, void *V, int32_t *iters, int8_t *status,
                      hipStream_t stream) {
    const long long blocks = std::min<long long>(4096, (tau + 255) / 256);
    if (dtype == TPF_C128)
        hipLaunchKernelGGL(start_only_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, stream, n,
                           (const double *)V0, (long long)tau, (double *)V, iters, status);
    else
        hipLaunchKernelGGL(start_only_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, n,
                           (const float *)V0, (long long)tau, (float *)V, iters, status);
    return TPF_OK;
}

int launch_zero_u64(unsigned long long *p, int count, hipStream_t stream) {
    hipLaunchKernelGGL(zero_u64_kernel, dim3((count + 63) / 64), dim3(64), 0, stream, p, count);
    return TPF_OK;
}

int launch_move(const void *src, void *dst, int dtype, int64_t count, hipStream_t stream) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    const bool up = static_cast<const char *>(dst) < static_cast<const char *>(src);
    if (dtype == TPF_C128)
        hipLaunchKernelGGL(move_kernel<d2>, dim3(1), dim3(kMoveThreads), 0, stream, (const d2 *)src, (d2 *)dst,
                           (long long)count, up);
    else
        hipLaunchKernelGGL(move_kernel<f2>, dim3(1), dim3(kMoveThreads), 0, stream, (const f2 *)src, (f2 *)dst,
                           (long long)count, up);
    return TPF_OK;
}

}  // namespace tpf
