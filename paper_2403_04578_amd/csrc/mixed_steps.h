// One bus's and one column's steps of the FP32 and mixed forms beyond the register-resident
// networks, shared by the per-sweep path (fpi_large.hip) and the persistent kernel
// (fpi_mid.hip): both compute the same iterates bit for bit.
#pragma once

#include "device_math.h"
#include "large_common.h"

namespace tpf {

typedef float f4x __attribute__((ext_vector_type(4)));

namespace {

struct MixState {
    int it, ph, want;            // sweeps done; 0 = full low sweeps, 1 = difference sweeps; refine wanted
    float dprev, sumd, uref;     // previous step, steps since the last refine, max |U| seen
    float ks, inv;               // B scale 2^sB and product unscale 2^-(sB + sZ) (FP16); 1, 1 (BF16)
};

typedef short s8x __attribute__((ext_vector_type(8)));
typedef __bf16 bf8x __attribute__((ext_vector_type(8)));
typedef _Float16 h8x __attribute__((ext_vector_type(8)));

template <int MODE>
struct Low16;
template <>
struct Low16<TPF_MODE_MIXED_BF16> {
    static constexpr float u = 0.00390625f;  // 2^-8
    __device__ static uint32_t enc2(float a, float b) {
        return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)a) |
               ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)b) << 16);
    }
    __device__ static f4x mma(const uint4 &a, const uint4 &b, const f4x &c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8x, a), __builtin_bit_cast(bf8x, b), c,
                                                       0, 0, 0);
    }
};
template <>
struct Low16<TPF_MODE_MIXED_FP16> {
    static constexpr float u = 0.00048828125f;  // 2^-11
    __device__ static uint32_t enc2(float a, float b) {
        a = __builtin_amdgcn_fmed3f(a, -65504.f, 65504.f);
        b = __builtin_amdgcn_fmed3f(b, -65504.f, 65504.f);
        return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)a) |
               ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)b) << 16);
    }
    __device__ static f4x mma(const uint4 &a, const uint4 &b, const f4x &c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8x, a), __builtin_bit_cast(h8x, b), c, 0,
                                                      0, 0);
    }
};

// a - b of the rounded terms (never fused with the product that made a).
__device__ __forceinline__ float rounded_difference(float a, float b) {
#pragma clang fp contract(off)
    return a - b;
}

// alpha_P conj(S./V) + alpha_I conj(S) + alpha_Z conj(S) V for ZIP loads, else conj(S./V)
// (given as ir, ii).
__device__ __forceinline__ float2 zip_injection(float ir, float ii, float sr, float si, float vr, float vi,
                                                const ZipShares &zs, int b) {
    if (!zs.aP) return make_float2(ir, ii);
    const float ap = (float)zs.aP[b], ai = (float)zs.aI[b];
    float2 o = make_float2(ap * ir + ai * sr, ap * ii - ai * si);
    if (zs.aZ) {
        const float az = (float)zs.aZ[b];
        o.x += az * (sr * vr + si * vi);
        o.y += az * (sr * vi - si * vr);
    }
    return o;
}

// FP32 injection of one bus with load s and drop u from w.
__device__ __forceinline__ float2 mixed_injection(float sr, float si, float wr, float wi, float ur, float ui,
                                                  const ZipShares &zs, int b) {
    const float vr = wr + ur, vi = wi + ui;
    const float r = reciprocal32(fmaxf(vr * vr + vi * vi, kMinV2));
    return zip_injection((sr * vr + si * vi) * r, (sr * vi - si * vr) * r, sr, si, vr, vi, zs, b);
}

// The FP32 mode's injection, evaluated in FP64 and rounded once: conj(S./V), or for ZIP loads
// alpha_P conj(S./V) + alpha_I conj(S) + alpha_Z conj(S) V (the constant-impedance current,
// carried in the injection: the same fixed point as eliminating diag(alpha_Z s*) into Y_dd).
__device__ __forceinline__ float2 full_injection(double sr, double si, double wr, double wi, float ur, float ui,
                                                 const ZipShares &zs, int b) {
    double vr = (double)ur, vi = (double)ui;
    vr += wr, vi += wi;
    const double inv = 1.0 / (vr * vr + vi * vi);
    double jr = (sr * vr + si * vi) * inv, ji = (sr * vi - si * vr) * inv;
    if (zs.aP) {
        const double ap = zs.aP[b], ai = zs.aI[b];
        jr = ap * jr + ai * sr;
        ji = ap * ji - ai * si;
        if (zs.aZ) {
            const double az = zs.aZ[b];
            jr += az * (sr * vr + si * vi);
            ji += az * (sr * vi - si * vr);
        }
    }
    return make_float2((float)jr, (float)ji);
}

// New drop of one bus from a low-precision product (p, unscaled by inv): the product itself
// on a full sweep (ph = 0), added to the old drop on a difference sweep; the step's square
// into emax, the largest |U| into umax.
__device__ __forceinline__ float2 low_update(float p0, float p1, float2 old, int ph, float inv, float &emax,
                                             float &umax, int &bad) {
    const float pr = p0 * inv, pi = p1 * inv;
    const float nr = ph ? old.x + pr : pr, ni = ph ? old.y + pi : pi;
    const float dr = nr - old.x, di = ni - old.y;
    const float e2 = dr * dr + di * di;
    bad |= !(e2 < HUGE_VALF);
    emax = e2 > emax ? e2 : emax;
    umax = fmaxf(umax, fmaxf(fabsf(nr), fabsf(ni)));
    return make_float2(nr, ni);
}

// The same from an FP32 product of the whole injection.
__device__ __forceinline__ float2 full_update(float p0, float p1, float2 old, double &emax, int &bad) {
    const double nr = (double)p0, ni = (double)p1;
    const double dr = nr - (double)old.x, di = ni - (double)old.y;
    const double e2 = dr * dr + di * di;
    bad |= !(e2 < HUGE_VAL);
    emax = e2 > emax ? e2 : emax;
    return make_float2((float)nr, (float)ni);
}

// Schedule state of a column whose largest load entry (times the shares' bound) is sm.
template <int MODE>
__device__ __forceinline__ MixState mixed_start(float sm, int sbad, int sZ) {
    int sB = 0;
    if (MODE == TPF_MODE_MIXED_FP16) {
        int e = 0;
        (void)frexpf(sm > 0.f && sm < 1e30f ? sm : 1.0f, &e);
        sB = 12 - e;  // max |S| 2^sB < 2^12: |I| 2^sB < 2^15 while |V| > 1/4
    }
    MixState m;
    m.it = m.ph = m.want = 0;
    m.dprev = m.sumd = m.uref = 0.f;
    m.ks = ldexpf(1.0f, sB);
    m.inv = ldexpf(1.0f, -(sB + (MODE == TPF_MODE_MIXED_FP16 ? sZ : 0)));
    // the FP16 saturation would clip a non-finite load; the unscale carries it into
    // the iterate instead, so the column ends NONFINITE
    if (sbad) m.inv = __builtin_nanf("");
    return m;
}

// After a sweep with step d (refine: the FP32 product's; um: the largest |U|): counts it,
// decides what the next one is (m.want: refine) and returns whether the column converged.
template <int MODE>
__device__ __forceinline__ bool mixed_schedule(MixState &m, bool refine, float d, float um, float tol) {
    constexpr float u = Low16<MODE>::u;
    const float theta = 4.0f * u, refresh = 6.7e-8f / u, margin = 1.0f + 8.0f * u;
    m.it += 1;
    bool conv = false;
    if (refine) {
        conv = d < tol;
        m.ph = 1;
        m.want = 0;
        m.sumd = 0.f;
    } else if (m.ph == 0) {
        m.uref = fmaxf(m.uref, um);
        if (!m.want && (d <= theta * m.uref || (m.it >= 2 && d > 0.5f * m.dprev))) m.want = 1;
    } else {
        conv = d * margin < tol;
        m.sumd += d;
        if (!m.want && m.sumd > refresh) m.want = 1;
    }
    m.dprev = d;
    return conv;
}

}  // namespace
}  // namespace tpf
