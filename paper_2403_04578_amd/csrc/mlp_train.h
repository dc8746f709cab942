// Training step of the learned warm start for networks whose padded layer widths are all at
// most 256 (the 99-bus network's 202 -> 256 x 3 -> 198), in three kernels:
//   train_chain_kernel  8 rows per workgroup from the (shuffled) loads through every layer
//                       forward, the loss, and every layer backward, activations in LDS;
//   train_dw_kernel     all layers' weight and bias gradients;
//   adamw_sync_kernel   AdamW on the FP32 master parameters and the BF16 copies.
// The step is bound by latency (launches, barriers, one L2 round trip of weights per
// layer), not by arithmetic: 1,024 rows are 1.4 GFLOP.  As separate kernels per layer and
// purpose (about 30 launches) a step of the 99-bus network took 277 us.
// Sums run in the same order as in the per-layer kernels of mlp.hip.
#pragma once

#include "device_math.h"

namespace tpf {
namespace {

constexpr int kChainWidth = 256, kChainRows = 8, kChainStride = 264, kChainThreads = 512;

// Place of element (row, k) in a fragment-ordered operand of `width` k values per row: the
// 16 x 32 fragments that a wave loads are contiguous (1 KB), lane (g, j) holding row 16 t + j,
// k = 32 s + 8 g .. + 7.  Row-major weights cost every line twice (a fragment uses half of
// each 128-byte line, and a layer does not fit L1): 5,500 cycles per layer instead of 2,300.
__device__ __forceinline__ int64_t frag_place(int row, int k, int width) {
    return (((int64_t)(row / 16) * (width / 32) + k / 32) * 64 + 16 * (k % 32 / 8) + row % 16) * 8 + k % 8;
}

struct TrainView {
    const __bf16 *Wt[17];  // W_l, fragment-ordered [out_p][in_p]
    const __bf16 *Wn[17];  // W_l^T, fragment-ordered [in_p][out_p]
    const float *b[17];    // padded
    __bf16 *HT[17];        // input of layer l, transposed [dp[l]][rp]
    __bf16 *GT[17];        // gradient at layer l's output (pre-activation), transposed [dp[l + 1]][rp]
    float *Z[17];          // pre-activation of hidden layer l = 1 .. L, [rp][dp[l]]
    int d[18], dp[18];
    int L, n;
};

struct Shuffle {
    int64_t total, first;  // rows of the whole set, first position of this batch in the epoch's order
    uint64_t key;
    int h;  // 0: no shuffle, row = position
};

// What a batch needs before its loads can be read: the row of each position, and its
// calendar phases.  Both are long serial chains (64-bit products, FP64 sines: 5 us at the head
// of the chain kernel), so the weight-gradient kernel prepares the next batch's beside its
// own work.  Thread i of a block of 128: position 32 block + i / 4, phase i % 4.
struct BatchRows {
    const int64_t *t_index;
    int64_t *src;  // [rows]
    float *phase;  // [rows][4]
    int64_t rows;  // 0: nothing to prepare
    Shuffle sh;
};

__device__ __forceinline__ void prepare_rows(const BatchRows &br, int block) {
    const int64_t r = 32 * (int64_t)block + threadIdx.x / 4;
    const int f = threadIdx.x & 3;
    if (r >= br.rows) return;
    const int64_t q = br.sh.h ? shuffled_row(br.sh.first + r, br.sh.total, br.sh.h, br.sh.key) : r;
    const int64_t t = br.t_index[q];
    const double mod = (double)(t % 1440) / 1440.0;
    const double day = (double)((t / 1440) % 365) / 365.0;
    const double ang = 2.0 * M_PI * (f < 2 ? mod : day);
    br.phase[4 * r + f] = (float)((f & 1) ? cos(ang) : sin(ang));
    if (f == 0) br.src[r] = q;
}

__global__ __launch_bounds__(128) void batch_rows_kernel(const BatchRows br) { prepare_rows(br, blockIdx.x); }

// One workgroup: rows r0 .. r0 + 7, 8 waves, wave w owning neurons 32 w .. 32 w + 31 of every
// layer as two product tiles (weights as the B operand, straight from L2: a layer's
// fragments are requested before the barrier that completes its inputs).  A tile's 16 rows
// repeat the 8; the upper half of the wave, whose rows are the repeats, takes the second
// tile's results instead, so that the GELUs, which take most of the kernel's time, run on
// full waves and over twice as many CUs as with 16 rows per workgroup.
template <typename IO>
__global__ __launch_bounds__(kChainThreads) void train_chain_kernel(
    const IO *__restrict__ S, const IO *__restrict__ V, const int64_t *__restrict__ order,
    const float *__restrict__ phase, int64_t rows, int64_t rp, const TrainView tv, double vs_re, double vs_im,
    float *__restrict__ lossp) {
    __shared__ __align__(16) __bf16 H[kChainRows][kChainStride];
    __shared__ int64_t src[kChainRows];
    __shared__ float red[8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;
    const int64_t r0 = (int64_t)blockIdx.x * kChainRows;
    const int n = tv.n, L = tv.L;
    const int nn = 32 * wave + 16 * (g >> 1) + j;  // this lane's neuron
    const int row = 4 * (g & 1);                   // and the first of its four rows
    if (tid < kChainRows) {
        const int64_t r = r0 + tid;
        src[tid] = r >= rows ? -1 : order[r];
    }
    b8 w[2][kChainWidth / 32];
    auto fetch = [&](const __bf16 *W, int out_p, int in_p) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kChainWidth / 32; ++s)
            if (32 * wave < out_p && 32 * s < in_p) {
                w[0][s] = reinterpret_cast<const b8 *>(W)[(2 * wave * (in_p / 32) + s) * 64 + lane];
                w[1][s] = reinterpret_cast<const b8 *>(W)[((2 * wave + 1) * (in_p / 32) + s) * 64 + lane];
            }
    };
    // neuron nn of the rows row .. row + 3
    auto product = [&](int out_p, int in_p) __attribute__((always_inline)) {
        f4 c0 = f4{0, 0, 0, 0}, c1 = f4{0, 0, 0, 0};
        if (32 * wave < out_p) {
#pragma unroll
            for (int s = 0; s < kChainWidth / 32; ++s)
                if (32 * s < in_p) {
                    const b8 a = *reinterpret_cast<const b8 *>(&H[j & 7][32 * s + 8 * g]);
                    c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[0][s], c0, 0, 0, 0);
                    c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[1][s], c1, 0, 0, 0);
                }
        }
        // the repeated rows 8 + 4 (g & 1) .. of the second tile are already in the upper half
        return g < 2 ? c0 : c1;
    };
    // the lane's four rows of neuron nn into LDS and, transposed, into T [width][rp]
    auto put = [&](const f4 &x, __bf16 *T) __attribute__((always_inline)) {
        const b4 q = b4{(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
#pragma unroll
        for (int r = 0; r < 4; ++r) H[row + r][nn] = q[r];
        *reinterpret_cast<b4 *>(T + (size_t)nn * rp + r0 + row) = q;
    };
    fetch(tv.Wt[0], tv.dp[1], tv.dp[0]);
    lds_barrier();
    // features 50 P, 50 Q (zero in the padding), and the calendar phases
    for (int e = tid; e < kChainRows * tv.dp[0]; e += kChainThreads) {
        const int r = e / tv.dp[0], f = e - r * tv.dp[0];
        const int64_t q = src[r];
        float v = 0.0f;
        if (q >= 0 && f < 2 * n) v = kFeatScale * (float)(f < n ? S[2 * (q * n + f)] : S[2 * (q * n + f - n) + 1]);
        if (f < 2 * n || f >= 2 * n + 4) H[r][f] = (__bf16)v;
    }
    if (tid >= kChainThreads - 4 * kChainRows) {
        const int r = (lane >> 2) & (kChainRows - 1), f = lane & 3;
        const float v = src[r] >= 0 ? phase[4 * (r0 + r) + f] : 0.0f;
        H[r][2 * n + f] = (__bf16)v;
    }
    lds_barrier();
    if (tid < tv.dp[0]) {
        b8 q;
#pragma unroll
        for (int i = 0; i < kChainRows; ++i) q[i] = H[i][tid];
        *reinterpret_cast<b8 *>(tv.HT[0] + (size_t)tid * rp + r0) = q;
    }
    // the targets of the lane's output, requested here and used after the forward pass
    IO tgt[4] = {0, 0, 0, 0};
    if (nn < 2 * n) {
        const int64_t o = nn < n ? 2 * (int64_t)nn : 2 * (int64_t)(nn - n) + 1;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (src[row + r] >= 0) tgt[r] = V[2 * src[row + r] * n + o];
    }
    // forward through the hidden layers
    for (int l = 0; l < L; ++l) {
        const bool mine = 32 * wave < tv.dp[l + 1];
        f4 v = product(tv.dp[l + 1], tv.dp[l]);
        fetch(tv.Wt[l + 1], tv.dp[l + 2], tv.dp[l + 1]);
        if (mine) {
            const float bias = tv.b[l][nn];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] += bias;
                tv.Z[l + 1][(r0 + row + r) * tv.dp[l + 1] + nn] = v[r];  // for the way back
                v[r] = nn < tv.d[l + 1] ? gelu(v[r]) : 0.0f;
            }
        }
        lds_barrier();  // every wave has read this layer's inputs
        if (mine) put(v, tv.HT[l + 1]);
        lds_barrier();
    }
    // output layer, loss and its gradient
    {
        const bool mine = 32 * wave < tv.dp[L + 1];
        f4 v = product(tv.dp[L + 1], tv.dp[L]);
        if (L > 0) fetch(tv.Wn[L], tv.dp[L], tv.dp[L + 1]);
        const float scale = 2.0f / (float)(rows * 2 * n);
        float part = 0.0f;
        if (mine) {
            const float bias = tv.b[L][nn];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float d = 0.0f;
                if (src[row + r] >= 0 && nn < 2 * n) {
                    const double t = (double)tgt[r] - (nn < n ? vs_re : vs_im);
                    d = (v[r] + bias) - (float)(kOutScale * t);
                    part += d * d;
                }
                v[r] = scale * d;
            }
        }
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
        if (lane == 0) red[wave] = part;
        lds_barrier();
        if (mine) put(v, tv.GT[L]);
        if (tid == 0) {
            float s = 0.0f;
            for (int k = 0; k < 8; ++k) s += red[k];
            lossp[blockIdx.x] = s / (float)(rows * 2 * n);
        }
        lds_barrier();
    }
    // backward: dZ_l = (dZ_{l+1} W_l) .* gelu'(Z_l)
    for (int l = L; l >= 1; --l) {
        const bool mine = 32 * wave < tv.dp[l];
        f4 v = product(tv.dp[l], tv.dp[l + 1]);
        if (l > 1) fetch(tv.Wn[l - 1], tv.dp[l - 1], tv.dp[l]);
        if (mine) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[r] = nn < tv.d[l] ? v[r] * gelu_grad(tv.Z[l][(r0 + row + r) * tv.dp[l] + nn]) : 0.0f;
        }
        lds_barrier();
        if (mine) put(v, tv.GT[l - 1]);
        lds_barrier();
    }
}

struct GradView {
    const __bf16 *HT[17], *GT[17];
    int64_t woff[17], boff[17];
    int d[18], dp[18];
    int tile0[18];  // first weight-tile block of layer l; tile0[L + 1] = their count
    int col0[18];   // first bias-gradient column of layer l, counted over all layers
    int L;
};

// Blocks below tile0[L + 1]: weight gradients dW_l[o][i] = sum_r G_l[r][o] H_l[r][i] in tiles of
// 64 outputs x 16 inputs, 32 x 16 per wave, both operands straight from L2 (their rows run
// along r, the contraction) through a four-deep register ring.  The others: one bias
// gradient per wave, db_l[o] = sum_r G_l[r][o], and after those the rows of the next batch.
__global__ __launch_bounds__(128) void train_dw_kernel(const GradView gv, int rp, float *__restrict__ grad,
                                                       const BatchRows next) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, j = lane & 15;
    if ((int)blockIdx.x < gv.tile0[gv.L + 1]) {
        int l = 0;
        while ((int)blockIdx.x >= gv.tile0[l + 1]) ++l;
        const int t = blockIdx.x - gv.tile0[l], ni = gv.dp[l] / 16;
        const int o0 = 64 * (t / ni) + 32 * wave, i0 = 16 * (t % ni);
        const __bf16 *A0 = gv.GT[l] + (size_t)(o0 + j) * rp + 8 * g, *A1 = A0 + (size_t)16 * rp;
        const __bf16 *B = gv.HT[l] + (size_t)(i0 + j) * rp + 8 * g;
        f4 c0 = f4{0, 0, 0, 0}, c1 = f4{0, 0, 0, 0};
        const int ks = rp / 32;
        b8 a0[4], a1[4], b[4];
        auto fetch = [&](int u, int k) __attribute__((always_inline)) {
            const int o = 32 * (k < ks ? k : ks - 1);
            a0[u] = *reinterpret_cast<const b8 *>(A0 + o);
            a1[u] = *reinterpret_cast<const b8 *>(A1 + o);
            b[u] = *reinterpret_cast<const b8 *>(B + o);
        };
#pragma unroll
        for (int u = 0; u < 4; ++u) fetch(u, u);
        for (int k = 0; k < ks; k += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (k + u < ks) {
                    c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[u], b[u], c0, 0, 0, 0);
                    c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[u], b[u], c1, 0, 0, 0);
                    fetch(u, k + u + 4);
                }
            }
        }
        const int i = i0 + j;
        if (i < gv.d[l]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = o0 + 4 * g + r;
                if (o < gv.d[l + 1]) grad[gv.woff[l] + (int64_t)o * gv.d[l] + i] = c0[r];
                if (o + 16 < gv.d[l + 1]) grad[gv.woff[l] + (int64_t)(o + 16) * gv.d[l] + i] = c1[r];
            }
        }
        return;
    }
    const int cb = (int)blockIdx.x - gv.tile0[gv.L + 1], ncb = (gv.col0[gv.L + 1] + 1) / 2;
    if (cb >= ncb) {
        prepare_rows(next, cb - ncb);
        return;
    }
    const int c = 2 * cb + wave;
    if (c >= gv.col0[gv.L + 1]) return;
    int l = 0;
    while (c >= gv.col0[l + 1]) ++l;
    const __bf16 *G = gv.GT[l] + (size_t)(c - gv.col0[l]) * rp;
    // partial sums over the rows t, t + 256, ... for t = 0 .. 255 (four per lane), then halving
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int r = 0; r < rp; r += 256)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (r + 64 * u + lane < rp) s[u] += (float)G[r + 64 * u + lane];
    float v = (s[0] + s[2]) + (s[1] + s[3]);
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    if (lane == 0) grad[gv.boff[l] + c - gv.col0[l]] = v;
}

struct ParamView {
    __bf16 *Wt[17], *Wn[17];
    uint16_t *Wf[17];
    float *bias[17], *bf[17];
    int64_t woff[18], boff[17];  // woff[L + 1]: the parameter count
    int d[18], dp[18];
    int L, n;
    bool chain;  // Wt and Wn are fragment-ordered for the chain kernel (else Wt row-major, no Wn)
};

// AdamW on every parameter, and its BF16 (weights) or FP32 (biases) copies at the places
// sync_kernel and frag_kernel give them (their padding stays zero).  With `loss_n` > 0 the first
// wave sums the chain kernel's partial losses: into loss_out, and scaled onto acc.
__global__ void adamw_sync_kernel(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                                  float *__restrict__ v, const ParamView pv, float lr, float wd, float b1, float b2,
                                  float eps, float bc1, float bc2, const float *__restrict__ lossp, int loss_n,
                                  float *__restrict__ acc, float scale) {
    const int64_t P = pv.woff[pv.L + 1];
    if (blockIdx.x == 0 && threadIdx.x < 64 && acc) {
        float s = 0.0f;
        for (int k = threadIdx.x; k < loss_n; k += 64) s += lossp[k];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (threadIdx.x == 0) acc[0] += s * scale;
    }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float mh = mi / bc1, vh = vi / bc2;
        p[i] -= lr * (mh / (sqrtf(vh) + eps) + wd * p[i]);
        int l = 0;
        while (i >= pv.woff[l + 1]) ++l;
        const int in = pv.d[l], in_p = pv.dp[l], out_p = pv.dp[l + 1];
        const bool last = l == pv.L;
        const int rel = (int)(i - pv.woff[l]);
        const bool weight = i < pv.boff[l];
        const int o = weight ? rel / in : (int)(i - pv.boff[l]), k = weight ? rel - o * in : 0;
        // row of the fragment copy: output-layer neurons (Re, Im) interleaved per bus
        const int r = last ? 2 * (o % pv.n) + o / pv.n : o;
        if (!weight) {
            pv.bias[l][o] = p[i];
            pv.bf[l][r] = p[i];
            continue;
        }
        const __bf16 q = (__bf16)p[i];
        pv.Wt[l][pv.chain ? frag_place(o, k, in_p) : (int64_t)o * in_p + k] = q;
        if (pv.chain) pv.Wn[l][frag_place(k, o, out_p)] = q;
        // input of the fragment copy: first-layer features (50 P, 50 Q) interleaved per bus
        const int kf = l == 0 && k < 2 * pv.n ? 2 * (k % pv.n) + k / pv.n : k;
        pv.Wf[l][frag_place(r, kf, in_p)] = __builtin_bit_cast(uint16_t, q);
    }
}

// loss_out = sum of the chain kernel's partial losses (one wave).
__global__ void loss_sum_kernel(const float *__restrict__ lossp, int count, float *__restrict__ loss_out) {
    float s = 0.0f;
    for (int k = threadIdx.x; k < count; k += 64) s += lossp[k];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (threadIdx.x == 0) loss_out[0] = s;
}

}  // namespace
}  // namespace tpf
