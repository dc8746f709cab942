// Learned warm start: a multilayer perceptron from loads to converged voltages,
// trained and evaluated with this library's own kernels (BF16 MFMA products,
// FP32 accumulation, FP32 master parameters, AdamW).
//
// Kernels
//   features_kernel    S, minute index -> X [rows][D0] bf16 (zero padded)
//   gemm_bf16_kernel   C = A B on 16x16x32 BF16 MFMA, 64x64 output tiles, A and B
//                      read through arbitrary element strides (so the same kernel
//                      does X W^T, dZ W and dZ^T X), fused epilogues: bias + GELU
//                      (hidden layers), bias (output), GELU' (backward), store of
//                      the weight gradient into the flat FP32 gradient vector
//   output_grad_kernel MSE loss and dY = 2 (y - target) / (rows outputs)
//   colsum_kernel      bias gradients
//   adamw_sync_kernel  decoupled-weight-decay Adam on the FP32 master vector, and the BF16
//                      copies of the changed weights (mlp_train.h)
//   sync_kernel        BF16 copies of the weights in the layouts the products read
//   predict_out_kernel y -> V0 = v_s + (y_re + j y_im)/20
//   gather_rows_kernel one shuffled mini-batch (S, V, minute index) for training
//   loss_accum_kernel  running mean of the batch losses of an epoch
#include <cmath>
#include <cstdio>
#include <cstring>

#include "tpf_internal.h"

namespace tpf {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kPad = 64;  // every layer width is padded to a multiple of 64
inline int padw(int x) { return (x + kPad - 1) / kPad * kPad; }
constexpr float kFeatScale = 50.0f, kOutScale = 20.0f;

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

template <typename IO>
__global__ void features_kernel(const IO *__restrict__ S, const int64_t *__restrict__ t_index, int n, int64_t rows,
                                int64_t rows_pad, int D0p, __bf16 *__restrict__ X) {
    const int64_t total = rows_pad * D0p;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = e / D0p;
        const int f = (int)(e - r * D0p);
        float v = 0.0f;
        if (r < rows) {
            if (f < n) {
                v = kFeatScale * (float)S[2 * (r * n + f)];
            } else if (f < 2 * n) {
                v = kFeatScale * (float)S[2 * (r * n + f - n) + 1];
            } else if (f < 2 * n + 4) {
                const int64_t t = t_index ? t_index[r] : r;
                const double mod = (double)(t % 1440) / 1440.0;
                const double day = (double)((t / 1440) % 365) / 365.0;
                const double ang = 2.0 * M_PI * (f < 2 * n + 2 ? mod : day);
                v = (float)(((f - 2 * n) & 1) ? cos(ang) : sin(ang));
            }
        }
        X[e] = (__bf16)v;
    }
}

enum { EP_HIDDEN = 0, EP_OUT = 1, EP_DGELU = 2, EP_DW = 3 };

// C[M][N] = sum_k A(m, k) B(k, n), A(m,k) = A[m sam + k sak], B(k,n) = B[k sbk + n sbn].
// M, N multiples of 64 and K a multiple of 32 (callers pad).  AK / BK: the operand is
// contiguous along k (else along m / n).
template <bool AK, bool BK, int EP>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const __bf16 *__restrict__ A, int64_t sam, int64_t sak,
                                                        const __bf16 *__restrict__ B, int64_t sbk, int64_t sbn,
                                                        int K, const float *__restrict__ bias,
                                                        float *__restrict__ Cf, __bf16 *__restrict__ Cb,
                                                        int64_t ldc, const float *__restrict__ Zin, int64_t ldz,
                                                        int valid_m, int valid_n, int64_t goff) {
    __shared__ __align__(16) __bf16 As[64][40];
    __shared__ __align__(16) __bf16 Bs[64][40];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, j = lane & 15;
    const int64_t m0 = (int64_t)blockIdx.x * 64;
    const int n0 = blockIdx.y * 64;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    f4 acc[2][2];
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = f4{0, 0, 0, 0};
    for (int k0 = 0; k0 < K; k0 += 32) {
        if (AK) {
            const int m = tid >> 2, kk = (tid & 3) * 8;
            const b8 v = *reinterpret_cast<const b8 *>(A + (m0 + m) * sam + (int64_t)(k0 + kk));
            *reinterpret_cast<b8 *>(&As[m][kk]) = v;
        } else {
            const int k = tid >> 3, mm = (tid & 7) * 8;
            const b8 v = *reinterpret_cast<const b8 *>(A + (m0 + mm) + (int64_t)(k0 + k) * sak);
#pragma unroll
            for (int i = 0; i < 8; ++i) As[mm + i][k] = v[i];
        }
        if (BK) {
            const int nn = tid >> 2, kk = (tid & 3) * 8;
            const b8 v = *reinterpret_cast<const b8 *>(B + (int64_t)(n0 + nn) * sbn + (k0 + kk));
            *reinterpret_cast<b8 *>(&Bs[nn][kk]) = v;
        } else {
            const int k = tid >> 3, nn = (tid & 7) * 8;
            const b8 v = *reinterpret_cast<const b8 *>(B + (int64_t)(k0 + k) * sbk + (n0 + nn));
#pragma unroll
            for (int i = 0; i < 8; ++i) Bs[nn + i][k] = v[i];
        }
        __syncthreads();
        b8 af[2], bf[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) af[a] = *reinterpret_cast<const b8 *>(&As[wm + 16 * a + j][8 * g]);
#pragma unroll
        for (int b = 0; b < 2; ++b) bf[b] = *reinterpret_cast<const b8 *>(&Bs[wn + 16 * b + j][8 * g]);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bf[b], acc[a][b], 0, 0, 0);
        __syncthreads();
    }
    // epilogue: lane holds C[row 4g + r][col j] of each 16x16 tile
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t m = m0 + wm + 16 * a + 4 * g + r;
                const int nn = n0 + wn + 16 * b + j;
                float v = acc[a][b][r];
                if (EP == EP_HIDDEN) {
                    v += bias[nn];
                    Cf[m * ldc + nn] = v;                       // pre-activation (for backward)
                    Cb[m * ldc + nn] = (__bf16)(nn < valid_n ? gelu(v) : 0.0f);
                } else if (EP == EP_OUT) {
                    Cf[m * ldc + nn] = v + bias[nn];
                } else if (EP == EP_DGELU) {
                    Cb[m * ldc + nn] = (__bf16)(nn < valid_n ? v * gelu_grad(Zin[m * ldz + nn]) : 0.0f);
                } else {  // EP_DW: gradient of W [valid_m][valid_n], row-major at goff
                    if (m < valid_m && nn < valid_n) Cf[goff + m * valid_n + nn] = v;
                }
            }
}

template <typename IO>
__global__ void output_grad_kernel(const float *__restrict__ Y, int64_t ldy, const IO *__restrict__ V, int n,
                                   int64_t rows, int64_t rows_pad, int Np, double vs_re, double vs_im,
                                   __bf16 *__restrict__ dY, float *__restrict__ loss) {
    const int64_t total = rows_pad * Np;
    const float scale = 2.0f / (float)(rows * 2 * n);
    float part = 0.0f;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = e / Np;
        const int c = (int)(e - r * Np);
        float d = 0.0f;
        if (r < rows && c < 2 * n) {
            const int b = c < n ? c : c - n;
            const double t = c < n ? ((double)V[2 * (r * n + b)] - vs_re) : ((double)V[2 * (r * n + b) + 1] - vs_im);
            d = Y[r * ldy + c] - (float)(kOutScale * t);
            part += d * d;
        }
        dY[e] = (__bf16)(scale * d);
    }
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
    if (loss && (threadIdx.x & 63) == 0) atomicAdd(loss, part / (float)(rows * 2 * n));
}

// bias gradient: g[c] = sum_r dZ[r][c] for c < nvalid
__global__ void colsum_kernel(const __bf16 *__restrict__ dZ, int64_t rows_pad, int Np, int nvalid,
                              float *__restrict__ g) {
    const int c = blockIdx.x;
    float s = 0.0f;
    for (int64_t r = threadIdx.x; r < rows_pad; r += blockDim.x) s += (float)dZ[r * Np + c];
    __shared__ float red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && c < nvalid) g[c] = red[0];
}

// BF16 MFMA A fragments of layer l, [T][K / 32][64 lanes][8] (lane (g, j) of fragment (t, s)
// holds row 16 t + j, inputs 32 s + 8 g .. 32 s + 8 g + 7): element (row r, input k) goes to
// ((t K/32 + s) 64 + 16 g + j) 8 + i with r = 16 t + j, k = 32 s + 8 g + i.  With
// n_out_pairs = n > 0 (the output layer) row r holds neuron (r % 2) n + r / 2, i.e. Re and
// Im of PQ bus r / 2 interleaved; otherwise row r is neuron r.  With n_in_pairs = n > 0 (the
// first layer) input k < 2 n is feature (k % 2) n + k / 2, i.e. 50 P and 50 Q of bus k / 2
// interleaved, and inputs from 2 n on (the calendar phases) keep their place.  Padding is zero.
__global__ void frag_kernel(const float *__restrict__ p, int64_t woff, int64_t boff, int in, int out, int in_p,
                            int rows, int n_out_pairs, int n_in_pairs, uint16_t *__restrict__ Wf,
                            float *__restrict__ bf) {
    const int64_t total = (int64_t)rows * in_p;
    const int ks = in_p / 32;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / in_p), k = (int)(e - (int64_t)r * in_p);
        int o = r;
        if (n_out_pairs > 0) o = r / 2 < n_out_pairs ? (r % 2) * n_out_pairs + r / 2 : out;
        int ki = k;
        if (n_in_pairs > 0 && k < 2 * n_in_pairs) ki = (k % 2) * n_in_pairs + k / 2;
        const float w = (o < out && ki < in) ? p[woff + (int64_t)o * in + ki] : 0.0f;
        const int t = r / 16, j = r % 16, s = k / 32, g = (k % 32) / 8, i = k % 8;
        const __bf16 h = (__bf16)w;
        Wf[((((int64_t)t * ks + s) * 64) + 16 * g + j) * 8 + i] = *reinterpret_cast<const uint16_t *>(&h);
        if (k == 0) bf[r] = o < out ? p[boff + o] : 0.0f;
    }
}

// ---- fused inference (every padded layer width <= 256)
//
// One workgroup of 4 waves carries a tile of 16 RT rows from the loads to the start
// voltages: features into LDS, every layer as BF16 MFMA products whose activations stay in
// LDS ([rows][264] BF16, updated in place between two barriers: the layer's outputs wait
// in the accumulators until every wave has read its inputs), and the voltage write.  Wave
// w owns output neurons 64 w .. 64 w + 63 of all rows (RT x 4 tiles of 16x16x32) and
// streams its weight fragments (the fragment copy: 1 KB contiguous per fragment) from L2
// one k-step ahead.  The weights are the products' A operand, so a lane's four outputs of
// a tile are consecutive neurons of one row: a hidden layer's leave as one 8-byte LDS
// store.  RT = 6 (96 rows, 50.7 KB of LDS) lets three workgroups share a CU, at most 168
// VGPRs each (three dwords per lane spill to scratch at that cap); 128-row tiles at two per
// CU, spill-free, measured 0.62 ms against 0.54 ms for the 100-bus year, 64-row tiles at
// four per CU 0.61 ms.  The first layer's inputs and the output
// layer's neurons are ordered (Re, Im) per bus, so each complex load of S becomes one
// 4-byte LDS write and each complex voltage two adjacent outputs; the output layer goes
// through LDS as FP32, half a tile at a time in the activations' bytes, so that the
// voltages leave as contiguous complex stores (stored straight from the accumulators,
// 128-byte pieces per row, the kernel ran twice as long).  Nothing but S and V0 touches HBM.
// Row strides of the activations (BF16) and of the output staging (FP32): 16 RT rows of
// one and 8 RT rows of the other take the same bytes.
constexpr int kFusedWidth = 256, kHStride = 264, kYStride = 264;

// Complex pairs as clang vectors, so that the streamed loads and stores can carry the
// nontemporal hint (S and V0 pass once; the weights should stay in L2).
template <typename IO>
struct Pair {
    typedef IO T __attribute__((ext_vector_type(2)));
};

struct MlpView {
    const uint16_t *W[17];  // BF16 MFMA fragments per layer (frag_kernel: interleaved first-layer
                            // inputs and output rows)
    const float *b[17];     // bias in the fragments' row order
    int T[17];              // row tiles of each layer's fragment copy
    int dp[18];             // padded widths
    int L, n;
};

// GELU with erf from Abramowitz and Stegun 7.1.26 (|error| < 1.5e-7, below the BF16
// rounding of the activation it produces).
__device__ __forceinline__ float gelu_as(float z) {
    const float x = fabsf(z) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * x);
    const float p =
        t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
    const float e = 1.0f - p * __expf(-x * x);
    return 0.5f * z * (1.0f + copysignf(e, z));
}

// GELU as z P(z) without transcendental functions: P approximates the normal CDF as
// 1/2 + y Q(y^2), y = z clamped to [-4.25, 4.25], Q a degree-8 minimax fit with P(4.25) = 1,
// and P clamped to [0, 1] (so P = 0 below -4.25 and 1 above 4.25).  |error| < 5.5e-5 |z| /
// 4.25 inside, 1.1e-5 |z| beyond: far below the BF16 rounding of the activation.
__device__ __forceinline__ float gelu_poly(float z) {
    const float y = __builtin_amdgcn_fmed3f(z, -4.25f, 4.25f);
    const float u = y * y;
    float q = 5.179778134190016e-11f;
    q = __builtin_fmaf(q, u, -5.024720195478949e-09f);
    q = __builtin_fmaf(q, u, 2.1581175246865314e-07f);
    q = __builtin_fmaf(q, u, -5.462514309328981e-06f);
    q = __builtin_fmaf(q, u, 9.186843817587942e-05f);
    q = __builtin_fmaf(q, u, -0.0011003842810168862f);
    q = __builtin_fmaf(q, u, 0.009793556295335293f);
    q = __builtin_fmaf(q, u, -0.06631755083799362f);
    q = __builtin_fmaf(q, u, 0.3988931477069855f);
    return z * __builtin_amdgcn_fmed3f(__builtin_fmaf(y, q, 0.5f), 0.0f, 1.0f);
}

template <int RT>
constexpr size_t fused_lds() {
    return (size_t)16 * RT * kHStride * 2;
}

// three workgroups per CU: at most 168 VGPRs
template <typename IO, int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void predict_fused_kernel(
    const IO *__restrict__ S, const int64_t *__restrict__ t_index, int64_t rows, const MlpView mv, double vs_re,
    double vs_im, IO *__restrict__ V0) {
    constexpr int R = 16 * RT;  // rows per workgroup
    static_assert(RT % 2 == 0, "the output layer leaves in two halves of RT / 2 row tiles");
    typedef typename Pair<IO>::T P2;
    extern __shared__ __align__(16) unsigned char smem[];
    __bf16 *H = reinterpret_cast<__bf16 *>(smem);  // [R][264]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;
    const int n = mv.n, dp0 = mv.dp[0];
    const int64_t r0 = (int64_t)blockIdx.x * R;
    const int64_t valid_rows = rows - r0 < R ? rows - r0 : R;
    // features: 50 P, 50 Q, then the calendar phases; zero padding and zero rows past the
    // end.  The tile's loads are one contiguous block of R n complex values; each thread
    // issues 16 independent loads before converting any.  Element e = 256 i + tid is
    // (row e / n, bus e % n), tracked incrementally.
    {
        const int total = R * n;
        const int64_t valid = valid_rows * (int64_t)n;
        const P2 *src = reinterpret_cast<const P2 *>(S) + r0 * n;
        int r = tid / n, b = tid - (tid / n) * n;
        const int dr = 256 / n, db = 256 - dr * n;
        for (int e0 = tid; e0 < total; e0 += 256 * 16) {
            P2 v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int e = e0 + 256 * u;
                v[u] = P2{0, 0};
                if (e < total && e < valid) v[u] = __builtin_nontemporal_load(src + e);
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                if (e0 + 256 * u < total) {  // (50 P, 50 Q) of bus b at inputs 2 b, 2 b + 1
                    const __bf16 hr = (__bf16)(kFeatScale * (float)v[u].x), hi = (__bf16)(kFeatScale * (float)v[u].y);
                    reinterpret_cast<uint32_t *>(H)[r * (kHStride / 2) + b] =
                        (uint32_t)*reinterpret_cast<const uint16_t *>(&hr) |
                        ((uint32_t)*reinterpret_cast<const uint16_t *>(&hi) << 16);
                }
                r += dr;
                b += db;
                if (b >= n) {
                    b -= n;
                    r += 1;
                }
            }
        }
        // calendar phases (one (row, phase) pair per thread per pass) and zero padding
        for (int p = tid; p < 4 * R; p += 256) {
            const int rr = p >> 2, f = 2 * n + (p & 3);
            float v = 0.0f;
            if (rr < valid_rows) {
                const int64_t t = t_index ? t_index[r0 + rr] : r0 + rr;
                const double mod = (double)(t % 1440) / 1440.0;
                const double day = (double)((t / 1440) % 365) / 365.0;
                const double ang = 2.0 * M_PI * (f < 2 * n + 2 ? mod : day);
                v = (float)(((f - 2 * n) & 1) ? cos(ang) : sin(ang));
            }
            H[rr * kHStride + f] = (__bf16)v;
        }
        for (int c = 2 * n + 4 + (tid & 63); c < dp0; c += 64)
            for (int rr = tid >> 6; rr < R; rr += 4) H[rr * kHStride + c] = (__bf16)0.0f;
    }
    __syncthreads();
    for (int l = 0; l <= mv.L; ++l) {
        const int K = mv.dp[l], T = mv.T[l];
        const int n0 = 64 * wave;
        const bool mine = 4 * wave < T;
        const bool last = l == mv.L;
        // The weights are the A operand and the activations the B operand, so that lane
        // (g, j) of product tile (a, b) accumulates neurons n0 + 16 b + 4 g .. + 3 of row
        // 16 a + j: four consecutive outputs of one row.  The accumulators start at the bias.
        const float *bias = mv.b[l];
        f4 acc[RT][4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const f4 bb = mine && 4 * wave + b < T ? *reinterpret_cast<const f4 *>(bias + n0 + 16 * b + 4 * g)
                                                    : f4{0, 0, 0, 0};
#pragma unroll
            for (int a = 0; a < RT; ++a) acc[a][b] = bb;
        }
        if (mine) {
            // weight fragments stream from L2 through two register sets, one k-step ahead
            // of the products that use them (K <= 256: at most 8 k-steps)
            const int ks = K / 32;
            // fragment (tile 4 wave + b, k-step k0 / 32): lane (g, j) holds neuron 16 t + j,
            // inputs k0 + 8 g .. k0 + 8 g + 7
            const uint16_t *Wl = mv.W[l] + (size_t)lane * 8;
            auto ldw = [&](b8(&w)[4], int k0) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int t = 4 * wave + b;
                    w[b] = t < T ? *reinterpret_cast<const b8 *>(Wl + ((size_t)t * ks + k0 / 32) * 512) : b8{};
                }
            };
            b8 w[2][4];
            ldw(w[0], 0);
#pragma unroll
            for (int st = 0; st < kFusedWidth / 32; ++st) {
                if (st < ks) {
                    if (st + 1 < ks) ldw(w[(st + 1) % 2], 32 * (st + 1));
#pragma unroll
                    for (int a = 0; a < RT; ++a) {
                        const b8 af = *reinterpret_cast<const b8 *>(H + (16 * a + j) * kHStride + 32 * st + 8 * g);
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[st % 2][b], af, acc[a][b], 0, 0, 0);
                    }
                }
            }
        }
        if (!last) {
            __syncthreads();  // every wave has read this layer's inputs
            if (mine) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
#pragma unroll
                    for (int a = 0; a < RT; ++a) {  // padding: W, b = 0 -> gelu(0) = 0
                        const b4 h = b4{(__bf16)gelu_poly(acc[a][b][0]), (__bf16)gelu_poly(acc[a][b][1]),
                                        (__bf16)gelu_poly(acc[a][b][2]), (__bf16)gelu_poly(acc[a][b][3])};
                        *reinterpret_cast<b4 *>(H + (16 * a + j) * kHStride + n0 + 16 * b + 4 * g) = h;
                    }
                }
            }
            __syncthreads();
            continue;
        }
        // output layer: half a tile (RT / 2 row tiles) at a time through the FP32 staging,
        // which takes the activations' bytes once every wave has read them, then contiguous
        // complex stores
        constexpr int HT = RT / 2, HR = 16 * HT;
        float *Yf = reinterpret_cast<float *>(smem);  // [HR][kYStride]
        __syncthreads();
        P2 *dst = reinterpret_cast<P2 *>(V0) + r0 * n;
        const double inv_scale = 1.0 / kOutScale;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (mine) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if (4 * wave + b >= T) continue;
#pragma unroll
                    for (int a = 0; a < HT; ++a)
                        *reinterpret_cast<f4 *>(Yf + (16 * a + j) * kYStride + n0 + 16 * b + 4 * g) =
                            acc[HT * half + a][b];
                }
            }
            __syncthreads();
            const int64_t rows_here = valid_rows - HR * half;
            const int64_t valid = (rows_here < HR ? rows_here : HR) * (int64_t)n;
            int r = tid / n, bus = tid - (tid / n) * n;
            const int dr = 256 / n, db = 256 - dr * n;
            for (int e = tid; e < HR * n && e < valid; e += 256) {
                const P2 o = P2{(IO)(vs_re + (double)Yf[r * kYStride + 2 * bus] * inv_scale),
                                (IO)(vs_im + (double)Yf[r * kYStride + 2 * bus + 1] * inv_scale)};
                __builtin_nontemporal_store(o, dst + (int64_t)HR * half * n + e);
                r += dr;
                bus += db;
                if (bus >= n) {
                    bus -= n;
                    r += 1;
                }
            }
            __syncthreads();  // the staging is reused by the second half
        }
    }
}

template <typename IO>
__global__ void predict_out_kernel(const float *__restrict__ Y, int64_t ldy, int n, int64_t rows, double vs_re,
                                   double vs_im, IO *__restrict__ V0) {
    const int64_t total = rows * n;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = e / n;
        const int b = (int)(e - r * n);
        V0[2 * e] = (IO)(vs_re + (double)Y[r * ldy + b] / kOutScale);
        V0[2 * e + 1] = (IO)(vs_im + (double)Y[r * ldy + n + b] / kOutScale);
    }
}

// Shuffling for mini-batch training: a pseudo-random permutation of [0, rows) per epoch,
// evaluated independently for every position.  A balanced Feistel network on 2h-bit
// integers (4 rounds, round function: the 64-bit finaliser of MurmurHash3 applied to the
// key, the round and the right half) is a bijection of [0, 4^h); "cycle walking" (apply
// it again while the value is >= rows) restricts it to a bijection of [0, rows), since
// every cycle of the permutation that starts inside [0, rows) comes back into it.  With
// 4^h < 4 rows the walk takes fewer than four steps on average.
__device__ __forceinline__ uint64_t fmix64(uint64_t k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdULL;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ULL;
    k ^= k >> 33;
    return k;
}

__device__ __forceinline__ uint64_t feistel(uint64_t x, int h, uint64_t key) {
    const uint64_t mask = (1ULL << h) - 1;
    uint64_t L = x >> h, R = x & mask;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint64_t F = fmix64(key ^ (0x9e3779b97f4a7c15ULL * (uint64_t)(r + 1)) ^ (R << 8)) & mask;
        const uint64_t T = L ^ F;
        L = R;
        R = T;
    }
    return (L << h) | R;
}

__device__ __forceinline__ int64_t shuffled_row(int64_t i, int64_t rows, int h, uint64_t key) {
    uint64_t x = (uint64_t)i;
    do {
        x = feistel(x, h, key);
    } while (x >= (uint64_t)rows);
    return (int64_t)x;
}

// Rows first .. first + count - 1 of an epoch's order: S, V (n complex each) and t into
// the contiguous batch buffers.
template <typename IO>
__global__ void gather_rows_kernel(const IO *__restrict__ S, const IO *__restrict__ V,
                                   const int64_t *__restrict__ t_index, int64_t rows, int n, int64_t first,
                                   int64_t count, int h, uint64_t key, IO *__restrict__ Sb, IO *__restrict__ Vb,
                                   int64_t *__restrict__ tb) {
    // one wavefront per row: the permuted index is computed once and the row copied by 64 lanes
    const int64_t r = blockIdx.x * (int64_t)(blockDim.x / 64) + threadIdx.x / 64;
    const int lane = threadIdx.x & 63;
    if (r >= count) return;
    const int64_t src = shuffled_row(first + r, rows, h, key);
    if (lane == 0) tb[r] = t_index[src];
    for (int e = lane; e < 2 * n; e += 64) {
        Sb[r * 2 * n + e] = S[src * 2 * n + e];
        Vb[r * 2 * n + e] = V[src * 2 * n + e];
    }
}

// acc[0] += loss[0] * scale (one lane)
__global__ void loss_accum_kernel(const float *__restrict__ loss, float *__restrict__ acc, float scale) {
    if (threadIdx.x == 0 && blockIdx.x == 0) acc[0] += loss[0] * scale;
}

__global__ void zero_f32_kernel(float *p, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0f;
}

unsigned grid_for(int64_t work, int64_t per_block = 256) {
    const int64_t b = (work + per_block - 1) / per_block;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 65536));
}

}  // namespace
}  // namespace tpf

#include "mlp_train.h"

namespace tpf {
namespace {

// BF16 copies of layer l's weights, zero in the padding: W for X W^T, and with `chain` also W^T
// for dZ W, both in the chain kernel's fragment order (else W row-major [out_p][in_p]).
__global__ void sync_kernel(const float *__restrict__ p, int64_t woff, int in, int out, int in_p, int out_p,
                            __bf16 *__restrict__ Wt, __bf16 *__restrict__ Wn, float *__restrict__ bias_p,
                            int64_t boff, bool chain) {
    const int64_t total = (int64_t)in_p * out_p;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int o = (int)(e / in_p), i = (int)(e - (int64_t)o * in_p);
        const float w = (o < out && i < in) ? p[woff + (int64_t)o * in + i] : 0.0f;
        Wt[chain ? frag_place(o, i, in_p) : e] = (__bf16)w;
        if (chain) Wn[frag_place(i, o, out_p)] = (__bf16)w;
        if (i == 0) bias_p[o] = o < out ? p[boff + o] : 0.0f;
    }
}

}  // namespace
}  // namespace tpf

using namespace tpf;

struct tpf_mlp_s {
    int n = 0, hidden = 0, layers = 0;  // layers = hidden layers
    int device = 0;
    double vs_re = 1.0, vs_im = 0.0;
    std::vector<int> d, dp;              // widths and padded widths, L+2 entries
    std::vector<int64_t> woff, boff;     // offsets in the flat vector
    int64_t P = 0;
    int64_t step = 0;                    // AdamW steps taken
    float *p = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;  // device FP32 [P]
    std::vector<__bf16 *> Wt, Wn;        // device BF16 copies per layer (sync_kernel)
    std::vector<float *> bias;           // device padded FP32 bias per layer
    std::vector<uint16_t *> Wf;          // BF16 MFMA A fragments per layer (frag_kernel)
    std::vector<float *> bf;             // bias in the fragments' row order
    std::vector<int> frows;              // rows of the fragment copy per layer (16 T)
    std::vector<void *> owned;
};

namespace {

int64_t rows_pad(int64_t rows) { return (rows + 63) / 64 * 64; }

// Workspace carving: X/activations bf16 [rows_pad][Dmax] x (L+1), pre-activations f32
// [rows_pad][Dmax] x L, output f32 [rows_pad][Dout], gradient scratch bf16 x 2, and the
// buffers of one gathered training batch (S, V, minute index) for tpf_mlp_train; for the
// chain kernel the transposed gradients of every layer.
struct MlpWs {
    std::vector<__bf16 *> H;   // H[0] = X, H[l] = activation of hidden layer l
    std::vector<float *> Z;    // Z[l] pre-activation of hidden layer l (1-based, l = 1..L)
    float *Y = nullptr;
    __bf16 *G0 = nullptr, *G1 = nullptr;
    std::vector<__bf16 *> GT;  // every layer's output gradient, transposed (chain kernel)
    float *loss = nullptr;     // the loss, or the chain kernel's partial losses (one per kChainRows rows)
    void *Sb = nullptr, *Vb = nullptr;  // a gathered training batch [rows][n] complex (up to complex128)
    int64_t *tb = nullptr;              // its minute indices, or the chain kernel's row order
    float *phase = nullptr;             // the chain kernel's calendar phases [rows][4]
};

size_t carve(const tpf_mlp_s &M, int64_t rows, void *base, MlpWs *ws) {
    const int64_t rp = rows_pad(rows);
    int Dmax = 0;
    for (int w : M.dp) Dmax = std::max(Dmax, w);
    size_t off = 0;
    auto take = [&](size_t bytes) -> char * {
        char *ptr = base ? static_cast<char *>(base) + off : nullptr;
        off += (bytes + 255) / 256 * 256;
        return ptr;
    };
    const int L = M.layers;
    if (ws) ws->H.assign(L + 1, nullptr), ws->Z.assign(L + 1, nullptr);
    for (int l = 0; l <= L; ++l) {
        char *q = take((size_t)rp * Dmax * 2);
        if (ws) ws->H[l] = reinterpret_cast<__bf16 *>(q);
    }
    for (int l = 1; l <= L; ++l) {
        char *q = take((size_t)rp * Dmax * 4);
        if (ws) ws->Z[l] = reinterpret_cast<float *>(q);
    }
    char *y = take((size_t)rp * Dmax * 4);
    char *g0 = take((size_t)rp * Dmax * 2);
    char *g1 = take((size_t)rp * Dmax * 2);
    if (ws) ws->GT.assign(L + 1, nullptr);
    if (Dmax <= kChainWidth)
        for (int l = 0; l <= L; ++l) {
            char *q = take((size_t)rp * Dmax * 2);
            if (ws) ws->GT[l] = reinterpret_cast<__bf16 *>(q);
        }
    char *ls = take((size_t)rp / kChainRows * 4 + 256);
    char *sb = take((size_t)rows * M.n * 16);
    char *vb = take((size_t)rows * M.n * 16);
    char *tb = take((size_t)rows * 8);
    char *ph = take((size_t)rows * 16);
    if (ws) {
        ws->Y = reinterpret_cast<float *>(y);
        ws->G0 = reinterpret_cast<__bf16 *>(g0);
        ws->G1 = reinterpret_cast<__bf16 *>(g1);
        ws->loss = reinterpret_cast<float *>(ls);
        ws->Sb = sb;
        ws->Vb = vb;
        ws->tb = reinterpret_cast<int64_t *>(tb);
        ws->phase = reinterpret_cast<float *>(ph);
    }
    return off;
}

int check_device(const tpf_mlp_s &M) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return fail(TPF_ERR_DEVICE, "hipGetDevice failed");
    if (dev != M.device) return fail(TPF_ERR_INVALID_ARG, "the MLP handle belongs to another device");
    return TPF_OK;
}

int last_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(TPF_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
    return TPF_OK;
}

// Whether the three-kernel training step applies.
bool chain_fits(const tpf_mlp_s &M) {
    int Dmax = 0;
    for (int w : M.dp) Dmax = std::max(Dmax, w);
    return Dmax <= kChainWidth;
}

int sync_weights(tpf_mlp_s &M, hipStream_t st) {
    for (int l = 0; l <= M.layers; ++l) {
        hipLaunchKernelGGL(sync_kernel, dim3(grid_for((int64_t)M.dp[l] * M.dp[l + 1])), dim3(256), 0, st, M.p,
                           M.woff[l], M.d[l], M.d[l + 1], M.dp[l], M.dp[l + 1], M.Wt[l], M.Wn[l], M.bias[l],
                           M.boff[l], chain_fits(M));
        hipLaunchKernelGGL(frag_kernel, dim3(grid_for((int64_t)M.frows[l] * M.dp[l])), dim3(256), 0, st, M.p,
                           M.woff[l], M.boff[l], M.d[l], M.d[l + 1], M.dp[l], M.frows[l], l == M.layers ? M.n : 0,
                           l == 0 ? M.n : 0, M.Wf[l], M.bf[l]);
    }
    return last_launch("weight sync");
}

// One AdamW step of the FP32 master parameters with the gradient in M.grad (step count
// advanced first: the bias corrections use t = 1 on the first step), then the BF16 copies.
// The partial losses in `lossp`, when given, are summed and added to acc times scale.
int adamw_update(tpf_mlp_s &M, float lr, float wd, hipStream_t st, const float *lossp = nullptr, int loss_n = 0,
                 float *acc = nullptr, float scale = 0.0f) {
    M.step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float bc1 = 1.0f - (float)std::pow((double)b1, (double)M.step);
    const float bc2 = 1.0f - (float)std::pow((double)b2, (double)M.step);
    ParamView pv{};
    pv.L = M.layers;
    pv.n = M.n;
    pv.chain = chain_fits(M);
    for (int l = 0; l <= M.layers; ++l) {
        pv.Wt[l] = M.Wt[l];
        pv.Wn[l] = M.Wn[l];
        pv.Wf[l] = M.Wf[l];
        pv.bias[l] = M.bias[l];
        pv.bf[l] = M.bf[l];
        pv.woff[l] = M.woff[l];
        pv.boff[l] = M.boff[l];
    }
    pv.woff[M.layers + 1] = M.P;
    for (int l = 0; l < M.layers + 2; ++l) pv.d[l] = M.d[l], pv.dp[l] = M.dp[l];
    hipLaunchKernelGGL(adamw_sync_kernel, dim3(grid_for(M.P)), dim3(256), 0, st, M.p, M.grad, M.m, M.v, pv, lr, wd, b1,
                       b2, 1e-8f, bc1, bc2, lossp, loss_n, acc, scale);
    return last_launch("AdamW");
}

// The shuffle key of an epoch: MurmurHash3's 64-bit finaliser of the seed and epoch.
uint64_t fmix64_host(uint64_t k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdULL;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ULL;
    k ^= k >> 33;
    return k;
}

template <bool AK, bool BK, int EP>
void gemm(const __bf16 *A, int64_t sam, int64_t sak, const __bf16 *B, int64_t sbk, int64_t sbn, int64_t Mrows,
          int N, int K, const float *bias, float *Cf, __bf16 *Cb, int64_t ldc, const float *Z, int64_t ldz, int vm,
          int vn, int64_t goff, hipStream_t st) {
    hipLaunchKernelGGL((gemm_bf16_kernel<AK, BK, EP>), dim3((unsigned)(Mrows / 64), (unsigned)(N / 64)), dim3(256),
                       0, st, A, sam, sak, B, sbk, sbn, K, bias, Cf, Cb, ldc, Z, ldz, vm, vn, goff);
}

// The rows of a batch (of a shuffled set with sh.h > 0) for the chain kernel.
BatchRows batch_rows(const MlpWs &ws, const int64_t *t, int64_t rows, const Shuffle &sh) {
    return BatchRows{t, ws.tb, ws.phase, rows, sh};
}

void launch_batch_rows(const BatchRows &br, hipStream_t st) {
    hipLaunchKernelGGL(batch_rows_kernel, dim3((unsigned)((br.rows + 31) / 32)), dim3(128), 0, st, br);
}

// Loss partials and gradient of the prepared batch of `rows` rows by the chain and
// weight-gradient kernels; the latter prepares the batch `next` (rows = 0: none).
template <typename IO>
int chain_loss_grad(tpf_mlp_s &M, const IO *S, const IO *V, int64_t rows, const BatchRows &next, float *gout,
                    const MlpWs &ws, hipStream_t st) {
    const int64_t rp = rows_pad(rows);
    TrainView tv{};
    GradView gv{};
    tv.L = gv.L = M.layers;
    tv.n = M.n;
    int tiles = 0, cols = 0;
    for (int l = 0; l <= M.layers; ++l) {
        tv.Wt[l] = M.Wt[l];
        tv.Wn[l] = M.Wn[l];
        tv.b[l] = M.bias[l];
        tv.HT[l] = ws.H[l];
        tv.GT[l] = ws.GT[l];
        tv.Z[l] = l ? ws.Z[l] : nullptr;
        gv.HT[l] = ws.H[l];
        gv.GT[l] = ws.GT[l];
        gv.woff[l] = M.woff[l];
        gv.boff[l] = M.boff[l];
        gv.tile0[l] = tiles;
        gv.col0[l] = cols;
        tiles += M.dp[l + 1] / 64 * (M.dp[l] / 16);
        cols += M.d[l + 1];
    }
    gv.tile0[M.layers + 1] = tiles;
    gv.col0[M.layers + 1] = cols;
    for (int l = 0; l < M.layers + 2; ++l) tv.d[l] = gv.d[l] = M.d[l], tv.dp[l] = gv.dp[l] = M.dp[l];
    hipLaunchKernelGGL(train_chain_kernel<IO>, dim3((unsigned)(rp / kChainRows)), dim3(kChainThreads), 0, st, S, V,
                       ws.tb, ws.phase, rows, rp, tv, M.vs_re, M.vs_im, ws.loss);
    hipLaunchKernelGGL(train_dw_kernel, dim3((unsigned)(tiles + (cols + 1) / 2 + (next.rows + 31) / 32)), dim3(128), 0,
                       st, gv, (int)rp, gout, next);
    return last_launch("MLP training step");
}

template <typename IO>
int forward(tpf_mlp_s &M, const IO *S, const int64_t *t, int64_t rows, const MlpWs &ws, hipStream_t st) {
    const int64_t rp = rows_pad(rows);
    int Dmax = 0;
    for (int w : M.dp) Dmax = std::max(Dmax, w);
    hipLaunchKernelGGL(features_kernel<IO>, dim3(grid_for(rp * M.dp[0])), dim3(256), 0, st, S, t, M.n, rows, rp,
                       M.dp[0], ws.H[0]);
    // H[0] is [rp][dp0] packed; later layers use row stride Dmax
    for (int l = 0; l < M.layers; ++l) {
        const int64_t lda = l == 0 ? M.dp[0] : Dmax;
        gemm<true, true, EP_HIDDEN>(ws.H[l], lda, 1, M.Wt[l], 1, M.dp[l], rp, M.dp[l + 1], M.dp[l], M.bias[l],
                                    ws.Z[l + 1], ws.H[l + 1], Dmax, nullptr, 0, 0, M.d[l + 1], 0, st);
    }
    const int L = M.layers;
    const int64_t lda = L == 0 ? M.dp[0] : Dmax;
    gemm<true, true, EP_OUT>(ws.H[L], lda, 1, M.Wt[L], 1, M.dp[L], rp, M.dp[L + 1], M.dp[L], M.bias[L], ws.Y, nullptr,
                             Dmax, nullptr, 0, 0, 0, 0, st);
    return last_launch("MLP forward");
}

template <typename IO>
int loss_grad(tpf_mlp_s &M, const IO *S, const int64_t *t, const IO *V, int64_t rows, float *loss_out, float *gout,
              const MlpWs &ws, hipStream_t st) {
    if (chain_fits(M)) {
        launch_batch_rows(batch_rows(ws, t, rows, Shuffle{}), st);
        int rc = chain_loss_grad(M, S, V, rows, BatchRows{}, gout, ws, st);
        if (rc != TPF_OK || !loss_out) return rc;
        hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(64), 0, st, ws.loss, (int)(rows_pad(rows) / kChainRows),
                           loss_out);
        return last_launch("MLP loss");
    }
    int rc = forward(M, S, t, rows, ws, st);
    if (rc != TPF_OK) return rc;
    const int64_t rp = rows_pad(rows);
    int Dmax = 0;
    for (int w : M.dp) Dmax = std::max(Dmax, w);
    const int L = M.layers;
    hipLaunchKernelGGL(zero_f32_kernel, dim3(1), dim3(64), 0, st, ws.loss, (int64_t)1);
    // dY [rp][dp_{L+1}] (row stride Dmax) into G0
    hipLaunchKernelGGL(output_grad_kernel<IO>, dim3(grid_for(rp * M.dp[L + 1])), dim3(256), 0, st, ws.Y,
                       (int64_t)Dmax, V, M.n, rows, rp, M.dp[L + 1], M.vs_re, M.vs_im, ws.G0, ws.loss);
    // output_grad writes packed [rp][dp_{L+1}]; keep that stride for the output layer
    int64_t ldg = M.dp[L + 1];
    __bf16 *Gc = ws.G0, *Gn = ws.G1;
    for (int l = L; l >= 0; --l) {
        const int in_p = M.dp[l], out_p = M.dp[l + 1];
        const __bf16 *Hin = ws.H[l];
        const int64_t ldh = l == 0 ? M.dp[0] : Dmax;
        // dW_l [out][in] = dZ^T H : C[o][i] = sum_r dZ[r][o] H[r][i]
        gemm<false, false, EP_DW>(Gc, 1, ldg, Hin, ldh, 1, out_p, in_p, (int)rp, nullptr, gout, nullptr, 0,
                                  nullptr, 0, M.d[l + 1], M.d[l], M.woff[l], st);
        hipLaunchKernelGGL(colsum_kernel, dim3(M.d[l + 1]), dim3(256), 0, st, Gc, rp, (int)ldg, M.d[l + 1],
                           gout + M.boff[l]);
        if (l > 0) {
            // dZ_{l-1} = (dZ_l W_l) .* gelu'(Z_l-1) : C[r][i] = sum_o dZ[r][o] W[o][i]
            gemm<true, false, EP_DGELU>(Gc, ldg, 1, M.Wt[l], in_p, 1, rp, in_p, out_p, nullptr, nullptr, Gn, Dmax,
                                        ws.Z[l], Dmax, 0, M.d[l], 0, st);
            std::swap(Gc, Gn);
            ldg = Dmax;
        }
    }
    if (loss_out)
        (void)hipMemcpyAsync(loss_out, ws.loss, sizeof(float), hipMemcpyDeviceToDevice, st);
    return last_launch("MLP backward");
}

}  // namespace

extern "C" int tpf_mlp_create(int32_t n_pq, int32_t hidden, int32_t layers, const float *params, double vs_re,
                              double vs_im, tpf_mlp *out) {
    clear_error();
    if (!out) return fail(TPF_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (n_pq < 1 || hidden < 1 || layers < 0 || layers > 16 || hidden > 4096 || n_pq > 4096)
        return fail(TPF_ERR_INVALID_ARG, "bad MLP sizes");
    auto *M = new (std::nothrow) tpf_mlp_s();
    if (!M) return fail(TPF_ERR_OOM, "host allocation failed");
    if (hipGetDevice(&M->device) != hipSuccess) {
        delete M;
        return fail(TPF_ERR_DEVICE, "hipGetDevice failed (no GPU?)");
    }
    M->n = n_pq;
    M->hidden = hidden;
    M->layers = layers;
    M->vs_re = vs_re;
    M->vs_im = vs_im;
    M->d.push_back(2 * n_pq + 4);
    for (int l = 0; l < layers; ++l) M->d.push_back(hidden);
    M->d.push_back(2 * n_pq);
    for (int w : M->d) M->dp.push_back(padw(w));
    int64_t o = 0;
    for (int l = 0; l <= layers; ++l) {
        M->woff.push_back(o);
        o += (int64_t)M->d[l] * M->d[l + 1];
        M->boff.push_back(o);
        o += M->d[l + 1];
    }
    M->P = o;
    auto dalloc = [&](void **ptr, size_t bytes) -> bool {
        if (hipMalloc(ptr, bytes) != hipSuccess) return false;
        M->owned.push_back(*ptr);
        return true;
    };
    bool ok = dalloc((void **)&M->p, M->P * 4) && dalloc((void **)&M->m, M->P * 4) &&
              dalloc((void **)&M->v, M->P * 4) && dalloc((void **)&M->grad, M->P * 4);
    M->Wt.resize(layers + 1);
    M->Wn.resize(layers + 1);
    M->bias.resize(layers + 1);
    M->Wf.resize(layers + 1);
    M->bf.resize(layers + 1);
    M->frows.resize(layers + 1);
    for (int l = 0; l <= layers; ++l) M->frows[l] = l < layers ? M->dp[l + 1] : 16 * ((n_pq + 7) / 8);
    for (int l = 0; ok && l <= layers; ++l)
        ok = dalloc((void **)&M->Wt[l], (size_t)M->dp[l] * M->dp[l + 1] * 2) &&
             dalloc((void **)&M->Wn[l], (size_t)M->dp[l] * M->dp[l + 1] * 2) &&
             dalloc((void **)&M->bias[l], (size_t)M->dp[l + 1] * 4) &&
             dalloc((void **)&M->Wf[l], (size_t)M->dp[l] * M->frows[l] * 2) &&
             dalloc((void **)&M->bf[l], (size_t)M->frows[l] * 4);
    if (!ok) {
        tpf_mlp_free(M);
        return fail(TPF_ERR_OOM, "device allocation failed (MLP)");
    }
    std::vector<float> host(M->P, 0.0f);
    if (params) std::memcpy(host.data(), params, M->P * 4);
    std::vector<float> zeros(M->P, 0.0f);
    if (hipMemcpy(M->p, host.data(), M->P * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(M->m, zeros.data(), M->P * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(M->v, zeros.data(), M->P * 4, hipMemcpyHostToDevice) != hipSuccess) {
        tpf_mlp_free(M);
        return fail(TPF_ERR_DEVICE, "host-to-device copy failed (MLP)");
    }
    int rc = sync_weights(*M, nullptr);
    if (rc == TPF_OK && hipDeviceSynchronize() != hipSuccess) rc = fail(TPF_ERR_DEVICE, "MLP init failed");
    if (rc != TPF_OK) {
        tpf_mlp_free(M);
        return rc;
    }
    *out = M;
    return TPF_OK;
}

extern "C" void tpf_mlp_free(tpf_mlp M) {
    if (!M) return;
    for (void *ptr : M->owned) (void)hipFree(ptr);
    delete M;
}

extern "C" int64_t tpf_mlp_num_params(tpf_mlp M) { return M ? M->P : fail(TPF_ERR_INVALID_ARG, "mlp is NULL"); }

extern "C" int tpf_mlp_get_params(tpf_mlp M, float *params_out) {
    clear_error();
    if (!M || !params_out) return fail(TPF_ERR_INVALID_ARG, "NULL argument");
    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(params_out, M->p, M->P * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return fail(TPF_ERR_DEVICE, "device-to-host copy failed");
    return TPF_OK;
}

extern "C" int tpf_mlp_set_params(tpf_mlp M, const float *params) {
    clear_error();
    if (!M || !params) return fail(TPF_ERR_INVALID_ARG, "NULL argument");
    int rc = check_device(*M);
    if (rc != TPF_OK) return rc;
    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(M->p, params, M->P * 4, hipMemcpyHostToDevice) != hipSuccess)
        return fail(TPF_ERR_DEVICE, "host-to-device copy failed");
    rc = sync_weights(*M, nullptr);
    if (rc == TPF_OK && hipDeviceSynchronize() != hipSuccess) rc = fail(TPF_ERR_DEVICE, "weight sync failed");
    return rc;
}

extern "C" size_t tpf_mlp_workspace_bytes(tpf_mlp M, int64_t rows) {
    if (!M || rows < 0) return 0;
    return carve(*M, std::max<int64_t>(rows, 1), nullptr, nullptr);
}

// Argument checks shared by the MLP calls; the workspace must hold ws_rows rows (the
// rows of the call, or one batch for tpf_mlp_train).
static int mlp_args(tpf_mlp M, const void *S, int32_t dtype, const int64_t *t, int64_t rows, void *ws, size_t wsb,
                    int64_t ws_rows = -1) {
    if (ws_rows < 0) ws_rows = rows;
    if (!M) return fail(TPF_ERR_INVALID_ARG, "mlp is NULL");
    if (dtype != TPF_C64 && dtype != TPF_C128) return fail(TPF_ERR_INVALID_ARG, "bad dtype");
    if (rows < 0 || rows > ((int64_t)1 << 31)) return fail(TPF_ERR_INVALID_ARG, "bad row count");
    if (rows > 0 && (!S || !t)) return fail(TPF_ERR_INVALID_ARG, "NULL array");
    if (rows > 0 && (!ws || wsb < tpf_mlp_workspace_bytes(M, ws_rows)))
        return fail(TPF_ERR_INVALID_ARG, "workspace missing or smaller than tpf_mlp_workspace_bytes()");
    return check_device(*M);
}

extern "C" int tpf_mlp_loss_grad(tpf_mlp M, const void *S, int32_t dtype, const int64_t *t_index, const void *V,
                                 int64_t rows, float *loss_out, float *grad_out, void *workspace,
                                 size_t workspace_bytes, void *stream) {
    clear_error();
    int rc = mlp_args(M, S, dtype, t_index, rows, workspace, workspace_bytes);
    if (rc != TPF_OK) return rc;
    if (rows == 0) return fail(TPF_ERR_INVALID_ARG, "a gradient needs at least one row");
    if (!V || !grad_out) return fail(TPF_ERR_INVALID_ARG, "NULL array");
    MlpWs ws;
    carve(*M, rows, workspace, &ws);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (dtype == TPF_C128)
        return loss_grad(*M, (const double *)S, t_index, (const double *)V, rows, loss_out, grad_out, ws, st);
    return loss_grad(*M, (const float *)S, t_index, (const float *)V, rows, loss_out, grad_out, ws, st);
}

extern "C" int tpf_mlp_train_step(tpf_mlp M, const void *S, int32_t dtype, const int64_t *t_index, const void *V,
                                  int64_t rows, float lr, float weight_decay, float *loss_out, void *workspace,
                                  size_t workspace_bytes, void *stream) {
    clear_error();
    if (!(lr >= 0.0f) || !(weight_decay >= 0.0f)) return fail(TPF_ERR_INVALID_ARG, "lr and weight_decay must be >= 0");
    int rc = tpf_mlp_loss_grad(M, S, dtype, t_index, V, rows, loss_out, M ? M->grad : nullptr, workspace,
                               workspace_bytes, stream);
    if (rc != TPF_OK) return rc;
    return adamw_update(*M, lr, weight_decay, reinterpret_cast<hipStream_t>(stream));
}

extern "C" int tpf_mlp_train(tpf_mlp M, const void *S, int32_t dtype, const int64_t *t_index, const void *V,
                             int64_t rows, int32_t first_epoch, int32_t epochs, int32_t total_epochs, int32_t batch,
                             float lr, float lr_min, float weight_decay, uint64_t seed, float *epoch_loss_out,
                             void *workspace, size_t workspace_bytes, void *stream) {
    clear_error();
    if (batch < 1) return fail(TPF_ERR_INVALID_ARG, "batch must be >= 1");
    if (rows < 1) return fail(TPF_ERR_INVALID_ARG, "training needs at least one row");
    const int64_t B = std::min<int64_t>(batch, rows);
    int rc = mlp_args(M, S, dtype, t_index, rows, workspace, workspace_bytes, B);
    if (rc != TPF_OK) return rc;
    if (!V) return fail(TPF_ERR_INVALID_ARG, "NULL array");
    if (first_epoch < 0 || epochs < 0 || total_epochs < 1 || first_epoch + (int64_t)epochs > total_epochs)
        return fail(TPF_ERR_INVALID_ARG, "need 0 <= first_epoch, 0 <= epochs, first_epoch + epochs <= total_epochs");
    if (!(lr >= 0.0f) || !(lr_min >= 0.0f) || !(weight_decay >= 0.0f))
        return fail(TPF_ERR_INVALID_ARG, "lr, lr_min and weight_decay must be >= 0");
    MlpWs ws;
    carve(*M, B, workspace, &ws);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int64_t nb = rows / B;  // batches per epoch; the rows past nb * B sit out the epoch
    const double total = (double)total_epochs * (double)nb;
    int h = 1;
    while (h < 32 && ((uint64_t)1 << (2 * h)) < (uint64_t)rows) ++h;
    for (int32_t e = first_epoch; e < first_epoch + epochs; ++e) {
        float *acc = epoch_loss_out ? epoch_loss_out + (e - first_epoch) : nullptr;
        if (acc) hipLaunchKernelGGL(zero_f32_kernel, dim3(1), dim3(64), 0, st, acc, (int64_t)1);
        const uint64_t key = fmix64_host(seed * 0x100000001b3ULL + (uint64_t)e);
        for (int64_t b = 0; b < nb; ++b) {
            const double k = (double)e * (double)nb + (double)b;
            const double rate = (double)lr_min + 0.5 * ((double)lr - (double)lr_min) *
                                                     (1.0 + std::cos(M_PI * k / std::max(1.0, total - 1.0)));
            if (chain_fits(*M)) {
                if (b == 0) launch_batch_rows(batch_rows(ws, t_index, B, Shuffle{rows, 0, key, h}), st);
                const BatchRows next =
                    b + 1 < nb ? batch_rows(ws, t_index, B, Shuffle{rows, (b + 1) * B, key, h}) : BatchRows{};
                rc = dtype == TPF_C128
                         ? chain_loss_grad(*M, (const double *)S, (const double *)V, B, next, M->grad, ws, st)
                         : chain_loss_grad(*M, (const float *)S, (const float *)V, B, next, M->grad, ws, st);
                if (rc != TPF_OK) return rc;
                rc = adamw_update(*M, (float)rate, weight_decay, st, ws.loss, (int)(rows_pad(B) / kChainRows), acc,
                                  1.0f / (float)nb);
                if (rc != TPF_OK) return rc;
                continue;
            }
            const unsigned blocks = (unsigned)((B + 3) / 4);
            if (dtype == TPF_C128) {
                hipLaunchKernelGGL(gather_rows_kernel<double>, dim3(blocks), dim3(256), 0, st, (const double *)S,
                                   (const double *)V, t_index, rows, M->n, b * B, B, h, key, (double *)ws.Sb,
                                   (double *)ws.Vb, ws.tb);
                rc = loss_grad(*M, (const double *)ws.Sb, ws.tb, (const double *)ws.Vb, B, nullptr, M->grad, ws, st);
            } else {
                hipLaunchKernelGGL(gather_rows_kernel<float>, dim3(blocks), dim3(256), 0, st, (const float *)S,
                                   (const float *)V, t_index, rows, M->n, b * B, B, h, key, (float *)ws.Sb,
                                   (float *)ws.Vb, ws.tb);
                rc = loss_grad(*M, (const float *)ws.Sb, ws.tb, (const float *)ws.Vb, B, nullptr, M->grad, ws, st);
            }
            if (rc != TPF_OK) return rc;
            if (acc) hipLaunchKernelGGL(loss_accum_kernel, dim3(1), dim3(64), 0, st, ws.loss, acc, 1.0f / (float)nb);
            rc = adamw_update(*M, (float)rate, weight_decay, st);
            if (rc != TPF_OK) return rc;
        }
    }
    return last_launch("MLP training");
}

namespace {

bool fused_predict_fits(const tpf_mlp_s &M) {
    int Dmax = 0;
    for (int w : M.dp) Dmax = std::max(Dmax, w);
    return Dmax <= kFusedWidth && 2 * M.n + 4 <= M.dp[0];
}

// V0 for `rows` rows: the fused kernel when every padded width is <= 256, else the
// layer-by-layer GEMMs in the carved workspace `ws`.  t_index may be NULL (t = row).
int predict_impl(tpf_mlp_s &M, const void *S, int32_t dtype, const int64_t *t_index, int64_t rows, void *V0_out,
                 void *workspace, hipStream_t st) {
    if (fused_predict_fits(M)) {
        MlpView mv{};
        for (int l = 0; l <= M.layers; ++l) {
            mv.W[l] = M.Wf[l];
            mv.b[l] = M.bf[l];
            mv.T[l] = M.frows[l] / 16;
        }
        for (int l = 0; l < M.layers + 2; ++l) mv.dp[l] = M.dp[l];
        mv.L = M.layers;
        mv.n = M.n;
        constexpr int RT = 6;
        constexpr size_t lds = fused_lds<RT>();
        const unsigned blocks = (unsigned)((rows + 16 * RT - 1) / (16 * RT));
        if (dtype == TPF_C128) {
            auto k = predict_fused_kernel<double, RT>;
            if (hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
                hipSuccess)
                return fail(TPF_ERR_DEVICE, "hipFuncSetAttribute failed");
            hipLaunchKernelGGL(k, dim3(blocks), dim3(256), lds, st, (const double *)S, t_index, rows, mv, M.vs_re,
                               M.vs_im, (double *)V0_out);
        } else {
            auto k = predict_fused_kernel<float, RT>;
            if (hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
                hipSuccess)
                return fail(TPF_ERR_DEVICE, "hipFuncSetAttribute failed");
            hipLaunchKernelGGL(k, dim3(blocks), dim3(256), lds, st, (const float *)S, t_index, rows, mv, M.vs_re,
                               M.vs_im, (float *)V0_out);
        }
        return last_launch("MLP fused predict");
    }
    MlpWs ws;
    carve(M, rows, workspace, &ws);
    int Dmax = 0;
    for (int w : M.dp) Dmax = std::max(Dmax, w);
    int rc;
    if (dtype == TPF_C128) {
        rc = forward(M, (const double *)S, t_index, rows, ws, st);
        if (rc == TPF_OK)
            hipLaunchKernelGGL(predict_out_kernel<double>, dim3(grid_for(rows * M.n)), dim3(256), 0, st, ws.Y,
                               (int64_t)Dmax, M.n, rows, M.vs_re, M.vs_im, (double *)V0_out);
    } else {
        rc = forward(M, (const float *)S, t_index, rows, ws, st);
        if (rc == TPF_OK)
            hipLaunchKernelGGL(predict_out_kernel<float>, dim3(grid_for(rows * M.n)), dim3(256), 0, st, ws.Y,
                               (int64_t)Dmax, M.n, rows, M.vs_re, M.vs_im, (float *)V0_out);
    }
    if (rc != TPF_OK) return rc;
    return last_launch("MLP predict");
}

}  // namespace

extern "C" int tpf_mlp_predict(tpf_mlp M, const void *S, int32_t dtype, const int64_t *t_index, int64_t rows,
                               void *V0_out, void *workspace, size_t workspace_bytes, void *stream) {
    clear_error();
    int rc = mlp_args(M, S, dtype, t_index, rows, workspace, workspace_bytes);
    if (rc != TPF_OK) return rc;
    if (rows == 0) return TPF_OK;
    if (!V0_out) return fail(TPF_ERR_INVALID_ARG, "NULL array");
    return predict_impl(*M, S, dtype, t_index, rows, V0_out, workspace, reinterpret_cast<hipStream_t>(stream));
}

namespace tpf {

size_t mlp_predict_scratch_bytes(tpf_mlp M, int64_t rows) {
    if (!M || fused_predict_fits(*M)) return 0;
    return carve(*M, std::max<int64_t>(rows, 1), nullptr, nullptr);
}

int mlp_predict_into(tpf_mlp M, const void *S, int dtype, const int64_t *t_index, int64_t rows, void *V0,
                     void *scratch, hipStream_t stream) {
    if (!M) return fail(TPF_ERR_INVALID_ARG, "warm-start network is NULL");
    int rc = check_device(*M);
    if (rc != TPF_OK) return rc;
    if (rows == 0) return TPF_OK;
    return predict_impl(*M, S, dtype, t_index, rows, V0, scratch, stream);
}

}  // namespace tpf

namespace {
// Parameter file: header, then the FP32 master parameters, the AdamW first and second
// moments (each [P] float32).  Version 01 files (parameters only) load with a restarted
// optimiser: step 0 and zero moments, so that the next step's bias corrections match.
struct MlpFileHeader {
    char magic[8];
    int32_t n, hidden, layers, reserved;
    double vs_re, vs_im;
    int64_t step, P;
};
constexpr char kMagicV1[9] = "TPFMLP01", kMagicV2[9] = "TPFMLP02";
}  // namespace

extern "C" int tpf_mlp_save(tpf_mlp M, const char *path) {
    clear_error();
    if (!M || !path) return fail(TPF_ERR_INVALID_ARG, "NULL argument");
    std::vector<float> host(3 * M->P);
    if (hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(host.data(), M->p, M->P * 4, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(host.data() + M->P, M->m, M->P * 4, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(host.data() + 2 * M->P, M->v, M->P * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return fail(TPF_ERR_DEVICE, "device-to-host copy failed");
    MlpFileHeader h{};
    std::memcpy(h.magic, kMagicV2, 8);
    h.n = M->n;
    h.hidden = M->hidden;
    h.layers = M->layers;
    h.vs_re = M->vs_re;
    h.vs_im = M->vs_im;
    h.step = M->step;
    h.P = M->P;
    FILE *f = std::fopen(path, "wb");
    if (!f) return fail(TPF_ERR_INVALID_ARG, std::string("cannot open ") + path);
    const bool ok = std::fwrite(&h, sizeof h, 1, f) == 1 && std::fwrite(host.data(), 4, 3 * M->P, f) == (size_t)(3 * M->P);
    const bool closed = std::fclose(f) == 0;
    return ok && closed ? TPF_OK : fail(TPF_ERR_INVALID_ARG, std::string("write failed: ") + path);
}

extern "C" int tpf_mlp_load(const char *path, tpf_mlp *out) {
    clear_error();
    if (!path || !out) return fail(TPF_ERR_INVALID_ARG, "NULL argument");
    *out = nullptr;
    FILE *f = std::fopen(path, "rb");
    if (!f) return fail(TPF_ERR_INVALID_ARG, std::string("cannot open ") + path);
    MlpFileHeader h{};
    bool ok = std::fread(&h, sizeof h, 1, f) == 1 && h.P > 0 && h.P < ((int64_t)1 << 31);
    const bool v2 = ok && std::memcmp(h.magic, kMagicV2, 8) == 0;
    ok = ok && (v2 || std::memcmp(h.magic, kMagicV1, 8) == 0);
    const int64_t count = (v2 ? 3 : 1) * (ok ? h.P : 0);
    std::vector<float> host(count);
    ok = ok && std::fread(host.data(), 4, count, f) == (size_t)count;
    std::fclose(f);
    if (!ok) return fail(TPF_ERR_INVALID_ARG, std::string("not a warm-start parameter file: ") + path);
    int rc = tpf_mlp_create(h.n, h.hidden, h.layers, host.data(), h.vs_re, h.vs_im, out);
    if (rc != TPF_OK) return rc;
    if ((*out)->P != h.P) {
        tpf_mlp_free(*out);
        *out = nullptr;
        return fail(TPF_ERR_INVALID_ARG, "parameter count mismatch");
    }
    if (v2) {
        if (hipMemcpy((*out)->m, host.data() + h.P, h.P * 4, hipMemcpyHostToDevice) != hipSuccess ||
            hipMemcpy((*out)->v, host.data() + 2 * h.P, h.P * 4, hipMemcpyHostToDevice) != hipSuccess) {
            tpf_mlp_free(*out);
            *out = nullptr;
            return fail(TPF_ERR_DEVICE, "host-to-device copy failed (AdamW moments)");
        }
        (*out)->step = h.step;
    }
    return TPF_OK;
}
