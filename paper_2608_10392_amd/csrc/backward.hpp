// Backward pass of the layer (gradients of sum(dY * Y)).
//
// The discrete decisions (b, I_shr, q, k) are those of the forward and are
// held fixed; gradients flow through alpha (Eq. alpha) to W_shr and x,
// through the selected affinities p_i (the softmax of Eq.
// residual-router-score) to W_1..W_K and x, and through the expert FFNs of
// Eq. block-expert-output. The prototypes get none (they only enter TopK).
//
// bf16 layers run on the matrix cores (the up and down engines of
// ffn_bf16.hpp with backward epilogues, and wgrad.hpp); the kernels here are
// the per-pair and per-token scalars (bwd_weights,
// bwd_dcoef_sum_kernel, bwd_token_kernel, the router kernels).
// fp32 layers run on the matrix cores in fp32 (ffn_f32.hpp); the kernels here
// serve both.
#pragma once
#include <type_traits>

#include "common.hpp"

namespace unifmoe {

struct BwdParams {
    int N, d, K, B, M, H;
    int alpha_adaptive;
    float tau, one_minus_2tau;
    const void* X;            // [N, d] layer format
    const void* dY;           // [N, d] layer format
    const float* Wr;          // [K+1, d]
    const float* alpha;       // routing record
    const int* nres;
    const int* eids;          // [N, K]
    const float* wts;         // [N, K]
    const int* pair_token;    // forward pair tables (pairs grouped by expert)
    const int* pair_expert;
    const uint64_t* pair_mask;
    const int* pair_of;       // [N, K+1]
    const int* seg_off;       // [K+2] first pair of each expert segment
    const int* totals;        // [0]: pairs
    float* dcoef;             // [pairs] dy . E_pair
    float* pw;                // [pairs] pair weight (alpha or p_i)
    float* dxp;               // [pairs, d] dx_pair
    float* dz;                // [N, K+1]: dz0, then dl_1..dl_K
    float* rpart;             // [kRouterChunks, K+1, d] partial router gradients
    float* dX;                // [N, d]
    float* dWr;               // [K+1, d]
};

// Weight of pair (t, e): alpha for the shared expert, else the affinity p_i
// of the residual expert e = q_i.
__device__ __forceinline__ float pair_weight(const BwdParams& p, int t, int e) {
    if (e == 0) return p.alpha[t];
    const int k = p.nres[t];
    for (int i = 0; i < k; ++i)
        if (p.eids[(size_t)t * p.K + i] == e) return p.wts[(size_t)t * p.K + i];
    return 0.f;
}

// Pair weights: alpha for the shared expert, p_i for residual expert q_i
// (workgroup b of n).
__device__ __forceinline__ void bwd_weights(const BwdParams& p, int b, int n) {
    const int P = p.totals[0];
    for (int pr = b * blockDim.x + threadIdx.x; pr < P; pr += n * blockDim.x)
        p.pw[pr] = pair_weight(p, p.pair_token[pr], p.pair_expert[pr]);
}
__global__ __launch_bounds__(256) void bwd_weight_kernel(BwdParams p) { bwd_weights(p, blockIdx.x, gridDim.x); }

// dcoef[pr] = dy_{tok(pr)} . E_pr from the partial sums that the dy V pass
// leaves per (pair, block), npb of them (bf16 layers: the two column halves;
// fp32 layers: two per 64-channel chunk): summed over the blocks of the
// pair's mask in increasing order (a pair with no block gets 0).
__global__ __launch_bounds__(256) void bwd_dcoef_sum_kernel(BwdParams p, const float* __restrict__ dcp, int npb) {
    const int P = p.totals[0];
    for (int pr = blockIdx.x * blockDim.x + threadIdx.x; pr < P; pr += gridDim.x * blockDim.x) {
        uint64_t m = p.pair_mask[pr];
        float s = 0.f;
        while (m) {
            const float* q = dcp + ((size_t)pr * p.B + __builtin_ctzll(m)) * npb;
            for (int i = 0; i < npb; i += 2) s += q[i] + q[i + 1];
            m &= m - 1;
        }
        p.dcoef[pr] = s;
    }
}

// Per token: the router-logit gradients dz (dz0 for W_shr through alpha,
// dl_j for W_j through the softmax) and dX = the sum of the token's dx_pair
// plus sum_j dz_j W_j. A workgroup takes kTokTile tokens: their dz first
// (one thread per (token, slot)), kept in LDS and written out for the
// router's weight gradient; then each thread takes columns n, holds W_j[n]
// for 16 j at a time in registers and adds their terms to all the tile's
// tokens. Fixed summation order: the pairs in slot order, then j = 0..K.
constexpr int kTokTile = 16;
constexpr int kDzRow = 80;   // K+1 <= 65, rounded up to whole groups of 16

__global__ __launch_bounds__(256) void bwd_token_kernel(BwdParams p) {
    __shared__ float dzs[kTokTile][kDzRow];
    __shared__ float sdp_s[kTokTile];
    __shared__ int pofs[kTokTile][kDzRow];   // the tile's pairs by slot (0 past a token's k)
    const int K1 = p.K + 1;
    const int t0 = blockIdx.x * kTokTile;
    const int nt = min(kTokTile, p.N - t0);
    for (int x = threadIdx.x; x < kTokTile * kDzRow; x += blockDim.x) dzs[x / kDzRow][x % kDzRow] = 0.f;
    // sum_m p_m dp_m with dp nonzero for the k selected experts
    if ((int)threadIdx.x < nt) {
        const int t = t0 + threadIdx.x;
        const int k = p.nres[t];
        const int* of = p.pair_of + (size_t)t * K1;
        float sdp = 0.f;
        for (int i = 0; i < k; ++i) sdp = fmaf(p.wts[(size_t)t * p.K + i], p.dcoef[of[1 + i]], sdp);
        sdp_s[threadIdx.x] = sdp;
    }
    __syncthreads();
    // Slot 0: alpha = tau + (1 - 2 tau) sigma(z0), so dz0 = dcoef_shr (1 - 2
    // tau) sigma (1 - sigma), sigma recovered from alpha. Slot i + 1: p_i =
    // s_{q_i}, dl_{q_i} = p_i (dp_{q_i} - sum_m p_m dp_{q_m}). Padded tokens
    // get zeros (slot i then stands for j = i).
    for (int x = threadIdx.x; x < nt * K1; x += blockDim.x) {
        const int tt = x / K1, i = x - tt * K1, t = t0 + tt;
        const int k = p.nres[t];
        float v = 0.f;
        int j = i;
        if (k > 0) {
            const int* of = p.pair_of + (size_t)t * K1;
            if (i == 0) {
                if (p.alpha_adaptive) {
                    const float sg = (p.alpha[t] - p.tau) / p.one_minus_2tau;
                    v = p.dcoef[of[0]] * p.one_minus_2tau * sg * (1.f - sg);
                }
            } else {
                const float pi = p.wts[(size_t)t * p.K + i - 1];
                const float dpi = (i - 1 < k) ? p.dcoef[of[i]] : 0.f;
                v = pi * (dpi - sdp_s[tt]);
                j = p.eids[(size_t)t * p.K + i - 1];
            }
        }
        dzs[tt][j] = v;
        p.dz[(size_t)t * K1 + j] = v;
    }
    __syncthreads();
    // dX, 4 columns per thread: the pair rows slot by slot across the tile's
    // tokens, then the router terms 8 j at a time with W_j[n..n+3] in
    // registers. The tile's pair indices are staged in LDS and a slot's 16
    // row loads are issued unconditionally (slots a token lacks re-read pair
    // 0 and add nothing), so they are all in flight together.
    int kk[kTokTile];
    int kmax = 0;
#pragma unroll
    for (int tt = 0; tt < kTokTile; ++tt) {
        kk[tt] = tt < nt ? p.nres[t0 + tt] : 0;
        kmax = max(kmax, kk[tt]);
    }
    for (int x = threadIdx.x; x < kTokTile * K1; x += blockDim.x) {
        const int tt = x / K1, i = x - tt * K1;
        const int k = tt < nt ? p.nres[t0 + tt] : 0;
        pofs[tt][i] = (k > 0 && i <= k) ? p.pair_of[(size_t)(t0 + tt) * K1 + i] : 0;
    }
    __syncthreads();
    const int nslot = (kmax > 0) ? kmax + 1 : 0;   // kmax = 0: every token of the tile is padded
    for (int n = 4 * (int)threadIdx.x; n < p.d; n += 4 * (int)blockDim.x) {
        f32x4 acc[kTokTile];
#pragma unroll
        for (int tt = 0; tt < kTokTile; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int i = 0; i < nslot; ++i) {
            f32x4 v[kTokTile];
#pragma unroll
            for (int tt = 0; tt < kTokTile; ++tt)
                v[tt] = *reinterpret_cast<const f32x4*>(p.dxp + (size_t)pofs[tt][i] * p.d + n);
#pragma unroll
            for (int tt = 0; tt < kTokTile; ++tt)
                if (i <= kk[tt] && kk[tt] > 0) acc[tt] += v[tt];
        }
        for (int j0 = 0; j0 < K1; j0 += 8) {
            f32x4 w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                w[u] = (j0 + u < K1) ? *reinterpret_cast<const f32x4*>(p.Wr + (size_t)(j0 + u) * p.d + n)
                                     : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tt = 0; tt < kTokTile; ++tt)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float z = dzs[tt][j0 + u];
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[tt][q] = fmaf(z, w[u][q], acc[tt][q]);
                }
        }
#pragma unroll
        for (int tt = 0; tt < kTokTile; ++tt)
            if (tt < nt)
                *reinterpret_cast<f32x4*>(p.dX + (size_t)(t0 + tt) * p.d + n) =
                    kk[tt] > 0 ? acc[tt] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// dW_router[j][n] = sum_t dz[t][j] x_t[n] in two passes: partial sums over
// kRouterChunks slices of the tokens (blockIdx.z), then their sum in slice
// order. One wave per (128 columns, 32 j, slice), on the matrix cores in
// fp32 (v_mfma_f32_32x32x2_f32, two tokens per step, four products side by
// side): lane l brings dz[t + l / 32][j0 + l % 32] as its A value and
// x_{t + l / 32}[n0 + 4 (l % 32) + b] as its B value of product b, so column
// cc of product b stands for n = n0 + 4 cc + b and one load gives a lane its
// four B values. The loads of the next 16 tokens are in flight while the
// current 16 are multiplied.
constexpr int kRouterChunks = 256;
constexpr int kRouterCols = 128;

// Four consecutive values of a layer-format tensor: the raw bytes (8 for
// bf16, 16 for fp32), then as floats.
template <bool BF16>
using raw4_t = typename std::conditional<BF16, uint2, f32x4>::type;

template <bool BF16>
__device__ __forceinline__ raw4_t<BF16> ld_raw4(const void* p, size_t i) {
    if constexpr (BF16) return *reinterpret_cast<const uint2*>(static_cast<const u16*>(p) + i);
    else return *reinterpret_cast<const f32x4*>(static_cast<const float*>(p) + i);
}

template <bool BF16>
__device__ __forceinline__ f32x4 raw4_f32(raw4_t<BF16> r) {
    if constexpr (BF16)
        return f32x4{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u), __uint_as_float(r.y << 16),
                     __uint_as_float(r.y & 0xffff0000u)};
    else return r;
}

template <bool BF16>
__global__ __launch_bounds__(64) void bwd_router_kernel(BwdParams p) {
    constexpr int U = 8;   // steps (two tokens each) per batch of loads
    const int K1 = p.K + 1;
    const int lane = (int)threadIdx.x, lr = lane & 31, lh = lane >> 5;
    const int n0 = (int)blockIdx.x * kRouterCols, j0 = (int)blockIdx.y * 32, c = (int)blockIdx.z;
    const int t0 = (int)((int64_t)c * p.N / kRouterChunks), t1 = (int)((int64_t)(c + 1) * p.N / kRouterChunks);
    const int j = j0 + lr, n = n0 + 4 * lr;
    const bool jok = j < K1, nok = n < p.d;   // d % 4 == 0: a lane's 4 columns are all in or all out
    // Loads are issued for every lane and step (out-of-range ones read a
    // valid element of the slice, row t1 - 1, and are zeroed afterwards), so
    // a batch's loads are all in flight together.
    const int jc = jok ? j : 0, nc = nok ? n : 0;
    f32x16 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = f32x16{};
    float a[2][U];
    raw4_t<BF16> x[2][U];
    auto load = [&](int t, int set) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int tt = min(t + 2 * u + lh, t1 - 1);
            a[set][u] = p.dz[(size_t)tt * K1 + jc];
            x[set][u] = ld_raw4<BF16>(p.X, (size_t)tt * p.d + nc);
        }
    };
    auto multiply = [&](int t, int set) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = t + 2 * u + lh < t1;
            const float av = (ok && jok) ? a[set][u] : 0.f;
            const f32x4 xv = raw4_f32<BF16>(x[set][u]);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, nok ? xv[q] : 0.f, acc[q], 0, 0, 0);
        }
    };
    if (t0 < t1) load(t0, 0);
    for (int t = t0; t < t1; t += 4 * U) {
        if (t + 2 * U < t1) load(t + 2 * U, 1);
        multiply(t, 0);
        if (t + 2 * U >= t1) break;
        if (t + 4 * U < t1) load(t + 4 * U, 0);
        multiply(t + 2 * U, 1);
    }
    // Lane l holds rows (v / 4) 8 + 4 (l / 32) + v % 4 of column l % 32 of
    // each product.
    if (nok)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = j0 + (v >> 2) * 8 + lh * 4 + (v & 3);
            if (r < K1)
                *reinterpret_cast<f32x4*>(p.rpart + ((size_t)c * K1 + r) * p.d + n) =
                    f32x4{acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
        }
}

// The slices' sum: four threads per element take 64 slices each (8 loads in
// flight), and their four sums are added in order (one thread per element took
// 12.7 us whatever the layer).
__global__ __launch_bounds__(256) void bwd_router_sum_kernel(BwdParams p) {
    __shared__ float part[4][64];
    const size_t n = (size_t)(p.K + 1) * p.d;
    const int lane = lane_id(), g = (int)threadIdx.x >> 6;
    const size_t item = (size_t)blockIdx.x * 64 + lane;
    float s = 0.f;
    if (item < n) {
        const float* src = p.rpart + (size_t)g * (kRouterChunks / 4) * n + item;
        for (int c = 0; c < kRouterChunks / 4; c += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(c + u) * n];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    }
    part[g][lane] = s;
    __syncthreads();
    if (g == 0 && item < n) p.dWr[item] = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
}

// Gram diversity loss of the augmented router (Eq. diversity-loss):
// L_div = || W W^T - I ||_F over the K+1 router rows W (W_shr, W_1..W_K),
// and dW += lambda (2 / L_div) (W W^T - I) W (none when L_div = 0). fp64
// throughout (the products of fp32 values are exact), every sum in a fixed
// order, so the result is the same on every call.
struct DivParams {
    int K1, d;
    const float* W;      // [K+1, d]
    double* G;           // [K+1, K+1] workspace
    float* loss;         // [1]
    float* dW;           // [K+1, d], updated
    float lambda;
};

// G[i][j] = W_i . W_j, one wave per pair i <= j (lanes take n = lane + 64 t,
// then a fixed shuffle tree).
__global__ __launch_bounds__(256) void div_gram_kernel(DivParams p) {
    const int w = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    const int npair = p.K1 * (p.K1 + 1) / 2;
    if (w >= npair) return;
    int i = 0, rem = w;
    while (rem >= p.K1 - i) {
        rem -= p.K1 - i;
        ++i;
    }
    const int j = i + rem;
    const float* a = p.W + (size_t)i * p.d;
    const float* b = p.W + (size_t)j * p.d;
    double s = 0.0;
    for (int n = lane_id(); n < p.d; n += kWave) s = fma((double)a[n], (double)b[n], s);
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane_id() == 0) {
        p.G[(size_t)i * p.K1 + j] = s;
        p.G[(size_t)j * p.K1 + i] = s;
    }
}

// L_div from G by one workgroup of 256 (strided partial sums, then a fixed
// tree in LDS): the same value in every workgroup that forms it.
__device__ __forceinline__ double div_loss(const DivParams& p, double* part) {
    const int n = p.K1 * p.K1;
    double s = 0.0;
    for (int x = threadIdx.x; x < n; x += 256) {
        const double v = p.G[x] - ((x / p.K1 == x % p.K1) ? 1.0 : 0.0);
        s = fma(v, v, s);
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
        __syncthreads();
    }
    return sqrt(part[0]);
}

// dW[i][n] += lambda (2 / L) sum_j (G - I)[i][j] W[j][n], one thread per (i, n);
// every workgroup forms L itself (a launch of its own took longer), the first
// writes it.
__global__ __launch_bounds__(256) void div_grad_kernel(DivParams p) {
    __shared__ double part[256];
    const double L = div_loss(p, part);
    if (blockIdx.x == 0 && threadIdx.x == 0) *p.loss = (float)L;
    const size_t item = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (item >= (size_t)p.K1 * p.d) return;
    if (L == 0.0 || p.lambda == 0.0f) return;
    const int i = (int)(item / p.d), n = (int)(item - (size_t)i * p.d);
    double g = 0.0;
    for (int j = 0; j < p.K1; ++j)
        g = fma(p.G[(size_t)i * p.K1 + j] - (i == j ? 1.0 : 0.0), (double)p.W[(size_t)j * p.d + n], g);
    p.dW[item] = (float)((double)p.dW[item] + (double)p.lambda * (2.0 / L) * g);
}

}  // namespace unifmoe
