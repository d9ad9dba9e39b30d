// The transformer block around the layer: LayerNorm of the FFN input
// (pre-LN) and the block's merge (Eq. output plus the b2 shares, the
// residual add and, post-LN, the LayerNorm of the sum).
//
// LayerNorm: LN(v) = (v - mean) / sqrt(var + eps) * gamma + beta, biased
// variance over the d features. Statistics and the normalisation run in
// fp64 (sums of d terms; the result then differs from the exact value by a
// few fp64 ulps, so rounding it to the layer's format almost never lands on
// the other side of a rounding midpoint). Row sums are butterfly
// reductions over the lanes of a row, after which every one of those lanes
// holds the same (commutative) sums.
#pragma once
#include "common.hpp"

namespace unifmoe {

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// fp64 -> bf16, round to nearest even, via round-to-odd fp32: the fp32 value
// truncated toward zero, with its last bit set when inexact; rounding that
// to 8 significant bits equals rounding the fp64 value directly (the fp32
// format has at least two more bits), in the normal range.
__device__ __forceinline__ u16 f64_to_bf16(double v) {
    const float f = (float)v;
    const double d = (double)f;
    uint32_t u = __float_as_uint(f);
    // f rounded away from zero: one step back, then the sticky bit.
    if (d != v) u = (u - (fabs(d) > fabs(v) ? 1u : 0u)) | 1u;
    return f2bf(__uint_as_float(u));
}

struct LayerNormParams {
    int N, d;
    const void* X;      // [N, d] layer format
    void* Xn;           // [N, d] layer format
    const float* gamma;
    const float* beta;
    double eps;
};

// Rows are walked in chunks: 8 bf16 (one 16-byte access) or one fp32
// element; lane l takes chunks l, l + 64, ...
template <bool BF16>
struct Chunk {
    static constexpr int E = BF16 ? 8 : 1;
    float v[E];
    __device__ __forceinline__ void load(const void* row, int ch) {
        if constexpr (BF16) {
            const u32x4 q = ld16(static_cast<const u16*>(row) + ch * 8);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i] = __uint_as_float(q[i] << 16);
                v[2 * i + 1] = __uint_as_float(q[i] & 0xffff0000u);
            }
        } else {
            v[0] = static_cast<const float*>(row)[ch];
        }
    }
};

template <bool BF16>
__device__ __forceinline__ void store_chunk(void* row, int ch, const double (&y)[Chunk<BF16>::E]) {
    if constexpr (BF16) {
        u32x4 q;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = (uint32_t)f64_to_bf16(y[2 * i]) | ((uint32_t)f64_to_bf16(y[2 * i + 1]) << 16);
        st16(static_cast<u16*>(row) + ch * 8, q);
    } else {
        static_cast<float*>(row)[ch] = (float)y[0];
    }
}

// Chunk ch (E values) of a per-feature fp32 parameter.
template <int E>
__device__ __forceinline__ void load_params(const float* p, int ch, float (&v)[E]) {
    if constexpr (E % 4 == 0) {
#pragma unroll
        for (int h = 0; h < E / 4; ++h) {
            const f32x4 q = ld_f32x4(p + (size_t)ch * E + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * h + e] = q[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = p[(size_t)ch * E + e];
    }
}

// Sum over the LPR consecutive lanes that share a row (LPR a power of two
// <= 64); every lane of the group ends with the same sum.
template <int LPR>
__device__ __forceinline__ double group_sum_f64(double v) {
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Pre-LN: Xn = LN(X), LPR lanes per row (several rows per wave, so each
// wave keeps more loads in flight). Rows of at most LPR MAXC chunks stay in
// registers (one read); longer rows are re-read from cache by each of the
// three passes (mean, variance, output).
template <bool BF16, int MAXC, int LPR>
__global__ __launch_bounds__(256) void layernorm_rows_kernel(LayerNormParams p) {
    using C = Chunk<BF16>;
    const int t = (int)((blockIdx.x * blockDim.x + threadIdx.x) / LPR);
    if (t >= p.N) return;
    const int sub = threadIdx.x % LPR, nch = p.d / C::E;
    const size_t esz = BF16 ? 2 : 4;
    const char* xr = static_cast<const char*>(p.X) + (size_t)t * p.d * esz;
    char* yr = static_cast<char*>(p.Xn) + (size_t)t * p.d * esz;
    const bool cached = nch <= LPR * MAXC;
    C cache[MAXC];
    if (cached) {
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if (sub + LPR * i < nch) cache[i].load(xr, sub + LPR * i);
    }
    // f(chunk, index) for this lane's chunks of the row, from registers or
    // from memory.
    auto each = [&](auto f) {
        if (cached) {
#pragma unroll
            for (int i = 0; i < MAXC; ++i)
                if (sub + LPR * i < nch) f(cache[i], sub + LPR * i);
        } else {
            for (int ch = sub; ch < nch; ch += LPR) {
                C c;
                c.load(xr, ch);
                f(c, ch);
            }
        }
    };
    double s = 0.0;
    each([&](const C& c, int) {
#pragma unroll
        for (int e = 0; e < C::E; ++e) s += (double)c.v[e];
    });
    const double mu = group_sum_f64<LPR>(s) / p.d;
    double q = 0.0;
    each([&](const C& c, int) {
#pragma unroll
        for (int e = 0; e < C::E; ++e) {
            const double u = (double)c.v[e] - mu;
            q = fma(u, u, q);
        }
    });
    const double rstd = 1.0 / sqrt(group_sum_f64<LPR>(q) / p.d + p.eps);
    each([&](const C& c, int ch) {
        float g[C::E], be[C::E];
        load_params<C::E>(p.gamma, ch, g);
        load_params<C::E>(p.beta, ch, be);
        double y[C::E];
#pragma unroll
        for (int e = 0; e < C::E; ++e) y[e] = ((double)c.v[e] - mu) * rstd * (double)g[e] + (double)be[e];
        store_chunk<BF16>(yr, ch, y);
    });
}

struct BlockCombineParams {
    int N, d, K, B;
    int nsplit;             // row buffers per pair (bf16: the down-projection's parts), summed in order
    size_t split_stride;    // floats between them
    const void* part;       // per-pair expert rows (fp32)
    const int* pair_of;     // [N, K+1] pair of (token, i-th pathway)
    const float* alpha;
    const int* nsh;         // b
    const int* nres;        // k
    const int* eids;        // [N, K] q_1..q_K
    const float* wts;       // [N, K] p_1..p_K
    const float* b_down;    // [K+1, d] or null
    const void* X;          // block input (residual), null: no residual add
    int post;               // nonzero: LayerNorm of the sum
    const float* gamma;
    const float* beta;
    double eps;
    void* Y;
    const int* totals;      // totals[5] != 0: the routing overflowed the pair capacity (Y = 0)
};

constexpr int kBlockCombineBatch = 4;

// E consecutive floats at p (16-byte aligned where E is a multiple of 4),
// read once: non-temporal.
template <int E>
__device__ __forceinline__ void load_row_once(const float* p, float (&v)[E]) {
    if constexpr (E % 4 == 0) {
#pragma unroll
        for (int h = 0; h < E / 4; ++h) {
            const f32x4 q = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p) + h);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * h + e] = q[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = p[e];
    }
}

// z over one chunk of token t's row: alpha E_shr^S + sum_{i <= k} p_i
// E_{q_i}^R (the expert rows in the layer's fixed order, fp32), then the b2
// shares alpha (b/B) b2_shr + sum_i p_i ((B-b)/B) b2_{q_i}, then x. The
// indices and weights of a batch of pathways, then its rows, are loaded
// before any is used, so the latencies overlap (one at a time they were most
// of the post-LN merge's time: 54.9 -> 34.6 us on the padded BERT-large
// batch, with one workgroup per token).
template <bool BF16, int E>
__device__ __forceinline__ void block_chunk_sum(const BlockCombineParams& c, int t, int ch, float (&z)[E]) {
    constexpr int U = kBlockCombineBatch;
    float x[E];
    if (c.X != nullptr) {
        const size_t at = (size_t)t * c.d + (size_t)ch * E;
        if constexpr (BF16) {
#pragma unroll
            for (int h = 0; h < E / 4; ++h) {
                const uint2 q = *reinterpret_cast<const uint2*>(static_cast<const u16*>(c.X) + at + 4 * h);
                x[4 * h] = __uint_as_float(q.x << 16);
                x[4 * h + 1] = __uint_as_float(q.x & 0xffff0000u);
                x[4 * h + 2] = __uint_as_float(q.y << 16);
                x[4 * h + 3] = __uint_as_float(q.y & 0xffff0000u);
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = static_cast<const float*>(c.X)[at + e];
        }
    }
    const int k = c.nres[t];
    const float a = c.alpha[t];
    const int* of = c.pair_of + (size_t)t * (c.K + 1);
    const float* wt = c.wts + (size_t)t * c.K;
    const float* part = static_cast<const float*>(c.part);
    // Pathway i's weight: alpha, p_1, p_2, ..
    auto weight = [&](int i) { return i == 0 ? a : wt[i - 1]; };
#pragma unroll
    for (int e = 0; e < E; ++e) z[e] = 0.f;
    for (int i0 = 0; i0 <= k && k > 0; i0 += U) {
        int pr[U];
        float w[U], r[U][E];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pr[u] = (i0 + u <= k) ? of[i0 + u] : 0;
            w[u] = (i0 + u <= k) ? weight(i0 + u) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u <= k) load_row_once<E>(part + (size_t)pr[u] * c.d + ch * E, r[u]);
        for (int sp = 1; BF16 && sp < c.nsplit; ++sp) {
            float r2[U][E];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u <= k) load_row_once<E>(part + sp * c.split_stride + (size_t)pr[u] * c.d + ch * E, r2[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u <= k)
#pragma unroll
                    for (int e = 0; e < E; ++e) r[u][e] += r2[u][e];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u <= k)
#pragma unroll
                for (int e = 0; e < E; ++e) z[e] = fmaf(w[u], r[u][e], z[e]);
    }
    if (c.b_down != nullptr && k > 0) {
        const int b = c.nsh[t];
        const float share_s = (float)b / (float)c.B, share_r = (float)(c.B - b) / (float)c.B;
        const int* q = c.eids + (size_t)t * c.K;
        for (int i0 = 0; i0 <= k; i0 += U) {
            int ex[U];
            float f[U], r[U][E];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u;
                ex[u] = (i > 0 && i <= k) ? q[i - 1] : 0;
                f[u] = (i <= k) ? weight(i) * (i == 0 ? share_s : share_r) : 0.f;
            }
            // b2 rows: E consecutive floats (16-byte aligned for bf16 layers).
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u <= k) load_params<E>(c.b_down + (size_t)ex[u] * c.d, ch, r[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u <= k)
#pragma unroll
                    for (int e = 0; e < E; ++e) z[e] = fmaf(f[u], r[u][e], z[e]);
        }
    }
    if (c.X != nullptr) {
#pragma unroll
        for (int e = 0; e < E; ++e) z[e] += x[e];
    }
}

// No post-LN: one thread per 4 outputs (bf16) or one (fp32), as the layer's
// merge.
template <bool BF16>
__global__ __launch_bounds__(256) void combine_block_flat_kernel(BlockCombineParams c) {
    constexpr int E = BF16 ? 4 : 1;
    const int nch = c.d / E;
    const size_t item = flat_block() * blockDim.x + threadIdx.x;
    if (item >= (size_t)c.N * nch) return;
    const int t = (int)(item / nch), ch = (int)(item - (size_t)t * nch);
    float z[E];
    if (ld_uniform(c.totals + 5) != 0) {
        // past the pair capacity no expert row exists: Y = 0
#pragma unroll
        for (int e = 0; e < E; ++e) z[e] = 0.f;
    } else {
        block_chunk_sum<BF16, E>(c, t, ch, z);
    }
    // One rounding from fp32 (what f64_to_bf16 gives for an fp32 value).
    if constexpr (BF16) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        u32x2 o;
#pragma unroll
        for (int i = 0; i < 2; ++i) o[i] = (uint32_t)f2bf(z[2 * i]) | ((uint32_t)f2bf(z[2 * i + 1]) << 16);
        __builtin_nontemporal_store(o, reinterpret_cast<u32x2*>(static_cast<u16*>(c.Y) + (size_t)t * c.d + ch * E));
    } else {
        static_cast<float*>(c.Y)[(size_t)t * c.d + ch] = z[0];
    }
}

// Sum over the workgroup (whole waves) in wave order; lds holds one word per
// wave (unused by a workgroup of one wave).
__device__ __forceinline__ double block_sum_f64(double v, double* lds) {
    v = wave_sum_f64(v);
    if (blockDim.x == 64) return v;
    __syncthreads();
    if (lane_id() == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += lds[w];
    return s;
}

// Post-LN: one workgroup per token, about one chunk per thread or one wave in
// all (kPostWaveTokens); z stays in LDS (d floats; each lane reads back only
// what it wrote) for the LayerNorm.
template <bool BF16>
__global__ __launch_bounds__(256) void combine_block_post_kernel(BlockCombineParams c) {
    constexpr int E = Chunk<BF16>::E;
    extern __shared__ __attribute__((aligned(16))) float zrow[];
    double* sums = reinterpret_cast<double*>(zrow + ((c.d + 1) & ~1));   // past one wave
    if (flat_block() >= (size_t)c.N) return;
    const int t = (int)flat_block(), T = blockDim.x;
    const int nch = c.d / E;
    char* yr = static_cast<char*>(c.Y) + (size_t)t * c.d * (BF16 ? 2 : 4);
    if (ld_uniform(c.totals + 5) != 0) {
        // past the pair capacity no expert row exists: Y = 0
        double y0[E];
#pragma unroll
        for (int e = 0; e < E; ++e) y0[e] = 0.0;
        for (int ch = threadIdx.x; ch < nch; ch += T) store_chunk<BF16>(yr, ch, y0);
        return;
    }
    double s = 0.0;
    for (int ch = threadIdx.x; ch < nch; ch += T) {
        float z[E];
        block_chunk_sum<BF16, E>(c, t, ch, z);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            zrow[ch * E + e] = z[e];
            s += (double)z[e];
        }
    }
    const double mu = block_sum_f64(s, sums) / c.d;
    double sq = 0.0;
    for (int ch = threadIdx.x; ch < nch; ch += T) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double u = (double)zrow[ch * E + e] - mu;
            sq = fma(u, u, sq);
        }
    }
    const double rstd = 1.0 / sqrt(block_sum_f64(sq, sums) / c.d + c.eps);
    for (int ch = threadIdx.x; ch < nch; ch += T) {
        float g[E], be[E];
        load_params<E>(c.gamma, ch, g);
        load_params<E>(c.beta, ch, be);
        double y[E];
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = ((double)zrow[ch * E + e] - mu) * rstd * (double)g[e] + (double)be[e];
        store_chunk<BF16>(yr, ch, y);
    }
}

}  // namespace unifmoe
