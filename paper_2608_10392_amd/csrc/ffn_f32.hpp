// fp32 layers (Eq. block-expert-output, fp32 end to end), forward and
// backward, on the matrix cores in fp32 (v_mfma_f32_32x32x2_f32):
//   f32_up_kernel     per up tile (64 rows of one (expert, block) slab's row
//                     list x 64 of the block's channels):
//                       kF32Gelu  act = GELU(x K^T + b1)
//                       kF32Pre   act = GELU(a), da = GELU'(a), a = x K^T
//                       kF32Da    g = dy V: the partial sums of act . g (the
//                                 pair's d loss / d weight), da = w g GELU'(a)
//   f32_down_kernel   per down row tile (64 pairs of one expert sorted by
//                     block mask) x 64 columns, over the union of the tile's
//                     blocks: part = act V, or dx_pair = da K
//   f32_wgrad_kernel  per slab: dW_up = da^T X, dW_down = (w dY)^T act over
//                     the slab's rows in token order
// Every product accumulates in fp32 in a fixed order.
//
// One workgroup of 4 waves (2 x 2, a 32 x 32 product each) per 64 x 64 output
// tile; 32 k per stage through two LDS slots, the next stage's values loaded
// into registers while one is multiplied. A 32 x 32 x 2 product takes 64
// cycles for two 4-byte operands per lane, so LDS and registers are idle most
// of the time and the small tile costs nothing there; it gives small layers
// enough workgroups and the row tiles small block unions. An operand is
// staged as it lies in memory: rows of k (read 16 bytes per lane, four
// products' worth) or rows of the output's index (4 bytes per lane).
// Rows may start at any 4-byte address and end anywhere.
//
// DeiT-S layer (d = 384, H = 1536, K = 6), 1,576 tokens: up and
// down 54 + 77 us (38 to 55 TFLOP/s of a 152 TFLOP/s peak; 12.1 ms as one
// workgroup per pair with a serial dot product per thread), the backward's
// products and weight gradients 55 + 66 + 86 + 64 + 70 us (2.7 ms on the
// vector units with 128 x 128 tiles over whole expert segments). What is left
// is a last wave of workgroups (440 to 1,000 tiles over 1,024 places) and the
// barrier and load latency of 12 to 50 stages per tile.
//
// A forward's activations take a bounded part of the workspace: layers that
// need more run in passes over ranges of experts, and where one expert's do not
// fit, of its channels (F32Pass), with the same bits.
//
// pair_ffn_f32_kernel is the forward for layers that have no room for
// activations and tables at all (the workspace-free forward): it holds one
// pair's activations in LDS and needs no memory.
#pragma once
#include "common.hpp"

namespace unifmoe {

constexpr int kF32T = 64;                    // output tile
constexpr int kF32K = 32;                    // k per stage
constexpr int kF32RowStride = kF32K + 4;     // LDS row of k (16-byte reads of 32 rows: no bank conflicts)
constexpr int kF32IdxStride = kF32T + 8;     // LDS row of the index (rows 4 apart on the other 32 banks)
constexpr int kF32Operand = kF32T * kF32RowStride;
static_assert(kF32Operand == kF32K * kF32IdxStride, "both stagings take the same space");
constexpr int kF32LdsFloats = 4 * kF32Operand;   // two operands, two slots

constexpr int kF32Gelu = 0, kF32Pre = 1, kF32Da = 2;

// Partial sums per pair of kF32Da: two column halves per 64-channel chunk.
__host__ __device__ __forceinline__ int f32_chunks(int M) { return ceil_div(M, kF32T); }
__host__ __device__ __forceinline__ int f32_partials(int B, int M) { return 2 * B * f32_chunks(M); }

// What a pass of a forward covers: experts [e0, e0 + ne) and channels [h0, h0 +
// hw) (cut at M) of blocks [c0, c0 + nc). The activations of the experts' pairs
// take `stride` floats each, from the first of them on, channel h of block c at
// (c - c0) hw + h - h0. One pass over everything: channel h of block c of a pair
// at c M + h. Parts of a block are multiples of 64 channels, so that the passes
// of an expert take the stages that one pass would take, in its order.
struct F32Pass {
    int e0, ne, c0, nc, h0, hw, stride;
    bool first;   // of its experts: the rows' sums start at zero
};

struct F32Params {
    int d, M, B, H;
    const float* X;
    const float* dY;
    const float* Wup;        // [K+1][H][d]
    const float* Wdown;      // [K+1][d][H]
    const float* b_up;       // [K+1][H] biases added before the GELU, or null
    F32Pass ps;              // what act holds (backward: everything)
    float* act;              // [pairs of the pass][ps.stride], active blocks only
    float* da;               // [pairs][H], active blocks only (backward)
    float* dcp;              // [pairs][f32_partials] (backward)
    const float* pw;         // pair weights (backward)
    float* part;             // [pairs][d]: expert rows, or dx per pair
    const int* slab_rows;    // up tiles, as for bf16 layers
    const int* slab_tok;
    const int* tile_info;
    const int* tile_rows;
    const int* totals;
    const int4* rt_info;     // down row tiles, as for bf16 layers
    const uint64_t* rt_masks;
    const uint64_t* pair_mask;
    const int* seg_off;      // [K+2] first pair of each expert
    const int* down_tile_off;   // [K+2] first down row tile of each expert
    const int* slab_off;     // first row of each slab in the lists, a multiple of a tile's rows
    const int* slab_count;
    float* dW;
};

// Elements [i, i + 4) of a row that ends at n, zero past it.
__device__ __forceinline__ f32x4 f32_load4(const float* row, int i, int n) {
    if (i + 4 <= n) return ld_f32x4(row + i);
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = (i + q < n) ? row[i + q] : 0.f;
    return v;
}

__device__ __forceinline__ bool f32_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }

// Which 4 values of a stage this thread loads as its piece u (0 or 1): for an
// operand of k rows, row f32_row(u) and k f32_k(); for index rows, k f32_kr(u)
// and index f32_idx().
__device__ __forceinline__ int f32_row(int u) { return ((int)threadIdx.x >> 3) + 32 * u; }
__device__ __forceinline__ int f32_k() { return ((int)threadIdx.x & 7) * 4; }
__device__ __forceinline__ int f32_kr(int u) { return ((int)threadIdx.x >> 4) + 16 * u; }
__device__ __forceinline__ int f32_idx() { return ((int)threadIdx.x & 15) * 4; }

// Sum over nst stages of A(row, k) B(col, k) for this wave's 32 x 32 part of
// the tile. fa(s, u), fb(s, u) load this thread's piece u of stage s; AROWS /
// BROWS: the operand is staged as rows of k (else rows of its index). Lane l
// gets column l % 32 and rows 8 j + 4 (l / 32) + i in element 4 j + i. The
// caller has passed a barrier since the last use of lds. The sum goes on from
// acc.
template <bool AROWS, bool BROWS, class FA, class FB>
__device__ __forceinline__ f32x16 f32_tile(float* lds, int nst, FA fa, FB fb, f32x16 acc = f32x16{}) {
    const int lane = lane_id(), wave = (int)threadIdx.x >> 6, lr = lane & 31, lh = lane >> 5;
    const int ra = (wave >> 1) * 32 + lr, rb = (wave & 1) * 32 + lr;
    if (nst <= 0) return acc;
    f32x4 va[2], vb[2];
    auto load = [&](int s) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            va[u] = fa(s, u);
            vb[u] = fb(s, u);
        }
    };
    auto store = [&](int s) {
        float* a = lds + (s & 1) * 2 * kF32Operand;
        float* b = a + kF32Operand;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            *reinterpret_cast<f32x4*>(a + (AROWS ? f32_row(u) * kF32RowStride + f32_k() : f32_kr(u) * kF32IdxStride + f32_idx())) = va[u];
            *reinterpret_cast<f32x4*>(b + (BROWS ? f32_row(u) * kF32RowStride + f32_k() : f32_kr(u) * kF32IdxStride + f32_idx())) = vb[u];
        }
    };
    // Four products' worth of one operand: k = k0 + 4 lh + 0..3.
    auto take = [&](const float* o, bool rows, int r, int k0) {
        if (rows) return *reinterpret_cast<const f32x4*>(o + r * kF32RowStride + k0 + 4 * lh);
        f32x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = o[(k0 + 4 * lh + q) * kF32IdxStride + r];
        return v;
    };
    load(0);
    store(0);
    for (int s = 0; s < nst; ++s) {
        __syncthreads();
        if (s + 1 < nst) load(s + 1);
        const float* a = lds + (s & 1) * 2 * kF32Operand;
        const float* b = a + kF32Operand;
#pragma unroll
        for (int k0 = 0; k0 < kF32K; k0 += 8) {
            const f32x4 x = take(a, AROWS, ra, k0), w = take(b, BROWS, rb, k0);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[q], w[q], acc, 0, 0, 0);
        }
        if (s + 1 < nst) store(s + 1);
    }
    return acc;
}

// Row of the tile held in element v of f32_tile's result, and its column.
__device__ __forceinline__ int f32_out_row(int v) {
    return ((int)threadIdx.x >> 7) * 32 + 8 * (v >> 2) + 4 * (lane_id() >> 5) + (v & 3);
}
__device__ __forceinline__ int f32_out_col() { return (((int)threadIdx.x >> 6) & 1) * 32 + (lane_id() & 31); }

template <int MODE>
__global__ __launch_bounds__(256) void f32_up_kernel(F32Params p) {
    __shared__ __attribute__((aligned(16))) float lds[kF32LdsFloats];
    __shared__ int tok[kF32T], pair[kF32T];
    if (p.totals[1] == 0) return;   // no rows, or past the pair capacity: no tables
    // Tiles are listed expert by expert, as many of each as its slabs fill.
    const int t0 = p.slab_off[p.ps.e0 * p.B] / kF32T, t1 = min(p.totals[1], p.slab_off[(p.ps.e0 + p.ps.ne) * p.B] / kF32T);
    const int hend = min(p.M, p.ps.h0 + p.ps.hw), pair0 = p.seg_off[p.ps.e0];
    const int chunks = f32_chunks(hend - p.ps.h0), n = (t1 - t0) * chunks;
    for (int t = blockIdx.x; t < n; t += gridDim.x) {
        const int tile = t0 + t / chunks, chunk = t % chunks, h0 = p.ps.h0 + chunk * kF32T;
        const int info = p.tile_info[tile], sl = info & 0xffff, nrows = info >> 16;
        const int e = sl / p.B, c = sl - e * p.B, hw = hend - h0;   // channels left
        if (c < p.ps.c0 || c >= p.ps.c0 + p.ps.nc) continue;
        const int first = p.tile_rows[tile];
        __syncthreads();   // the last tile's products and rows are done with
        if (threadIdx.x < kF32T) {
            const bool in = (int)threadIdx.x < nrows;
            tok[threadIdx.x] = in ? p.slab_tok[first + threadIdx.x] : -1;
            pair[threadIdx.x] = in ? p.slab_rows[first + threadIdx.x] : pair0;
        }
        __syncthreads();
        const float* xs = MODE == kF32Da ? p.dY : p.X;
        auto fa = [&](int s, int u) {
            const int r = tok[f32_row(u)];
            return r >= 0 ? f32_load4(xs + (size_t)r * p.d, s * kF32K + f32_k(), p.d) : f32x4{0.f, 0.f, 0.f, 0.f};
        };
        f32x16 acc;
        if constexpr (MODE == kF32Da) {
            const float* w = p.Wdown + (size_t)e * p.d * p.H + (size_t)c * p.M + h0;
            acc = f32_tile<true, false>(lds, ceil_div(p.d, kF32K), fa, [&](int s, int u) {
                const int k = s * kF32K + f32_kr(u);
                return k < p.d ? f32_load4(w + (size_t)k * p.H, f32_idx(), hw) : f32x4{0.f, 0.f, 0.f, 0.f};
            });
        } else {
            const float* w = p.Wup + ((size_t)e * p.H + (size_t)c * p.M + h0) * p.d;
            acc = f32_tile<true, true>(lds, ceil_div(p.d, kF32K), fa, [&](int s, int u) {
                const int r = f32_row(u);
                return r < hw ? f32_load4(w + (size_t)r * p.d, s * kF32K + f32_k(), p.d) : f32x4{0.f, 0.f, 0.f, 0.f};
            });
        }
        const int col = f32_out_col();
        const bool cok = col < hw;
        const size_t ch = (size_t)c * p.M + h0 + col;
        const float b1 = (MODE == kF32Gelu && p.b_up != nullptr && cok) ? p.b_up[(size_t)e * p.H + ch] : 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = f32_out_row(v);
            const bool ok = cok && r < nrows;
            const size_t off = (size_t)(pair[r] - pair0) * p.ps.stride + (size_t)(c - p.ps.c0) * p.ps.hw + (h0 - p.ps.h0) + col;
            if constexpr (MODE == kF32Gelu) {
                if (ok) p.act[off] = gelu_erf(acc[v] + b1);
            } else if constexpr (MODE == kF32Pre) {
                if (ok) {
                    p.act[off] = gelu_erf(acc[v]);
                    p.da[off] = gelu_grad_erf(acc[v]);
                }
            } else {
                float dc = 0.f;
                if (ok) {
                    dc = p.act[off] * acc[v];
                    p.da[off] = p.pw[pair[r]] * acc[v] * p.da[off];
                }
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) dc += __shfl_xor(dc, o);
                if ((lane_id() & 31) == 0 && r < nrows)
                    p.dcp[(size_t)pair[r] * f32_partials(p.B, p.M) + 2 * (c * chunks + chunk) + (col >> 5)] = dc;
            }
        }
    }
}

// DX: dx_pair = da K, else the expert rows act V. FIRST: the first (or only)
// pass of its experts; later ones go on from the rows' sums.
template <bool DX, bool FIRST>
__global__ __launch_bounds__(256) void f32_down_kernel(F32Params p) {
    __shared__ __attribute__((aligned(16))) float lds[kF32LdsFloats];
    __shared__ uint64_t rmask[kF32T];
    __shared__ int blocks[64];
    const int rt0 = p.down_tile_off[p.ps.e0], rt1 = min(p.totals[4], p.down_tile_off[p.ps.e0 + p.ps.ne]);
    const int ncol = ceil_div(p.d, kF32T), n = (rt1 - rt0) * ncol, pair0 = p.seg_off[p.ps.e0];
    const int hw = min(p.M - p.ps.h0, p.ps.hw);   // channels per block
    const int spb = ceil_div(hw, kF32K);          // stages per block
    const uint64_t in_pass = (p.ps.nc == 64 ? ~0ull : (1ull << p.ps.nc) - 1ull) << p.ps.c0;
    const float* src = DX ? p.da : p.act;
    for (int t = blockIdx.x; t < n; t += gridDim.x) {
        const int rt = rt0 + t / ncol, n0 = (t % ncol) * kF32T;
        const int4 info = p.rt_info[rt];
        const int p0 = info.x, nrows = info.y, e = info.z;
        const uint64_t all = p.rt_masks[(size_t)rt * (kF32T / 32 + 1) + kF32T / 32] & in_pass;
        if (!FIRST && all == 0) continue;
        __syncthreads();   // the last tile's products and rows are done with
        if (threadIdx.x < kF32T) {
            rmask[threadIdx.x] = (int)threadIdx.x < nrows ? p.pair_mask[p0 + threadIdx.x] & in_pass : 0ull;
            if ((all >> threadIdx.x) & 1ull) blocks[__popcll(all & lanes_below())] = threadIdx.x;
        }
        __syncthreads();
        auto fa = [&](int s, int u) {
            const int q = s / spb, c = blocks[q], k = (s - q * spb) * kF32K + f32_k(), r = f32_row(u);
            return ((rmask[r] >> c) & 1ull)
                       ? f32_load4(src + (size_t)(p0 - pair0 + r) * p.ps.stride + (size_t)(c - p.ps.c0) * p.ps.hw, k, hw)
                       : f32x4{0.f, 0.f, 0.f, 0.f};
        };
        const int nst = __popcll(all) * spb, col = n0 + f32_out_col();
        f32x16 acc = f32x16{};
        if constexpr (!FIRST) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = f32_out_row(v);
                if (r < nrows && col < p.d) acc[v] = p.part[(size_t)(p0 + r) * p.d + col];
            }
        }
        if constexpr (DX) {
            const float* w = p.Wup + ((size_t)e * p.H + p.ps.h0) * p.d + n0;
            acc = f32_tile<true, false>(lds, nst, fa, [&](int s, int u) {
                const int q = s / spb, k = (s - q * spb) * kF32K + f32_kr(u);
                return k < hw ? f32_load4(w + ((size_t)blocks[q] * p.M + k) * p.d, f32_idx(), p.d - n0)
                              : f32x4{0.f, 0.f, 0.f, 0.f};
            }, acc);
        } else {
            const float* w = p.Wdown + ((size_t)e * p.d + n0) * p.H + p.ps.h0;
            acc = f32_tile<true, true>(lds, nst, fa, [&](int s, int u) {
                const int q = s / spb, k = (s - q * spb) * kF32K + f32_k(), r = f32_row(u);
                return n0 + r < p.d ? f32_load4(w + (size_t)r * p.H + (size_t)blocks[q] * p.M, k, hw)
                                    : f32x4{0.f, 0.f, 0.f, 0.f};
            }, acc);
        }
        uint32_t again = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = f32_out_row(v);
            if (r < nrows && col < p.d) {
                if (!f32_finite(acc[v]) && rmask[r] != all) again |= 1u << v;
                else p.part[(size_t)(p0 + r) * p.d + col] = acc[v];
            }
        }
        // A row that lacks one of the tile's blocks has zeros there, and zero
        // times a weight that is not finite is a NaN. Such a block must not
        // reach the rows that do not run it: their sums are formed again from
        // their own blocks alone.
        while (again) {
            const int r = f32_out_row(__builtin_ctz(again));
            again &= again - 1;
            const float* a = src + (size_t)(p0 - pair0 + r) * p.ps.stride;
            float sum = FIRST ? 0.f : p.part[(size_t)(p0 + r) * p.d + col];
            for (uint64_t m = rmask[r]; m; m &= m - 1) {
                const int c = __builtin_ctzll(m);
                for (int h = 0; h < hw; ++h) {
                    const size_t ch = (size_t)c * p.M + p.ps.h0 + h;
                    sum = fmaf(a[(size_t)(c - p.ps.c0) * p.ps.hw + h],
                               DX ? p.Wup[((size_t)e * p.H + ch) * p.d + col] : p.Wdown[((size_t)e * p.d + col) * p.H + ch],
                               sum);
                }
            }
            p.part[(size_t)(p0 + r) * p.d + col] = sum;
        }
    }
}

// One 64 x 64 tile of a slab's weight gradient per workgroup: rows h and
// columns n of dW_up (UP), else rows n and columns h of dW_down.
template <bool UP>
__global__ __launch_bounds__(256) void f32_wgrad_kernel(F32Params p) {
    __shared__ __attribute__((aligned(16))) float lds[kF32LdsFloats];
    const int th = f32_chunks(p.M), tn = ceil_div(p.d, kF32T);
    const int sl = blockIdx.x / (th * tn), rem = blockIdx.x - sl * (th * tn);
    const int h0 = (rem / tn) * kF32T, n0 = (rem - (rem / tn) * tn) * kF32T;
    const int e = sl / p.B, c = sl - e * p.B, cnt = p.slab_count[sl];
    const int* rows = p.slab_rows + p.slab_off[sl];
    const int* toks = p.slab_tok + p.slab_off[sl];
    const size_t ch = (size_t)c * p.M + h0;
    const int hw = p.M - h0, nw = p.d - n0;
    auto channels = [&](const float* src, int s, int u) {   // 4 channels of a row's pair
        const int k = s * kF32K + f32_kr(u);
        return k < cnt ? f32_load4(src + (size_t)rows[k] * p.H + ch, f32_idx(), hw) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    const int nst = ceil_div(cnt, kF32K);
    f32x16 acc;
    if constexpr (UP) {
        acc = f32_tile<false, false>(
            lds, nst, [&](int s, int u) { return channels(p.da, s, u); },
            [&](int s, int u) {
                const int k = s * kF32K + f32_kr(u);
                return k < cnt ? f32_load4(p.X + (size_t)toks[k] * p.d + n0, f32_idx(), nw) : f32x4{0.f, 0.f, 0.f, 0.f};
            });
    } else {
        acc = f32_tile<false, false>(
            lds, nst,
            [&](int s, int u) {
                const int k = s * kF32K + f32_kr(u);
                if (k >= cnt) return f32x4{0.f, 0.f, 0.f, 0.f};
                const float w = p.pw[rows[k]];
                f32x4 v = f32_load4(p.dY + (size_t)toks[k] * p.d + n0, f32_idx(), nw);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] *= w;
                return v;
            },
            [&](int s, int u) { return channels(p.act, s, u); });
    }
    const int col = f32_out_col();
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = f32_out_row(v);
        if (r >= (UP ? hw : nw) || col >= (UP ? nw : hw)) continue;
        if constexpr (UP) p.dW[((size_t)e * p.H + ch + r) * p.d + n0 + col] = acc[v];
        else p.dW[((size_t)e * p.d + n0 + r) * p.H + ch + col] = acc[v];
    }
}

struct PairF32Params {
    int d, M, B, H;
    const float* X;
    const float* Wup;    // [K+1][H][d]
    const float* Wdown;  // [K+1][d][H]
    float* part;         // [pairs][d]
    const int* pair_token;
    const int* pair_expert;
    const uint64_t* pair_mask;
    const int* totals;   // [0] pairs, [5] nonzero: more pairs than the buffers hold (nothing to run)
    const float* b_up;   // [K+1][H] biases added before the GELU, or null
};

__global__ __launch_bounds__(256) void pair_ffn_f32_kernel(PairF32Params p) {
    extern __shared__ float g_act[];
    const int P = p.totals[5] ? 0 : p.totals[0];
    for (int pr = blockIdx.x; pr < P; pr += gridDim.x) {
        const int e = p.pair_expert[pr], t = p.pair_token[pr];
        const uint64_t m = p.pair_mask[pr];
        const float* x = p.X + (size_t)t * p.d;
        const float* Wu = p.Wup + (size_t)e * p.H * p.d;
        __syncthreads();
        for (int h = threadIdx.x; h < p.H; h += blockDim.x) {
            float a = 0.f;
            if ((m >> (h / p.M)) & 1ull) {
                const float* w = Wu + (size_t)h * p.d;
                for (int i = 0; i < p.d; ++i) a = fmaf(x[i], w[i], a);
                if (p.b_up != nullptr) a += p.b_up[(size_t)e * p.H + h];
                a = gelu_erf(a);
            }
            g_act[h] = a;
        }
        __syncthreads();
        const float* Wd = p.Wdown + (size_t)e * p.d * p.H;
        for (int j = threadIdx.x; j < p.d; j += blockDim.x) {
            const float* w = Wd + (size_t)j * p.H;
            float s = 0.f;
            for (int c = 0; c < p.B; ++c) {
                if (!((m >> c) & 1ull)) continue;
                for (int h = c * p.M; h < (c + 1) * p.M; ++h) s = fmaf(g_act[h], w[h], s);
            }
            p.part[(size_t)pr * p.d + j] = s;
        }
    }
}

}  // namespace unifmoe
