// Routing (Sec. III-B and III-C): router logits, shared demand, shared block
// count and prototype selection, residual softmax, sort, cumulative-mass
// expert count, and the per-tile counts that the permutation needs.
//
// Logits, 1 + K + B per token (x W_shr, x W_1..x W_K, x mu_1..x mu_B):
//   * bf16 tokens: x W_1.., x mu_1.. on the matrix cores. The fp32 router
//     and prototype weights are pre-split into three bf16 parts (hi + mid +
//     lo carries all 24 significand bits), so every bf16 x bf16 product is
//     exact and only the fp32 accumulation order differs from a sequential
//     dot product. x W_shr is an fp32 dot product on the vector units.
//   * fp32 tokens: the matrix cores in fp32 (v_mfma_f32_16x16x4_f32).
// Decisions: one lane per token (decide_tile), the record and the counts by
// the waves that share the tile of 64 tokens.
// Every step is the paper's order in fp32 with explicitly rounded operations;
// the rankings (ties toward the lower index) are sorting networks in the
// lane's registers. Per tile, the rows per (expert, block) slab and the pairs
// per expert are counted for the permutation.
//
// Three launches share the work by size (launch_route):
//   route_logits_kernel + route_decide_kernel   routers of at most 32 columns,
//                   d <= 1024: the router stays in registers
//   route_wide_kernel    wider bf16 routers, many tokens: one tile per wave,
//                   the router streams through LDS for four tiles at once
//   route_split_k_kernel few tokens, or fp32: one tile per workgroup, its
//                   waves share the contraction
#pragma once
#include "common.hpp"

namespace unifmoe {

// Tokens are routed in tiles of kTileTok (a wave's lanes); the permutation's
// per-tile counts use the same tiles.
constexpr int kTileTok = 64;

struct RouteParams {
    int N, d, K, B, NL, NLP, lstride, key_bits;
    float tau, one_minus_2tau, t_mass, alpha_fixed;
    int max_shared, alpha_mode, mass_mode, fixed_k, select_mode;
    const void* X;
    const uint8_t* valid;
    const float* Wr;    // fp32 logits: [K+1][d]
    const float* mu;    // fp32 logits: [B][d]
    const u16* Wsplit;  // bf16 logits: the router's three parts (split_at), rows W_1..W_K, mu_1..mu_B, 0...
    float* alpha;
    int* nsh;
    uint64_t* mask;
    int* nres;
    int* eids;
    float* wts;
    int* bin_count;   // [kBinCopies][(K+1) << key_bits] pairs per (expert, mask key), or null
    int* tile_cnt;    // [ceil(N / kTileTok)][(K+1) B + K+1]: per tile of tokens, rows per (expert, block)
                      // slab, then pairs per expert; or null
    int* exp_total;   // [kExpCopies][K+1] pairs per expert (tile i adds into copy i % kExpCopies)
    int* pair_rank;   // [N][K+1]: slot of each pair within its bin copy
    // Copy job carried by the decisions launch (forward of bf16 layers): the
    // last cvt_blocks workgroups convert cvt_n8 16-byte chunks of bf16 at
    // cvt_src to fp16 at cvt_dst (bf16_to_f16_chunks). The decisions are
    // bound by latency and leave HBM bandwidth idle, which the copy uses.
    const u16* cvt_src;
    u16* cvt_dst;
    size_t cvt_n8;
    int cvt_blocks;
};

// bf16 -> fp16 of chunks [i0, n8) with stride `stride` (16-byte chunks of 8
// values). Each value is rounded to nearest even (exact for bf16 magnitudes
// in [2^-17, 65504]; larger ones become infinities). Four chunks per pass are
// loaded before any is converted, so each thread keeps four loads in flight.
__device__ __forceinline__ void bf16_to_f16_chunks(const u16* __restrict__ src, u16* __restrict__ dst, size_t n8,
                                                   size_t i0, size_t stride) {
    constexpr int U = 4;
    for (size_t i = i0; i < n8; i += U * stride) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * stride < n8) v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src) + i + u * stride);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u * stride < n8) {
                u32x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    o[q] = pack_f16x2(__uint_as_float(v[u][q] << 16), __uint_as_float(v[u][q] & 0xffff0000u));
                reinterpret_cast<u32x4*>(dst)[i + u * stride] = o;
            }
        }
    }
}

// The copy role of a routing launch: true (after doing its share of the
// copy) for the last p.cvt_blocks workgroups of the grid.
__device__ __forceinline__ bool route_copy_role(const RouteParams& p) {
    const int first = (int)gridDim.x - p.cvt_blocks;
    if ((int)blockIdx.x < first) return false;
    bf16_to_f16_chunks(p.cvt_src, p.cvt_dst, p.cvt_n8, (size_t)(blockIdx.x - first) * blockDim.x + threadIdx.x,
                       (size_t)p.cvt_blocks * blockDim.x);
    return true;
}

// Place of element k of row `row` of part `part` in the split router: blocks
// of 64 k, each holding all 3 NLP rows as 128-byte lines, so that what a k
// step reads is one contiguous stretch, whatever d.
__host__ __device__ __forceinline__ size_t split_at(int NLP, int part, int row, int k) {
    return ((size_t)(k >> 6) * 3 * NLP + (size_t)part * NLP + row) * 64 + (k & 63);
}

// Exact three-way split of an fp32 value into bf16 parts, in workgroups
// [0, nsplit); the workgroups after them zero zwords words at zero (the
// forward's counters, in the same launch).
__global__ void split_router_kernel(const float* __restrict__ Wr, const float* __restrict__ mu,
                                    int K, int B, int d, int NLP, u16* __restrict__ out, int nsplit,
                                    uint32_t* __restrict__ zero, size_t zwords) {
    if ((int)blockIdx.x >= nsplit) {
        const size_t stride = (size_t)(gridDim.x - nsplit) * blockDim.x;
        for (size_t i = (size_t)(blockIdx.x - nsplit) * blockDim.x + threadIdx.x; i < zwords; i += stride)
            zero[i] = 0u;
        return;
    }
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int total = NLP * d;
    if (i >= total) return;
    const int j = i / d, k = i - (i / d) * d;
    float w = 0.f;
    if (j < K) w = Wr[(size_t)(j + 1) * d + k];
    else if (j < K + B) w = mu[(size_t)(j - K) * d + k];
    const u16 hi = f2bf(w);
    const float r1 = w - bf2f(hi);
    const u16 mid = f2bf(r1);
    const float r2 = r1 - bf2f(mid);
    out[split_at(NLP, 0, j, k)] = hi;
    out[split_at(NLP, 1, j, k)] = mid;
    out[split_at(NLP, 2, j, k)] = f2bf(r2);
}

// Total-order key of a float for ranking: for non-NaN values it orders as
// the float comparison does (-0 is first mapped to +0, so the two tie), and
// a NaN gets a fixed place, so ranks computed with it always form a
// permutation, whatever the inputs hold.
__device__ __forceinline__ uint32_t rank_key(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Entry c of a list of L as one number that orders by (value descending,
// index ascending) under > : the value's rank_key in the top 32 mantissa
// bits of a double, L - 1 - c in the low ones. All entries share one binade
// (exponent field 1), so they compare as integers do, as finite normal
// numbers, and a compare-exchange is one v_max_f64 and one v_min_f64. 0.0
// comes after every entry.
template <int L>
__device__ __forceinline__ double order_key(float f, int c) {
    const uint32_t r = rank_key(f);
    return __hiloint2double((int)(0x00100000u | (r >> 12)), (int)((r << 20) | (uint32_t)(L - 1 - c)));
}
// The value's rank_key and the index of an order_key.
__device__ __forceinline__ uint32_t order_value(double k) {
    return ((uint32_t)__double2hiint(k) << 12) | ((uint32_t)__double2loint(k) >> 20);
}
template <int L>
__device__ __forceinline__ int order_index(double k) {
    return (L - 1) - (int)((uint32_t)__double2loint(k) & (L - 1));
}

// Batcher's odd-even merge sort of a[LO .. LO + N), largest first (N a power
// of two): 19, 63, 191 and 543 compare-exchanges for 8, 16, 32 and 64.
__device__ __forceinline__ void order_pair(double& a, double& b) {
    const double x = __builtin_fmax(a, b), y = __builtin_fmin(a, b);
    a = x;
    b = y;
}
template <int LO, int N, int R, int L>
__device__ __forceinline__ void odd_even_merge(double (&a)[L]) {
    if constexpr (2 * R < N) {
        odd_even_merge<LO, N, 2 * R>(a);
        odd_even_merge<LO + R, N, 2 * R>(a);
#pragma unroll
        for (int i = LO + R; i + R < LO + N; i += 2 * R) order_pair(a[i], a[i + R]);
    } else {
        order_pair(a[LO], a[LO + R]);
    }
}
template <int LO, int N, int L>
__device__ __forceinline__ void sort_descending(double (&a)[L]) {
    if constexpr (N > 1) {
        sort_descending<LO, N / 2>(a);
        sort_descending<LO + N / 2, N / 2>(a);
        odd_even_merge<LO, N, 1>(a);
    }
}

// The set of indices of the first n entries of a sorted list (n per lane).
template <int L>
__device__ __forceinline__ uint64_t first_indices(const double (&a)[L], int n) {
    if constexpr (L <= 32) {
        uint32_t m = 0;   // bit L - 1 - index
#pragma unroll
        for (int i = 0; i < L; ++i) m |= (i < n) ? 1u << ((uint32_t)__double2loint(a[i]) & (L - 1)) : 0u;
        return __brev(m) >> (32 - L);
    } else {
        uint64_t m = 0;
#pragma unroll
        for (int i = 0; i < L; ++i) m |= (i < n) ? 1ull << ((uint32_t)__double2loint(a[i]) & (L - 1)) : 0ull;
        return __brevll(m);
    }
}

// Orders this wave's LDS accesses for the compiler (a wave's LDS operations
// execute in order).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lanes of the wave that add to the same counter, gathered so that one of them
// can add for all: up to kGatherRounds times the first lane left takes those
// with its key along (key < 0: not taking part); the rest stay alone. A key
// that many lanes share is met in the first rounds. Without this the 64 atomics
// of a wave on one counter queue up at the L2: with few masks over all tokens
// (prefix selection, skewed demand, 51,328 tokens) the decisions' launch took
// 82 us, 38 us now. Used where the masks are few (prefix selection, or at most
// 4 key bits); elsewhere the rounds cost more than they save (2.5 us of one
// image of a DeiT-S layer).
constexpr int kGatherRounds = 4;
struct Gather {
    int lead, rank, count;   // the lane that adds, this lane's place, lanes in its group
};
__device__ __forceinline__ Gather gather_key(int key, bool few) {
    Gather g{lane_id(), 0, 1};
    if (!few) return g;
    bool todo = key >= 0;
#pragma unroll
    for (int r = 0; r < kGatherRounds; ++r) {
        const uint64_t left = ballot(todo);
        const int f = left ? __builtin_ctzll(left) : 0;
        const bool same = todo && key == __builtin_amdgcn_readlane(key, f);
        const uint64_t m = ballot(same);
        if (same) g = Gather{f, (int)__popcll(m & lanes_below()), (int)__popcll(m)};
        todo = todo && !same;
    }
    return g;
}

// x / n for x < 2^16 and 1 <= n <= 2^15, with m = div_magic(n).
__device__ __forceinline__ uint32_t div_magic(int n) { return n > 1 ? 0xffffffffu / (uint32_t)n + 1u : 0u; }
__device__ __forceinline__ int div_by(int x, uint32_t m) { return m ? (int)__umulhi((uint32_t)x, m) : x; }

// Padded length of the sorted lists: the smallest power of two >= max(K, B),
// at least 8.
__host__ __device__ __forceinline__ int decide_length(int K, int B) {
    const int n = K > B ? K : B;
    return n <= 8 ? 8 : n <= 16 ? 16 : (n <= 32 ? 32 : 64);
}

// Decisions of Sec. III-B and III-C for one tile of 64 tokens, one lane of one
// wave per token. `rows` (LDS, stride p.lstride, odd) holds the tokens'
// logits: shared demand, K experts, B priorities; `bits` is tile_words
// 8-byte words of LDS. Tokens past the layer write nothing.
//   alpha, b    from the shared logit
//   I_shr       the first b of the sorted priorities
//   softmax     maximum, exponentials, their sum in index order, fp32
//   q, p        the sorted affinities
//   P_r, k      sums p_0..p_r in order; k is the first r whose prefix
//               reaches the target, else K
// All arithmetic is the paper's order in fp32 with explicitly rounded
// operations. With one lane per token nothing crosses lanes until the record
// is written (through LDS, so the stores are whole lines): 64 tokens cost
// about as many wave instructions as the 4 tokens of a pass did when a group
// of lanes shared a token and every broadcast was an LDS permute.
//
// NW waves work on the tile (whole workgroups of NW waves, or NW = 1 and any
// number of them): the first decides, then all of them write the record and
// the tile's counts, and the others take the pair slots. Where there are few
// tiles, what follows the decisions is a chain of instructions and round trips
// on an otherwise idle compute unit (see kDecideWaves for what it costs).
__host__ __device__ __forceinline__ int tile_words(int B, int K, int nw) {
    return B + K + 1 + (nw > 1 ? kTileTok + kTileTok / 2 : 0);
}

template <int L, int NW>
__device__ __forceinline__ void decide_tile(const RouteParams& p, float* rows, uint64_t* bits, int tile, int wave) {
    const int K = p.K, B = p.B, ls = p.lstride;
    const int lane = lane_id(), tok0 = tile * kTileTok, tok = tok0 + lane;
    const int tid = wave * kWave + lane;   // among the tile's threads
    constexpr int T = NW * kWave;
    const int ntok = min(kTileTok, p.N - tok0);
    float* row = rows + lane * ls;
    int* irow = reinterpret_cast<int*>(row);
    const int* irows = reinterpret_cast<const int*>(rows);
    // For the other waves: the tokens' I_shr, and their k (0: not valid).
    uint64_t* const masks = bits + B + K + 1;
    int* const ks_of = reinterpret_cast<int*>(masks + kTileTok);
    const bool lead = NW == 1 || wave == 0;
    // Orders the tile's LDS accesses between its waves.
    auto settle = [&]() {
        if constexpr (NW == 1) wave_lds_order();
        else __syncthreads();
    };
    const uint64_t full = (B == 64) ? ~0ull : ((1ull << B) - 1ull);
    const bool v = lead && lane < ntok && (p.valid == nullptr || p.valid[tok] != 0);
    double a[L];
    uint64_t mask = 0, sel = 0;
    int k = 0;
    if (lead) {
        // Eq. alpha (adaptive) or the fixed-alpha ablation.
        float alpha;
        if (p.alpha_mode == 0) {
            const float sig = __fdiv_rn(1.0f, __fadd_rn(1.0f, expf(-row[0])));
            alpha = __fadd_rn(p.tau, __fmul_rn(p.one_minus_2tau, sig));
        } else {
            alpha = p.alpha_fixed;
        }
        // Eq. block-count, half to even; clamp to [1, B-1] (adaptive), cap.
        // (fminf/fmaxf drop a NaN alpha, so b stays in range for any input.)
        int b = (int)rintf(fminf(fmaxf(__fmul_rn((float)B, alpha), 0.0f), (float)B));
        if (p.alpha_mode == 0) b = min(max(b, 1), B - 1);
        b = min(b, p.max_shared);

        // Eq. block-priority / shared-indices: the b largest priorities, ties to
        // the lower index.
        if (p.select_mode == 0) {
#pragma unroll
            for (int c = 0; c < L; ++c) a[c] = (c < B) ? order_key<L>(row[1 + K + c], c) : 0.0;
            sort_descending<0, L>(a);
            mask = first_indices<L>(a, b);
        } else {
            mask = (b >= 64) ? ~0ull : ((1ull << b) - 1ull);
        }

        // Eq. residual-router-score: max-subtracted softmax, index-order sum.
        float e[L];
        float m = -INFINITY;
#pragma unroll
        for (int j = 0; j < L; ++j)
            if (j < K) {
                e[j] = row[1 + j];
                m = fmaxf(m, e[j]);
            }
        float S = 0.f;
#pragma unroll
        for (int j = 0; j < L; ++j)
            if (j < K) {
                e[j] = expf(__fsub_rn(e[j], m));
                S = __fadd_rn(S, e[j]);
            }
        // Eq. sorted-affinity: by decreasing affinity, ties to the lower index.
#pragma unroll
        for (int j = 0; j < L; ++j) a[j] = (j < K) ? order_key<L>(__fdiv_rn(e[j], S), j) : 0.0;
        sort_descending<0, L>(a);
        // The affinities back as floats (what rank_key maps to them), in order.
        auto affinity = [&](int i) {
            const uint32_t r = order_value(a[i]);
            return __uint_as_float((r & 0x80000000u) ? r & 0x7fffffffu : ~r);
        };
        // Eq. beta / expert-count: the smallest prefix reaching the target.
        if (p.mass_mode == 2) {
            k = p.fixed_k;
        } else {
            const float beta = __fsub_rn(1.0f, alpha);
            const float target = (p.mass_mode == 0) ? fminf(beta, p.t_mass) : p.t_mass;
            float P = 0.f;
            bool reached = false;
            k = 1;
#pragma unroll
            for (int i = 0; i < L; ++i)
                if (i < K) {
                    P = __fadd_rn(P, affinity(i));
                    reached = reached || P >= target;
                    k += reached ? 0 : 1;
                }
            k = min(k, K);
        }
        sel = v ? first_indices<L>(a, k) : 0ull;   // bit j: expert j + 1

        // The record. Rows of K values per token go through the token's LDS row.
        if (lane < ntok) {
            p.alpha[tok] = v ? alpha : 0.f;
            p.nsh[tok] = v ? b : 0;
            p.mask[tok] = v ? mask : 0ull;
            p.nres[tok] = v ? k : 0;
        }
#pragma unroll
        for (int i = 0; i < L; ++i)
            if (i < K) row[i] = v ? affinity(i) : 0.f;
        if constexpr (NW > 1) {
            masks[lane] = mask;
            ks_of[lane] = v ? k : 0;
        }
    }
    const uint32_t mk = div_magic(K);
    settle();
    for (int x = tid; x < ntok * K; x += T) {
        const int t = div_by(x, mk);
        p.wts[(size_t)tok0 * K + x] = rows[t * ls + x - t * K];
    }
    settle();
    if (lead) {
#pragma unroll
        for (int i = 0; i < L; ++i)
            if (i < K) irow[i] = v ? 1 + order_index<L>(a[i]) : -1;
    }
    settle();
    for (int x = tid; x < ntok * K; x += T) {
        const int t = div_by(x, mk);
        p.eids[(size_t)tok0 * K + x] = irows[t * ls + x - t * K];
    }
    if (p.bin_count == nullptr) return;

    // Pairs per (expert, key of the pair's block mask): one shared pair and
    // k residual pairs per valid token. The count a bin copy had before a
    // pair adds itself is the pair's slot within that copy (pair_rank), so
    // the scatter needs no atomics; slots inside a bin follow the order the
    // atomics land in, and no result depends on it (every GEMM row is
    // computed from its own pair). The atomics of a batch are all issued
    // before a slot is stored. With several waves the first one makes the
    // tile's bit matrices meanwhile, and the others take a batch each in turn.
    const int kb = p.key_bits, K1 = K + 1, nbin = K1 << kb;
    settle();
    if (NW == 1 || !lead) {
        const int kv = NW == 1 ? (v ? k : 0) : ks_of[lane];
        const uint64_t ms = NW == 1 ? mask : masks[lane];
        const bool valid = kv > 0;   // k >= 1 for every valid token
        const int ks = mask_key(ms, B, kb), kr = mask_key(~ms & full, B, kb);
        const int bc = tile % kBinCopies;
        int kmax = kv;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o));
        kmax = __builtin_amdgcn_readfirstlane(kmax);
        constexpr int kBatch = 4, WB = NW == 1 ? 1 : NW - 1;   // waves that take batches
        const int w = NW == 1 ? 0 : wave - 1;
        const bool few = p.select_mode != 0 || kb <= 4;
        Gather g0{lane, 0, 1};
        int r0 = 0;
        if (w == 0) {
            g0 = gather_key(valid ? ks : -1, few);
            if (valid && g0.rank == 0) r0 = atomicAdd(&p.bin_count[bin_counter(ks, bc, nbin)], g0.count);
        }
        for (int i0 = w * kBatch; i0 < kmax; i0 += WB * kBatch) {
            Gather g[kBatch];
            int s[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const bool in = i0 + u < kv;
                const int key = in ? (irow[i0 + u] << kb) + kr : -1;
                g[u] = gather_key(key, few);
                s[u] = 0;
                if (in && g[u].rank == 0) s[u] = atomicAdd(&p.bin_count[bin_counter(key, bc, nbin)], g[u].count);
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int slot = __shfl(s[u], g[u].lead) + g[u].rank;
                if (i0 + u < kv) irow[i0 + u] = slot;
            }
        }
        if (w == 0) {
            r0 = __shfl(r0, g0.lead) + g0.rank;
            irow[K] = r0;
        }
    }
    // The tile's bit matrices: bits[c] the tokens that share block c,
    // bits[B + e] the tokens on expert e.
    if (lead && p.tile_cnt != nullptr) {
        uint64_t mine = 0;
        const uint64_t vm = v ? mask : 0ull;
        for (int c = 0; c < B; ++c) {
            const uint64_t t = ballot((vm >> c) & 1ull);
            mine = (lane == c) ? t : mine;
        }
        if (lane < B) bits[lane] = mine;
        const uint64_t all = ballot(v);
        for (int j = 0; j < K; ++j) {
            const uint64_t t = ballot((sel >> j) & 1ull);
            mine = (lane == j) ? t : mine;
        }
        if (lane < K) bits[B + 1 + lane] = mine;
        if (lane == 0) bits[B] = all;
    }
    settle();
    const uint32_t mk1 = div_magic(K1);
    for (int x = tid; x < ntok * K1; x += T) {
        const int t = div_by(x, mk1), j = x - t * K1;
        p.pair_rank[(size_t)tok0 * K1 + x] = irows[t * ls + (j == 0 ? K : j - 1)];
    }
    if (p.tile_cnt == nullptr) return;

    // The tile's counts: rows per slab (the shared expert on I_shr, each
    // selected residual expert on I_res) and pairs per expert.
    const int nslab = K1 * B, ncnt = nslab + K1;
    const uint32_t mb = div_magic(B);
    int* cnt = p.tile_cnt + (size_t)tile * ncnt;
    for (int x = tid; x < nslab; x += T) {
        const int ee = div_by(x, mb);
        const uint64_t sh = bits[x - ee * B], te = bits[B + ee];
        cnt[x] = __popcll(te & (ee == 0 ? sh : ~sh));
    }
    for (int x = tid; x < K1; x += T) {
        const int c = __popcll(bits[B + x]);
        cnt[nslab + x] = c;
        // Pairs per expert also into the totals (few atomics, spread).
        if (c) atomicAdd(&p.exp_total[(tile % kExpCopies) * K1 + x], c);
    }
}

// decide_tile with the list length of the layer (see decide_length).
template <int NW>
__device__ __forceinline__ void decide_tile_any(const RouteParams& p, float* rows, uint64_t* bits, int tile, int wave) {
    switch (decide_length(p.K, p.B)) {
        case 8: decide_tile<8, NW>(p, rows, bits, tile, wave); break;
        case 16: decide_tile<16, NW>(p, rows, bits, tile, wave); break;
        case 32: decide_tile<32, NW>(p, rows, bits, tile, wave); break;
        default: decide_tile<64, NW>(p, rows, bits, tile, wave); break;
    }
}

// This lane's 8 products of a k step with W_shr added to s in fp32.
__device__ __forceinline__ float shared_dot(u32x4 x, u32x4 w0, u32x4 w1, float s) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        s = fmaf(__uint_as_float(x[q] << 16), __uint_as_float(q < 2 ? w0[2 * q] : w1[2 * q - 4]), s);
        s = fmaf(__uint_as_float(x[q] & 0xffff0000u), __uint_as_float(q < 2 ? w0[2 * q + 1] : w1[2 * q - 3]), s);
    }
    return s;
}

// One wave's (partial) logits of its 64 tokens into LDS rows of stride ls:
// column 0 the shared demand, columns 1.. the MFMA tiles.
template <int NCT>
__device__ __forceinline__ void put_logits(float* P, int ls, const f32x4 (&acc)[4][NCT], const float (&sh)[4]) {
    const int lane = lane_id();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float v = sh[r];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        if (lane < 16) P[(r * 16 + lane) * ls] = v;
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                P[(r * 16 + (lane >> 4) * 4 + e) * ls + 1 + ct * 16 + (lane & 15)] = acc[r][ct][e];
    }
}

// One tile per workgroup of kSplitWaves waves, which share the contraction;
// the partial logits are summed in wave order and wave 0 decides the tile.
// For few tiles the chain of k steps of one wave sets the time, and this
// splits it (16,384 tokens of d = 768, K = B = 16: 21 us against 25 us in two
// launches; d = 1024, K = B = 32: 38 against 46 us); with more tiles the router
// rows it re-reads per tile make it slower (see kSplitKTiles). (Routers of 113
// to 128 columns spill 18 registers in the loop of k steps; 16,000 tokens of
// d = 1024, K = B = 64 take 72 us.)
// NCT: 16-column tiles of the bf16 router; 0: fp32 tokens. The
// last p.cvt_blocks workgroups do the launch's copy job.
constexpr int kSplitWaves = 4;

template <int NCT>
__device__ __forceinline__ void split_k_logits_bf16(const RouteParams& p, float* P, int tok0, int wave) {
    constexpr int RT = kTileTok / 16;
    const int lane = lane_id();
    const u16* X = static_cast<const u16*>(p.X);
    f32x4 acc[RT][NCT];
    float sh[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        sh[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NCT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int kof = (lane >> 4) * 8;
    const u16* xr[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)   // rows past N read row N - 1; their logits are never used
        xr[i] = X + (size_t)min(tok0 + i * 16 + (lane & 15), p.N - 1) * p.d + kof;
    const float* wsh = p.Wr + kof;           // row 0 of the fp32 router: W_shr
    const int nks = p.d / 32;
    const int ks0 = wave * nks / kSplitWaves, n = (wave + 1) * nks / kSplitWaves - ks0;
    // Every operand of a k step is loaded together, a step ahead of its use.
    struct Set {
        u32x4 a[RT], b[3][NCT], s0, s1;
    };
    Set ring[2];
    auto load = [&](int ks, Set& S) {
        const int k0 = (ks0 + ks) * 32;
#pragma unroll
        for (int i = 0; i < RT; ++i) S.a[i] = ld16(xr[i] + k0);
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct)
                S.b[part][ct] = ld16(p.Wsplit + split_at(16 * NCT, part, ct * 16 + (lane & 15), k0 + kof));
        S.s0 = ld16(wsh + k0);
        S.s1 = ld16(wsh + k0 + 4);
    };
    auto compute = [&](const Set& S) {
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
            for (int part = 0; part < 3; ++part) {
                const bf16x8 b = as_bf16x8(S.b[part][ct]);
#pragma unroll
                for (int i = 0; i < RT; ++i) acc[i][ct] = mfma16x16x32(as_bf16x8(S.a[i]), b, acc[i][ct]);
            }
#pragma unroll
        for (int i = 0; i < RT; ++i) sh[i] = shared_dot(S.a[i], S.s0, S.s1, sh[i]);
    };
    if (n > 0) load(0, ring[0]);
    for (int ks = 0; ks < n; ks += 2) {
        if (ks + 1 < n) load(ks + 1, ring[1]);
        compute(ring[0]);
        if (ks + 1 < n) {
            if (ks + 2 < n) load(ks + 2, ring[0]);
            compute(ring[1]);
        }
    }
    put_logits<NCT>(P, p.lstride, acc, sh);
}

// fp32 tokens: all 1 + K + B columns on the matrix cores in fp32, 64 columns
// at a time. Lane l brings row l % 16 of its operand and, per 16 k, the four
// values k0 + 4 (l / 16) + 0..3, one per product (both operands take the same
// k, in whatever order). d need not be a multiple of 16 nor the rows aligned.
__device__ __forceinline__ void split_k_logits_f32(const RouteParams& p, float* P, int tok0, int wave) {
    constexpr int RT = kTileTok / 16, CT = 4;
    const int lane = lane_id(), kof = (lane >> 4) * 4;
    const float* X = static_cast<const float*>(p.X);
    const int nks = ceil_div(p.d, 16);
    const int ks0 = wave * nks / kSplitWaves, ks1 = (wave + 1) * nks / kSplitWaves;
    auto load4 = [&](const float* r, int k) {   // r[k..k+3], zero past d
        f32x4 v;
        if (k + 4 <= p.d) {
            v = ld_f32x4(r + k);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (k + i < p.d) ? r[k + i] : 0.f;
        }
        return v;
    };
    const float* xr[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) xr[i] = X + (size_t)min(tok0 + i * 16 + (lane & 15), p.N - 1) * p.d;
    for (int c0 = 0; c0 < p.NL; c0 += 16 * CT) {
        const float* wr[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int c = min(c0 + j * 16 + (lane & 15), p.NL - 1);
            wr[j] = (c <= p.K) ? p.Wr + (size_t)c * p.d : p.mu + (size_t)(c - 1 - p.K) * p.d;
        }
        f32x4 acc[RT][CT];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int ks = ks0; ks < ks1; ++ks) {
            f32x4 x[RT], w[CT];
#pragma unroll
            for (int i = 0; i < RT; ++i) x[i] = load4(xr[i], ks * 16 + kof);
#pragma unroll
            for (int j = 0; j < CT; ++j) w[j] = load4(wr[j], ks * 16 + kof);
#pragma unroll
            for (int j = 0; j < CT; ++j)
                if (c0 + j * 16 < p.NL)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int i = 0; i < RT; ++i)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][q], w[j][q], acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int c = c0 + j * 16 + (lane & 15);
            if (c < p.NL)
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) P[(i * 16 + (lane >> 4) * 4 + e) * p.lstride + c] = acc[i][j][e];
        }
    }
}

template <int NCT>
__global__ __launch_bounds__(kSplitWaves * 64) void route_split_k_kernel(RouteParams p) {
    if (route_copy_role(p)) return;
    extern __shared__ __attribute__((aligned(16))) float lds_route[];
    const int ls = p.lstride, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tile = NCT > 0 ? (int)blockIdx.x : (int)flat_block(), part = kTileTok * ls;
    if (NCT == 0 && flat_block() >= (size_t)(p.N + kTileTok - 1) / kTileTok) return;
    if constexpr (NCT > 0) split_k_logits_bf16<NCT>(p, lds_route + wave * part, tile * kTileTok, wave);
    else split_k_logits_f32(p, lds_route + wave * part, tile * kTileTok, wave);
    __syncthreads();
    for (int x = threadIdx.x; x < part; x += kSplitWaves * 64) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kSplitWaves; ++w) v += lds_route[w * part + x];
        lds_route[x] = v;
    }
    __syncthreads();
    decide_tile_any<kSplitWaves>(p, lds_route, reinterpret_cast<uint64_t*>(lds_route + kSplitWaves * part), tile, wave);
}

// bf16 routers of any width over many tokens: 4 waves, one 64-token tile
// each. The router's three parts stream through LDS 64 k at a time (one
// 128-byte line per row, the GEMM engine's swizzle; two slots), shared by the
// four tiles, the token rows into registers, both one stage ahead; then each
// wave decides its own tile from its logits in LDS (no logits in memory).
// What bounds it is the HBM read of X and, per stage, the chain of fragment
// reads and products of one wave (two workgroups share a compute unit, so
// registers are the limit: W_shr goes through LDS and only one step's
// fragments are read ahead; with spills in the loop a stage took 4 us, since
// every reload waits behind the copies in flight. The nine or ten registers
// that the kernels of 17 to 64 columns spill now are the decisions', after the
// loop). d = 1024, K = B = 32:
// 100,001 tokens 477 us with one fused kernel of 4 tokens per decision pass,
// 79 us here; 32,768 tokens 71 us with a tile per workgroup, 47 us here.
// The last p.cvt_blocks workgroups do the launch's copy job.
constexpr int kWideWaves = 4;

template <int NCT>
__global__ __launch_bounds__(kWideWaves * 64, NCT <= 4 ? 2 : 1) void route_wide_kernel(RouteParams p) {
    if (route_copy_role(p)) return;
    constexpr int RT = kTileTok / 16, ROWS = 48 * NCT, COPIES = ROWS / 8, SLOT = ROWS * 128;
    extern __shared__ __attribute__((aligned(16))) float lds_route[];
    char* const stage = reinterpret_cast<char*>(lds_route);
    char* const shr = stage + 2 * SLOT;
    const int ls = p.lstride, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tile = blockIdx.x * kWideWaves + wave, tok0 = tile * kTileTok;
    const u16* X = static_cast<const u16*>(p.X);
    const int nks = p.d / 32, nst = (nks + 1) / 2;
    const int kof = (lane >> 4) * 8;
    const u16* xr[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)   // rows past N read row N - 1; their logits are never used
        xr[i] = X + (size_t)min(tok0 + i * 16 + (lane & 15), p.N - 1) * p.d + kof;
    f32x4 acc[RT][NCT];
    float sh[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        sh[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NCT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto copy_stage = [&](int st) {
        char* base = stage + (st & 1) * SLOT;
        for (int q = wave; q < COPIES; q += kWideWaves) {
            const int r = q * 8 + (lane >> 3);
            dma16(p.Wsplit + ((size_t)st * ROWS + r) * 64 + 8 * ((lane & 7) ^ ((r >> 1) & 7)), base + q * 1024);
        }
        if (wave == 0) dma4(p.Wr + min(st * 64 + lane, p.d - 1), shr + (st & 1) * 256);   // W_shr
    };
    struct Set {
        u32x4 a[2][RT];
    };
    Set ring[2];
    auto load = [&](int st, Set& S) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k0 = min(2 * st + h, nks - 1) * 32;
#pragma unroll
            for (int i = 0; i < RT; ++i) S.a[h][i] = ld16(xr[i] + k0);
        }
    };
    // The router's fragments of step x of a stage: column tile x / 2, k step
    // x % 2, three parts.
    auto fragments = [&](int st, int x, u32x4 (&w)[3]) {
        const char* base = stage + (st & 1) * SLOT;
#pragma unroll
        for (int part = 0; part < 3; ++part) {
            const int r = part * 16 * NCT + (x >> 1) * 16 + (lane & 15);
            w[part] = ld16(base + r * 128 + (((4 * (x & 1) + (lane >> 4)) ^ ((r >> 1) & 7)) << 4));
        }
    };
    // A stage's products are summed on their own, small parts first, and then
    // added to the logits: a sixth of the roundings at the logits' magnitude
    // that one running accumulator would take. The next step's fragments are
    // read while this one's are multiplied.
    auto compute = [&](int st, const Set& S) {
        const bool both = 2 * st + 1 < nks;   // the last stage of an odd count of k steps has one
        u32x4 w[2][3];
        f32x4 t[RT];
        fragments(st, 0, w[0]);
#pragma unroll
        for (int x = 0; x < 2 * NCT; ++x) {
            if (x + 1 < 2 * NCT) fragments(st, x + 1, w[(x + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            if ((x & 1) == 0) {
#pragma unroll
                for (int i = 0; i < RT; ++i) t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            if ((x & 1) == 0 || both) {
#pragma unroll
                for (int part = 2; part >= 0; --part)
#pragma unroll
                    for (int i = 0; i < RT; ++i)
                        t[i] = mfma16x16x32(as_bf16x8(S.a[x & 1][i]), as_bf16x8(w[x & 1][part]), t[i]);
            }
            if (x & 1) {
#pragma unroll
                for (int i = 0; i < RT; ++i) acc[i][x >> 1] += t[i];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const char* ws = shr + (st & 1) * 256 + kof * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 1 && !both) break;
            const u32x4 s0 = ld16(ws + h * 128), s1 = ld16(ws + h * 128 + 16);
#pragma unroll
            for (int i = 0; i < RT; ++i) sh[i] = shared_dot(S.a[h][i], s0, s1, sh[i]);
        }
    };
    // At the top of a stage its copies and rows have landed and every wave
    // has left the slot that the next stage fills.
    auto step = [&](int st, const Set& S, Set& next) {
        wait_vmcnt<0>();
        __syncthreads();
        if (st + 1 < nst) {
            copy_stage(st + 1);
            load(st + 1, next);
        }
        __builtin_amdgcn_sched_barrier(0);
        compute(st, S);
    };
    copy_stage(0);
    load(0, ring[0]);
    for (int st = 0; st < nst; st += 2) {
        step(st, ring[0], ring[1]);
        if (st + 1 < nst) step(st + 1, ring[1], ring[0]);
    }
    __syncthreads();   // the logit rows take the place of the stages
    float* rows = lds_route + wave * kTileTok * ls;
    put_logits<NCT>(rows, ls, acc, sh);
    wave_lds_order();
    if (tok0 >= p.N) return;
    uint64_t* bits = reinterpret_cast<uint64_t*>(lds_route + kWideWaves * kTileTok * ls) + wave * tile_words(p.B, p.K, 1);
    decide_tile_any<1>(p, rows, bits, tile, 0);
}

// Logits of bf16 tokens when the router fits in registers (1 + K + B <= 32
// columns, d <= 1024), persistent: one workgroup of 8 waves takes the 64-token
// tiles blockIdx.x, blockIdx.x + gridDim.x, ... Wave w owns k steps
// [w nks / 8, (w + 1) nks / 8) and keeps the router's three bf16 parts and
// W_shr for them in registers for all its tiles, so only token rows stream
// from memory (the next tile's rows load while this tile's partial logits
// are reduced); the 8 partial sets are summed in a fixed order and each
// token's 1 + 16 NCT logits written to logits[N][1 + 16 NCT]. The decisions
// run in route_decide_kernel.
constexpr int kRpTok = kTileTok;
constexpr int kRpWaves = 8;
constexpr int kRpThreads = kRpWaves * 64;

template <int NCT, int KPW>
__global__ __launch_bounds__(kRpThreads) void route_logits_kernel(RouteParams p, float* __restrict__ logits) {
    constexpr int RT = kRpTok / 16;          // 16-row fragments per tile
    constexpr int ncols = 1 + 16 * NCT;
    extern __shared__ float lds_route[];
    const int ls = p.lstride;
    float* Pbuf = lds_route;                                     // [8][64][ls] partial logits
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntile_all = (p.N + kRpTok - 1) / kRpTok;
    const int nt = (ntile_all - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;

    // This wave's k steps (32 deep) and the router parts for them.
    const int nks = p.d / 32;
    const int kb = wave * nks / kRpWaves, kn = (wave + 1) * nks / kRpWaves - kb;   // kn <= KPW
    const int kof = (lane >> 4) * 8;
    u32x4 W[KPW][3][NCT], S0[KPW], S1[KPW];
#pragma unroll
    for (int j = 0; j < KPW; ++j) {
        const int k0 = (kb + (j < kn ? j : 0)) * 32;
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct)
                W[j][part][ct] = ld16(p.Wsplit + split_at(16 * NCT, part, ct * 16 + (lane & 15), k0 + kof));
        S0[j] = ld16(p.Wr + kof + k0);
        S1[j] = ld16(p.Wr + kof + k0 + 4);
    }
    const u16* X = static_cast<const u16*>(p.X);
    u32x4 xa[KPW][RT];
    auto load_x = [&](int i) {
        const int tok0 = ((int)blockIdx.x + i * (int)gridDim.x) * kRpTok;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            // Rows past N read row N - 1; their logits are never written.
            const u16* xr = X + (size_t)min(tok0 + r * 16 + (lane & 15), p.N - 1) * p.d + kof;
#pragma unroll
            for (int j = 0; j < KPW; ++j) xa[j][r] = ld16(xr + (kb + (j < kn ? j : 0)) * 32);
        }
    };
    if (nt > 0) load_x(0);
    for (int i = 0; i < nt; ++i) {
        const int tok0 = ((int)blockIdx.x + i * (int)gridDim.x) * kRpTok;
        f32x4 acc[RT][NCT];
        float sh[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            sh[r] = 0.f;
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) acc[r][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < KPW; ++j) {
            if (j < kn) {
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
                    for (int part = 0; part < 3; ++part)
#pragma unroll
                        for (int r = 0; r < RT; ++r)
                            acc[r][ct] = mfma16x16x32(as_bf16x8(xa[j][r]), as_bf16x8(W[j][part][ct]), acc[r][ct]);
#pragma unroll
                for (int r = 0; r < RT; ++r) sh[r] = shared_dot(xa[j][r], S0[j], S1[j], sh[r]);
            }
        }
        // The next tile's rows are in flight during the reduction.
        if (i + 1 < nt) load_x(i + 1);
        // This wave's partial logits. (The barrier after the previous tile's
        // sum orders its reads of Pbuf before these writes.)
        put_logits<NCT>(Pbuf + wave * kRpTok * ls, ls, acc, sh);
        lds_barrier();
        // Sum of the 8 k slices, in wave order, straight to memory.
        const int ntok = min(kRpTok, p.N - tok0);
        for (int e = tid; e < ntok * ncols; e += blockDim.x) {
            const int t = e / ncols, c = e - t * ncols;
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < kRpWaves; ++w) v += Pbuf[(w * kRpTok + t) * ls + c];
            logits[(size_t)tok0 * ncols + e] = v;
        }
        lds_barrier();
    }
}

// Decisions from the logits route_logits_kernel wrote ([N][lstride]), one
// 64-token tile per workgroup of NW waves: kDecideWaves while the tiles are
// few (see kDecideTiles), else one. A forward's decisions of 20,000 tokens
// (313 tiles, K = 16, B = 8), which also take the pair slots and the counts,
// need 24.9 us from one wave per tile, and four take 4 to 6 us off the call
// (17,000 tokens of d = 512: 282 -> 277 us). The last p.cvt_blocks workgroups
// do the launch's copy job instead.
constexpr int kDecideWaves = 4;

template <int L, int NW>
__global__ __launch_bounds__(NW * 64) void route_decide_kernel(RouteParams p, const float* __restrict__ logits) {
    if (route_copy_role(p)) return;
    extern __shared__ __attribute__((aligned(16))) float lds_dec[];
    const int tile = blockIdx.x, tok0 = tile * kTileTok, ntok = min(kTileTok, p.N - tok0);
    const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const float* src = logits + (size_t)tok0 * p.lstride;
    // Rows past the layer keep whatever LDS holds; they are not decided.
    batched_copy(ntok * p.lstride, [&](int i) { return src[i]; }, [&](int i, float v) { lds_dec[i] = v; });
    if constexpr (NW == 1) wave_lds_order();
    else __syncthreads();
    decide_tile<L, NW>(p, lds_dec, reinterpret_cast<uint64_t*>(lds_dec + kTileTok * p.lstride), tile, wave);
}

}  // namespace unifmoe
