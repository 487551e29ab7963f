// PFT construction (paper: Listing 1 PFT_construction() step 1 + histogram; Section 4.1.1 ERI-arrays):
// a stable counting sort of the T*k flat entries by expert id, in one kernel for up to kEriDirectChunks chunks of
// entries (eri_direct_kernel) and in three small ones beyond:
//   1. per-chunk histograms of expert ids            (chunk = 1024 consecutive flat entries)
//   2. column scan over chunks + scan over experts   -> tokens_per_expert, expert_offsets, chunk bases
//   3. per-chunk stable ranking and scatter          -> token_ids, expert_ids, combine_weights, row_of_slot
// Within an expert, rows keep ascending flat order, so the result is unique and reproducible.
#include "xmoe_internal.h"
#include "xmoe_sizes.h"

namespace xmoe {

constexpr int kSubPerChunk = kEriChunk / 64;   // 16 wave-sized sub-chunks

__global__ __launch_bounds__(256) void eri_hist_kernel(const int32_t* __restrict__ topk_idx, int B, int E,
                                                       int32_t* __restrict__ chunk_counts) {
    __shared__ int hist[XMOE_MAX_EXPERTS];
    for (int e = threadIdx.x; e < E; e += 256) hist[e] = 0;
    __syncthreads();
    const int base = blockIdx.x * kEriChunk;
#pragma unroll
    for (int r = 0; r < kEriChunk / 256; ++r) {
        int n = base + r * 256 + threadIdx.x;
        if (n < B) {
            int e = topk_idx[n];
            if ((unsigned)e < (unsigned)E) atomicAdd(&hist[e], 1);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 256) chunk_counts[(size_t)blockIdx.x * E + e] = hist[e];
}

// one block: turns chunk_counts[c][e] into the exclusive prefix over chunks, writes tokens_per_expert and
// expert_offsets
__global__ __launch_bounds__(512) void eri_scan_kernel(int32_t* __restrict__ chunk_counts, int nchunks, int E,
                                                       int32_t* __restrict__ tokens_per_expert,
                                                       int32_t* __restrict__ expert_offsets) {
    __shared__ int tot[XMOE_MAX_EXPERTS];
    const int e = threadIdx.x;
    if (e < E) {
        // 16 chunks at a time: the loads of a batch are independent, so the walk costs nchunks/16 round trips to
        // memory instead of nchunks
        constexpr int kBatch = 16;
        int run = 0;
        for (int c0 = 0; c0 < nchunks; c0 += kBatch) {
            int v[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) v[j] = c0 + j < nchunks ? chunk_counts[(size_t)(c0 + j) * E + e] : 0;
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (c0 + j < nchunks) chunk_counts[(size_t)(c0 + j) * E + e] = run;
                run += v[j];
            }
        }
        tot[e] = run;
        tokens_per_expert[e] = run;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int i = 0; i < E; ++i) {
            expert_offsets[i] = run;
            run += tot[i];
        }
        expert_offsets[E] = run;
    }
}

// Rank of each of this thread's four entries among its 64-entry sub-chunk's entries of the same expert, and
// sub_count[s][e] (zeroed before): entries of expert e in sub-chunk s.
__device__ __forceinline__ void eri_rank(const int32_t* __restrict__ topk_idx, int base, int B, int E, int ebits,
                                         int* sub_count, int (&my_e)[kSubPerChunk / 4], int (&my_rank)[kSubPerChunk / 4]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < kSubPerChunk / 4; ++r) {
        const int sub = r * 4 + wave;
        const int n = base + sub * 64 + lane;
        const int e = n < B ? topk_idx[n] : -1;
        const bool ok = (unsigned)e < (unsigned)E;   // out-of-range ids (never produced by xmoe_route) are skipped
        // lanes of this wave holding the same expert: intersect ballots bit by bit
        unsigned long long same = __ballot(ok);
        for (int b = 0; b < ebits; ++b) {
            unsigned long long bal = __ballot(ok && ((e >> b) & 1));
            same &= ((e >> b) & 1) ? bal : ~bal;
        }
        const unsigned long long below = (1ull << lane) - 1ull;
        my_e[r] = e;
        my_rank[r] = __popcll(same & below);
        if (ok && (same & below) == 0ull) sub_count[sub * E + e] = __popcll(same);   // first lane of its group
    }
}

// sub_count[.][e] -> first row of every sub-chunk's entries of expert e
__device__ __forceinline__ void eri_sub_prefix(int* sub_count, int e, int E, int run) {
#pragma unroll
    for (int s2 = 0; s2 < kSubPerChunk; ++s2) {
        int v = sub_count[s2 * E + e];
        sub_count[s2 * E + e] = run;
        run += v;
    }
}

// FLAT: the intermediate table of the token-dropping construction: token_ids receives the flat entry n itself,
// expert_ids and row_of_slot are not written.
template <bool FLAT>
__device__ __forceinline__ void eri_write(const float* __restrict__ topk_w, int base, int B, int E, int k,
                                          const int* sub_count, const int (&my_e)[kSubPerChunk / 4],
                                          const int (&my_rank)[kSubPerChunk / 4], int32_t* __restrict__ token_ids,
                                          int32_t* __restrict__ expert_ids, float* __restrict__ combine_weights,
                                          int32_t* __restrict__ row_of_slot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < kSubPerChunk / 4; ++r) {
        const int sub = r * 4 + wave;
        const int n = base + sub * 64 + lane;
        const int e = my_e[r];
        if (n < B && (unsigned)e < (unsigned)E) {
            const int row = sub_count[sub * E + e] + my_rank[r];
            combine_weights[row] = topk_w[n];
            if (FLAT) {
                token_ids[row] = n;
            } else {
                token_ids[row] = n / k;
                expert_ids[row] = e;
                row_of_slot[n] = row;
            }
        }
    }
}

template <bool FLAT>
__global__ __launch_bounds__(256) void eri_scatter_kernel(const int32_t* __restrict__ topk_idx,
                                                          const float* __restrict__ topk_w, int B, int E, int k,
                                                          int ebits, const int32_t* __restrict__ chunk_prefix,
                                                          const int32_t* __restrict__ expert_offsets,
                                                          int32_t* __restrict__ token_ids,
                                                          int32_t* __restrict__ expert_ids,
                                                          float* __restrict__ combine_weights,
                                                          int32_t* __restrict__ row_of_slot) {
    // sub_count[s][e]: entries of expert e in sub-chunk s; turned into an exclusive prefix over s
    extern __shared__ int sub_count[];
    for (int i = threadIdx.x; i < kSubPerChunk * E; i += 256) sub_count[i] = 0;
    __syncthreads();
    const int base = blockIdx.x * kEriChunk;
    int my_e[kSubPerChunk / 4], my_rank[kSubPerChunk / 4];
    eri_rank(topk_idx, base, B, E, ebits, sub_count, my_e, my_rank);
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 256)
        eri_sub_prefix(sub_count, e, E, chunk_prefix[(size_t)blockIdx.x * E + e] + expert_offsets[e]);
    __syncthreads();
    eri_write<FLAT>(topk_w, base, B, E, k, sub_count, my_e, my_rank, token_ids, expert_ids, combine_weights,
                    row_of_slot);
}

// The whole construction in one launch: a block counts the experts of all flat entries, and of those in front of its
// chunk, by itself instead of taking them from two earlier launches, then ranks and writes its chunk as
// eri_scatter_kernel does.  Block 0 writes tokens_per_expert and expert_offsets.  Bound by launch latency where a call
// is small.  Measured (MI355X, replayed from a graph, three launches | one, us):
//     chunks            1             4             8            16       16, every entry on one expert
//     8 experts     8.0 | 5.4     8.8 | 6.4     9.0 | 7.4     9.2 | 9.2      9.0 | 8.9
//    64 experts     9.5 | 6.4    10.4 | 7.5    10.5 | 8.4    10.9 | 10.2    10.4 | 9.7
//   512 experts    15.7 | 8.1    17.0 | 9.4    17.6 | 10.8   18.0 | 12.8    17.3 | 11.7
// A chunk more costs every block 0.2 to 0.3 us, the three launches next to nothing: 8 experts break even at 16 chunks,
// and the line is drawn there.
// COPIES (from 5 chunks on): every expert has kEriCopies counters, chosen by the lane, so that a load that falls on few
// experts does not send a whole wave to one address (one counter each: 18.5, 19.1 and 20.8 us in the last column); up to
// 4 chunks adding them up costs more than it saves.
constexpr int kEriDirectChunks = 16;
constexpr int kEriPlainChunks = 4, kEriCopies = 4;

template <bool COPIES>
__global__ __launch_bounds__(256) void eri_direct_kernel(const int32_t* __restrict__ topk_idx,
                                                         const float* __restrict__ topk_w, int B, int E, int k,
                                                         int ebits, int32_t* __restrict__ tokens_per_expert,
                                                         int32_t* __restrict__ expert_offsets,
                                                         int32_t* __restrict__ token_ids,
                                                         int32_t* __restrict__ expert_ids,
                                                         float* __restrict__ combine_weights,
                                                         int32_t* __restrict__ row_of_slot) {
    extern __shared__ int sub_count[];             // as in eri_scatter_kernel
    __shared__ int total[XMOE_MAX_EXPERTS];        // entries of every expert, then their exclusive prefix
    __shared__ int before[XMOE_MAX_EXPERTS];       // those in front of this block's chunk
    __shared__ int total_c[COPIES ? XMOE_MAX_EXPERTS * kEriCopies : 1], before_c[COPIES ? XMOE_MAX_EXPERTS * kEriCopies : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kSubPerChunk * E; i += 256) sub_count[i] = 0;
    for (int i = threadIdx.x; i < XMOE_MAX_EXPERTS; i += 256) total[i] = before[i] = 0;
    if (COPIES)
        for (int i = threadIdx.x; i < kEriCopies * E; i += 256) total_c[i] = before_c[i] = 0;
    __syncthreads();
    const int base = blockIdx.x * kEriChunk;
    constexpr int kR = (COPIES ? 4 : 1) * kEriChunk / 256;   // entries per thread that are fetched together
    for (int n0 = 0; n0 < B; n0 += kR * 256) {
        int e[kR];
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            const int n = n0 + r * 256 + threadIdx.x;
            e[r] = topk_idx[n < B ? n : B - 1];
        }
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            const int n = n0 + r * 256 + threadIdx.x;
            if (n >= B || (unsigned)e[r] >= (unsigned)E) continue;
            const bool front = n0 + r * 256 < base;
            if (COPIES)
                atomicAdd((front ? before_c : total_c) + e[r] * kEriCopies + (lane & (kEriCopies - 1)), 1);
            else
                atomicAdd((front ? before : total) + e[r], 1);
        }
    }
    int my_e[kSubPerChunk / 4], my_rank[kSubPerChunk / 4];
    eri_rank(topk_idx, base, B, E, ebits, sub_count, my_e, my_rank);
    __syncthreads();
    if (COPIES) {
        for (int e = threadIdx.x; e < E; e += 256) {
            int a = 0, b = 0;
#pragma unroll
            for (int c = 0; c < kEriCopies; ++c) {
                a += total_c[e * kEriCopies + c];
                b += before_c[e * kEriCopies + c];
            }
            total[e] = a;
            before[e] = b;
        }
        __syncthreads();
    }
    // `total` holds the entries from the chunk on; one wave adds those in front and scans
    if (wave == 0) {
        constexpr int kPer = XMOE_MAX_EXPERTS / 64;
        int v[kPer], sum = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            v[j] = total[lane * kPer + j] + before[lane * kPer + j];
            sum += v[j];
        }
        int inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(inc, o, 64);
            if (lane >= o) inc += up;
        }
        int run = inc - sum;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int e = lane * kPer + j;
            total[e] = run;
            if (blockIdx.x == 0 && e < E) {
                tokens_per_expert[e] = v[j];
                expert_offsets[e] = run;
            }
            run += v[j];
        }
        if (blockIdx.x == 0 && lane == 63) expert_offsets[E] = run;   // experts from E on have no entries
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 256) eri_sub_prefix(sub_count, e, E, total[e] + before[e]);
    __syncthreads();
    eri_write<false>(topk_w, base, B, E, k, sub_count, my_e, my_rank, token_ids, expert_ids, combine_weights,
                     row_of_slot);
}

// ---------------------------------------------------------------------------------------------------------
// Token dropping (paper: Listing 1 PFT_construction() step 2; Appendix B.2): every expert keeps at most C rows, the
// ones with the largest combine weights, equal weights keeping the lower flat entry first.  Input is the dropless
// table (rows sorted by expert, ascending flat entry inside an expert): so "lower flat entry" is "earlier row", and
// the survivors, taken in row order, are already in their final order.
// Block e < E handles expert e: a three-pass radix select over the order-preserving bit pattern of the weights
// finds the C-th largest weight, then the segment is compacted in row order.  Blocks >= E write the sentinels of
// the rows behind the last retained one.  No floating-point arithmetic takes part in the decision.
//
// Bound: one CU per expert, and the fullest expert's block is the launch: latency of its loads, its barriers, and the LDS
// atomics of the first pass, whose bins (sign, exponent, two bits) the weights of a softmax share.  So 16 waves, a window
// of 8192 rows with eight loads in flight per thread (a segment that fits one is read once for the three passes), four
// copies of the histogram, and one barrier per window of the compaction: a row's place is the number of heavier rows in
// front of it plus the number of equal ones, as far as they are kept, so both prefixes come from the same ballots.
// T 8192, E 64, k 6, C 960, Zipf-like load: 256 threads, a row each per step | this: 62 | 16 us.
// ---------------------------------------------------------------------------------------------------------
constexpr int kCapThreads = 1024, kCapWaves = kCapThreads / 64;
constexpr int kCapRows = 8;                              // rows per thread and window
constexpr int kCapWindow = kCapThreads * kCapRows;
constexpr int kCapCopies = 4;
__device__ __forceinline__ uint32_t weight_key(float w) {
    uint32_t u = __float_as_uint(w);
    if (u == 0x80000000u) u = 0u;                          // -0.0 ties with +0.0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);   // ascending in w
}

// exclusive prefix of `v` over the block's threads in thread order; total in *total
__device__ __forceinline__ int block_excl_sum(int v, int* wave_tot, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(inc, o, 64);
        if (lane >= o) inc += up;
    }
    __syncthreads();   // wave_tot may still be read from the previous call
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kCapWaves; ++w) {
        const int t = wave_tot[w];
        before += w < wave ? t : 0;
        all += t;
    }
    *total = all;
    return before + inc - v;
}

__global__ __launch_bounds__(kCapThreads) void eri_cap_kernel(const int32_t* __restrict__ off0,      // dropless offsets [E+1]
                                                      const int32_t* __restrict__ flat0,     // flat entry of row [B]
                                                      const float* __restrict__ w0,          // weight of row [B]
                                                      int B, int E, int k, int C,
                                                      int32_t* __restrict__ tokens_per_expert,
                                                      int32_t* __restrict__ expert_offsets,
                                                      int32_t* __restrict__ token_ids,
                                                      int32_t* __restrict__ expert_ids,
                                                      float* __restrict__ combine_weights,
                                                      int32_t* __restrict__ row_of_slot) {
    __shared__ int4 hist[2048];               // one int per copy
    static_assert(kCapCopies == 4, "");
    __shared__ int wave_tot[kCapWaves];
    __shared__ int2 wave_cnt[2][kCapWaves];   // heavier, equal rows of a wave's part of the window
    __shared__ uint32_t s_prefix, s_mask;
    __shared__ int s_remaining, s_new_lo, s_kept_total;
    const int tid = threadIdx.x;
    // retained rows before this block's expert, and in total: every block recomputes the short prefix it needs
    {
        int before_me = 0, all = 0;
        for (int i = tid; i < E; i += kCapThreads) {
            const int n = off0[i + 1] - off0[i];
            const int c = n < C ? n : C;
            all += c;
            if (i < (int)blockIdx.x) before_me += c;
        }
        int tot_before, tot_all;
        block_excl_sum(before_me, wave_tot, &tot_before);
        block_excl_sum(all, wave_tot, &tot_all);
        if (tid == 0) {
            s_new_lo = tot_before;
            s_kept_total = tot_all;
        }
    }
    __syncthreads();
    const int kept_total = s_kept_total;
    if ((int)blockIdx.x >= E) {
        // rows behind the last retained one
        const int base = ((int)blockIdx.x - E) * kEriChunk;
        for (int r = base + tid; r < base + kEriChunk && r < B; r += kCapThreads) {
            if (r >= kept_total) {
                token_ids[r] = -1;
                expert_ids[r] = E;
                combine_weights[r] = 0.0f;
            }
        }
        return;
    }
    const int e = blockIdx.x;
    const int lo = off0[e], n = off0[e + 1] - lo;
    const int new_lo = s_new_lo;
    const int keep_n = n < C ? n : C;
    if (tid == 0) {
        tokens_per_expert[e] = keep_n;
        expert_offsets[e] = new_lo;
        if (e == E - 1) expert_offsets[E] = kept_total;
    }
    // Row r of a thread's kCapRows of the window at `base`: a wave's 64 lanes hold consecutive rows, a wave the next
    // kCapRows groups of 64, so that ballots and the waves' totals give prefixes in row order
    const int lane = tid & 63, wave = tid >> 6;
    uint32_t key[kCapRows];
    float w[kCapRows];
    const uint32_t un = (uint32_t)n;   // unsigned: the last window may reach past 2^31
    auto row_at = [&](uint32_t base, int r) { return base + (wave * kCapRows + r) * 64 + lane; };
    auto load = [&](uint32_t base) {
#pragma unroll
        for (int r = 0; r < kCapRows; ++r) {
            const uint32_t i = row_at(base, r);
            w[r] = w0[lo + (i < un ? i : 0)];
        }
#pragma unroll
        for (int r = 0; r < kCapRows; ++r) key[r] = weight_key(w[r]);
    };
    if (n == 0) return;   // the same for the whole block
    load(0);
    // the C-th largest key of the segment (only needed when something is dropped)
    uint32_t vstar = 0;
    int need_eq = 0;   // how many rows with key == vstar are kept
    const bool select = n > C && C > 0;
    if (select) {
        if (tid == 0) {
            s_prefix = 0;
            s_mask = 0;
            s_remaining = C;
        }
        const int shifts[3] = {21, 10, 0}, widths[3] = {11, 11, 10};
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const int shift = shifts[p], nb = 1 << widths[p];
            for (int i = tid; i < nb; i += kCapThreads) hist[i] = make_int4(0, 0, 0, 0);
            __syncthreads();
            const uint32_t prefix = s_prefix, mask = s_mask;
            for (uint32_t base = 0; base < un; base += kCapWindow) {
                if (n > kCapWindow) load(base);
#pragma unroll
                for (int r = 0; r < kCapRows; ++r)
                    if (row_at(base, r) < un && (key[r] & mask) == prefix)
                        atomicAdd(reinterpret_cast<int*>(&hist[(key[r] >> shift) & (nb - 1)]) + (tid & (kCapCopies - 1)), 1);
            }
            __syncthreads();
            // which bin holds the `remaining`-th largest key: thread t owns the bins nb-1 - t*bpt .. (downwards);
            // an exclusive prefix of the threads' sums, then the one thread whose range the target falls into
            // walks its few bins
            {
                const int bpt = nb / kCapThreads;
                const int hi = nb - 1 - tid * bpt;
                auto bin = [&](int i) {
                    const int4 h = hist[i];
                    return (h.x + h.y) + (h.z + h.w);
                };
                int mine = 0;
                for (int j = 0; j < bpt; ++j) mine += bin(hi - j);
                int tot_unused;
                const int before = block_excl_sum(mine, wave_tot, &tot_unused);
                const int remaining = s_remaining;
                __syncthreads();   // everyone has read s_remaining before the owner overwrites it
                if (before < remaining && remaining <= before + mine) {
                    int rem = remaining - before, b = hi;
                    while (bin(b) < rem) {
                        rem -= bin(b);
                        --b;
                    }
                    s_remaining = rem;
                    s_prefix = prefix | ((uint32_t)b << shift);
                    s_mask = mask | ((uint32_t)(nb - 1) << shift);
                }
            }
            __syncthreads();
        }
        vstar = s_prefix;
        need_eq = s_remaining;
    }
    // compaction in row order: rows heavier than vstar stay, and the first need_eq of those equal to it
    int gt_seen = 0, eq_seen = 0;
    for (uint32_t base = 0; base < un; base += kCapWindow) {
        if (n > kCapWindow) load(base);
        int flat[kCapRows];
#pragma unroll
        for (int r = 0; r < kCapRows; ++r) {
            const uint32_t i = row_at(base, r);
            flat[r] = flat0[lo + (i < un ? i : 0)];
        }
        unsigned long long gt[kCapRows], eq[kCapRows];
        int2 mine = make_int2(0, 0);
#pragma unroll
        for (int r = 0; r < kCapRows; ++r) {
            const bool in = row_at(base, r) < un;
            gt[r] = __ballot(in && (n <= C || (select && key[r] > vstar)));
            eq[r] = __ballot(in && select && key[r] == vstar);
            mine.x += __popcll(gt[r]);
            mine.y += __popcll(eq[r]);
        }
        // two sets of totals: one is written while slower waves still read the other
        int2* cnt = wave_cnt[(base / kCapWindow) & 1];
        if (lane == 0) cnt[wave] = mine;
        __syncthreads();
        int g = gt_seen, q = eq_seen;
#pragma unroll
        for (int v = 0; v < kCapWaves; ++v) {
            const int2 t = cnt[v];
            g += v < wave ? t.x : 0;
            q += v < wave ? t.y : 0;
            gt_seen += t.x;
            eq_seen += t.y;
        }
#pragma unroll
        for (int r = 0; r < kCapRows; ++r) {
            const unsigned long long below = (1ull << lane) - 1ull;
            const int g_at = g + __popcll(gt[r] & below), q_at = q + __popcll(eq[r] & below);
            const bool is_eq = (eq[r] >> lane) & 1ull;
            const bool keep = ((gt[r] >> lane) & 1ull) || (is_eq && q_at < need_eq);
            g += __popcll(gt[r]);
            q += __popcll(eq[r]);
            if (row_at(base, r) >= un) continue;
            if (keep) {
                const int row = new_lo + g_at + (q_at < need_eq ? q_at : need_eq);
                token_ids[row] = flat[r] / k;
                expert_ids[row] = e;
                combine_weights[row] = w[r];
                row_of_slot[flat[r]] = row;
            } else {
                row_of_slot[flat[r]] = -1;
            }
        }
    }
}

}  // namespace xmoe

using namespace xmoe;

// the three launches of the dropless construction; counts: eri_num_chunks(B) * E ints of scratch (every one of them is
// written by the histogram kernel before it is read, so the memory needs no clearing)
static int build_eri_launch(const int32_t* topk_idx, const float* topk_w, int T, int E, int k,
                            int32_t* tokens_per_expert, int32_t* expert_offsets, int32_t* token_ids,
                            int32_t* expert_ids, float* combine_weights, int32_t* row_of_slot, int32_t* counts,
                            hipStream_t s) {
    const int B = T * k;
    const int nchunks = eri_num_chunks(B);
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    if (nchunks > 0 && nchunks <= kEriDirectChunks) {
#define XMOE_CALL(COPIES)                                                                                             \
    XMOE_LAUNCH(K_ERI_DIRECT, s,                                                                                      \
                hipLaunchKernelGGL(eri_direct_kernel<COPIES>, dim3(nchunks), dim3(256),                               \
                                   (size_t)kSubPerChunk * E * sizeof(int), s, topk_idx, topk_w, B, E, k, ebits,       \
                                   tokens_per_expert, expert_offsets, token_ids, expert_ids, combine_weights,         \
                                   row_of_slot))
        if (nchunks <= kEriPlainChunks)
            XMOE_CALL(false);
        else
            XMOE_CALL(true);
#undef XMOE_CALL
        return XMOE_OK;
    }
    if (nchunks > 0)
        XMOE_LAUNCH(K_ERI_HIST, s,
                    hipLaunchKernelGGL(eri_hist_kernel, dim3(nchunks), dim3(256), 0, s, topk_idx, B, E, counts));
    XMOE_LAUNCH(K_ERI_SCAN, s,
                hipLaunchKernelGGL(eri_scan_kernel, dim3(1), dim3(512), 0, s, counts, nchunks, E, tokens_per_expert,
                                   expert_offsets));
    if (nchunks > 0)
        XMOE_LAUNCH(K_ERI_SCATTER, s,
                    hipLaunchKernelGGL(eri_scatter_kernel<false>, dim3(nchunks), dim3(256),
                                       (size_t)kSubPerChunk * E * sizeof(int), s, topk_idx, topk_w, B, E, k, ebits,
                                       counts, expert_offsets, token_ids, expert_ids, combine_weights, row_of_slot));
    return XMOE_OK;
}

static int build_eri_check(const int32_t* topk_idx, const float* topk_w, int T, int E, int k,
                           int32_t* tokens_per_expert, int32_t* expert_offsets, int32_t* token_ids,
                           int32_t* expert_ids, float* combine_weights, int32_t* row_of_slot) {
    if (T < 0 || E < 1 || k < 1 || k > E) return XMOE_ERR_INVALID_ARG;
    if (E > XMOE_MAX_EXPERTS) return XMOE_ERR_UNSUPPORTED;
    if ((long long)T * k >= (1ll << 31)) return XMOE_ERR_INVALID_ARG;
    if (!tokens_per_expert || !expert_offsets) return XMOE_ERR_INVALID_ARG;
    if (T > 0 && (!topk_idx || !topk_w || !token_ids || !expert_ids || !combine_weights || !row_of_slot))
        return XMOE_ERR_INVALID_ARG;
    return XMOE_OK;
}

extern "C" int xmoe_build_eri(const int32_t* topk_idx, const float* topk_w, int T, int E, int k,
                              int32_t* tokens_per_expert, int32_t* expert_offsets, int32_t* token_ids,
                              int32_t* expert_ids, float* combine_weights, int32_t* row_of_slot, void* ws,
                              size_t ws_bytes, void* stream) {
    const int st = build_eri_check(topk_idx, topk_w, T, E, k, tokens_per_expert, expert_offsets, token_ids, expert_ids,
                                   combine_weights, row_of_slot);
    if (st != XMOE_OK) return st;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) || ws_bytes < eri_ws_bytes(T, E, k)) return XMOE_ERR_WORKSPACE;
    return build_eri_launch(topk_idx, topk_w, T, E, k, tokens_per_expert, expert_offsets, token_ids, expert_ids,
                            combine_weights, row_of_slot, (int32_t*)ws, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------------------------
// xmoe_build_eri for callers that cannot allocate: the chunk histograms live in a static device array instead of a
// caller-provided workspace.  Every device holds its own copy of the array at its own address, looked up once per
// device (hipGetSymbolAddress with that device current); host code only ever uses that address.
// ---------------------------------------------------------------------------------------------------------
static __device__ __align__(256) int32_t scratch[XMOE_STATIC_ERI_SCRATCH_BYTES / sizeof(int32_t)];

namespace {
constexpr int kMaxScratchDevices = 64;
int32_t* g_scratch_ptr[kMaxScratchDevices];   // device address of `scratch` on device i, or NULL before the first call there

int scratch_for_current_device(int32_t** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return XMOE_ERR_HIP;
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return XMOE_ERR_HIP;
        g_scratch_ptr[dev] = static_cast<int32_t*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return XMOE_OK;
}
}  // namespace

extern "C" int xmoe_build_eri_static(const int32_t* topk_idx, const float* topk_w, int T, int E, int k,
                                     int32_t* tokens_per_expert, int32_t* expert_offsets, int32_t* token_ids,
                                     int32_t* expert_ids, float* combine_weights, int32_t* row_of_slot,
                                     void* stream) {
    const int st = build_eri_check(topk_idx, topk_w, T, E, k, tokens_per_expert, expert_offsets, token_ids, expert_ids,
                                   combine_weights, row_of_slot);
    if (st != XMOE_OK) return st;
    if (eri_ws_bytes(T, E, k) > (size_t)XMOE_STATIC_ERI_SCRATCH_BYTES) return XMOE_ERR_WORKSPACE;
    int32_t* counts = nullptr;
    const int sp = scratch_for_current_device(&counts);
    if (sp != XMOE_OK) return sp;
    return build_eri_launch(topk_idx, topk_w, T, E, k, tokens_per_expert, expert_offsets, token_ids, expert_ids,
                            combine_weights, row_of_slot, counts, (hipStream_t)stream);
}

// Segments of n all-token experts directly behind the PFT's last row, which only the device knows after token
// dropping: offsets[E + 1 + s] = offsets[E] + (s+1)*T, and for the rows of those segments token id t and weight 1.
__global__ __launch_bounds__(256) void shared_segments_kernel(int32_t* __restrict__ offsets,
                                                              int32_t* __restrict__ token_ids,
                                                              float* __restrict__ combine_weights, int T, int E,
                                                              int n) {
    const int base = offsets[E];
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < (long)n * T) {
        token_ids[base + i] = (int)(i % T);
        combine_weights[base + i] = 1.0f;
    }
    if (i < n) offsets[E + 1 + i] = base + ((int)i + 1) * T;
}

extern "C" int xmoe_append_shared_segments(int32_t* expert_offsets, int32_t* token_ids, float* combine_weights, int T,
                                           int E, int n_shared, void* stream) {
    if (T < 0 || E < 1 || n_shared < 0) return XMOE_ERR_INVALID_ARG;
    if ((long long)T * n_shared >= (1ll << 31)) return XMOE_ERR_INVALID_ARG;
    if (n_shared == 0) return XMOE_OK;
    if (!expert_offsets || (T > 0 && (!token_ids || !combine_weights))) return XMOE_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    const long n = (long)n_shared * T > n_shared ? (long)n_shared * T : n_shared;
    XMOE_LAUNCH(K_SHARED_SEGMENTS, s,
                hipLaunchKernelGGL(shared_segments_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                                   expert_offsets, token_ids, combine_weights, T, E, n_shared));
    return XMOE_OK;
}

extern "C" int xmoe_build_eri_capped(const int32_t* topk_idx, const float* topk_w, int T, int E, int k,
                                     int max_token_count, int32_t* tokens_per_expert, int32_t* expert_offsets,
                                     int32_t* token_ids, int32_t* expert_ids, float* combine_weights,
                                     int32_t* row_of_slot, void* ws, size_t ws_bytes, void* stream) {
    if (T < 0 || E < 1 || k < 1 || k > E || max_token_count < 0) return XMOE_ERR_INVALID_ARG;
    if (E > XMOE_MAX_EXPERTS) return XMOE_ERR_UNSUPPORTED;
    if ((long long)T * k >= (1ll << 31)) return XMOE_ERR_INVALID_ARG;
    if (!tokens_per_expert || !expert_offsets) return XMOE_ERR_INVALID_ARG;
    if (T > 0 && (!topk_idx || !topk_w || !token_ids || !expert_ids || !combine_weights || !row_of_slot))
        return XMOE_ERR_INVALID_ARG;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) || ws_bytes < eri_capped_ws_bytes(T, E, k))
        return XMOE_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    const int B = T * k;
    const int nchunks = eri_num_chunks(B);
    // workspace: chunk histograms | dropless offsets [E+1] | dropless counts [E] | flat entry of row [B] | weight of row [B]
    char* p = (char*)ws;
    int32_t* counts = (int32_t*)p;
    p += eri_ws_bytes(T, E, k);
    int32_t* off0 = (int32_t*)p;
    p += align_up((size_t)(E + 1) * sizeof(int32_t), 256);
    int32_t* tpe0 = (int32_t*)p;
    p += align_up((size_t)E * sizeof(int32_t), 256);
    int32_t* flat0 = (int32_t*)p;
    p += align_up((size_t)(B > 0 ? B : 1) * sizeof(int32_t), 256);
    float* w0 = (float*)p;
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    if (nchunks > 0)
        XMOE_LAUNCH(K_ERI_HIST, s,
                    hipLaunchKernelGGL(eri_hist_kernel, dim3(nchunks), dim3(256), 0, s, topk_idx, B, E, counts));
    XMOE_LAUNCH(K_ERI_SCAN, s,
                hipLaunchKernelGGL(eri_scan_kernel, dim3(1), dim3(512), 0, s, counts, nchunks, E, tpe0, off0));
    if (nchunks > 0)
        XMOE_LAUNCH(K_ERI_SCATTER, s,
                    hipLaunchKernelGGL(eri_scatter_kernel<true>, dim3(nchunks), dim3(256),
                                       (size_t)kSubPerChunk * E * sizeof(int), s, topk_idx, topk_w, B, E, k, ebits,
                                       counts, off0, flat0, nullptr, w0, nullptr));
    XMOE_LAUNCH(K_ERI_CAP, s,
                hipLaunchKernelGGL(eri_cap_kernel, dim3(E + nchunks), dim3(kCapThreads), 0, s, off0, flat0, w0, B, E, k,
                                   max_token_count, tokens_per_expert, expert_offsets, token_ids, expert_ids,
                                   combine_weights, row_of_slot));
    return XMOE_OK;
}
