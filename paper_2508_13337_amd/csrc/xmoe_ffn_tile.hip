// Expert MLP over ragged segments (paper: Listing 1 mlp(); Appendix B.4 "Sequential GeMM"), general version: serves
// float32 workloads and every bf16 shape the direct-to-LDS kernels (256 x 256, 128 x 128) do not take, on the tiles of
// xmoe_tile_gemm.h.
// One launch covers every expert: a tile map built on the device says which expert and which rows each row tile
// belongs to, so there is no host round trip on tokens_per_expert and no per-expert launch.
//
// Measured (MI355X, one training step of the layer, row tiles numbered down the segments -> runs of neighbouring tiles per
// XCD; float32: with the float32 matrix instruction -> as three bf16 parts as well):
//   float32 T 2048 d 1024 f 704, 16 experts + 1 shared, k 4:   1613 -> 1108 us, the products at 85 to 147 TFLOP/s
//   bf16    T 3001 d 1000 f 712, 24 experts + 1 shared, k 3:    627 ->  558 us (417 on the 128 x 128 direct tiles)
#include "xmoe_ffn.h"
#include "xmoe_tile_gemm.h"

namespace xmoe {

// ---------------------------------------------------------------------------------------------------------
// tile map: header {total tiles, 0, 0, 0} then (expert, first row) per row tile; unused entries have expert -1.
// sched: the experts sorted by descending row count (ties: lower index first; RANK, for the weight gradients, which hand out
// their tiles longest first), then kSchedCounters zeroed counters.
// Latency: one block.  From 65 experts on the running tile count is a scan over the block (one thread's walk over E counts
// is 30 ns per expert) and an expert's rank is counted by several threads: E 257 14.4 -> 4.8 us, with the ranks 9.2.
// ---------------------------------------------------------------------------------------------------------
template <bool RANK>
__global__ __launch_bounds__(1024) void tile_map_kernel(const int32_t* __restrict__ off, int E, int tile_rows,
                                                       int max_tiles, int32_t* __restrict__ map,
                                                       int32_t* __restrict__ sched) {
    __shared__ int start[XMOE_MAX_EXPERTS + 1];
    __shared__ __align__(16) int count[XMOE_MAX_EXPERTS];
    __shared__ int wave_sum[16];
    const int e = threadIdx.x;
    int nt = 0, lo = 0, m = 0;
    if (e < E) {
        lo = off[e];
        m = off[e + 1] - lo;
        nt = m > 0 ? (m + tile_rows - 1) / tile_rows : 0;
    }
    if (e < XMOE_MAX_EXPERTS) count[e] = e < E ? m : -1;   // (the block has at least as many threads)
    if (threadIdx.x < kSchedCounters) sched[E + threadIdx.x] = 0;
    int first = 0, all = 0;   // tiles before this thread's expert, of all experts
    if (E <= 64) {
        start[e < E ? e : XMOE_MAX_EXPERTS] = nt;
        __syncthreads();
        if (threadIdx.x == 0) {
            int run = 0;
            for (int i = 0; i < E; ++i) {
                const int v = start[i];
                start[i] = run;
                run += v;
            }
            wave_sum[0] = run;
        }
        __syncthreads();
        first = e < E ? start[e] : 0;
        all = wave_sum[0];
    } else {
        int v = nt;
#pragma unroll
        for (int w = 1; w < 64; w *= 2) {
            const int o = __shfl_up(v, w, 64);
            if ((int)(threadIdx.x & 63) >= w) v += o;
        }
        if ((threadIdx.x & 63) == 63) wave_sum[threadIdx.x >> 6] = v;
        __syncthreads();
        first = v - nt;
#pragma unroll
        for (int w = 0; w < 8; ++w) {   // experts belong to the first 512 threads
            if (w < (int)(threadIdx.x >> 6)) first += wave_sum[w];
            all += wave_sum[w];
        }
    }
    const int total = all < max_tiles ? all : max_tiles;
    if (threadIdx.x == 0) {
        map[0] = total;
        map[1] = map[2] = map[3] = 0;
    }
    if (e < E) {
        for (int i = 0; i < nt; ++i) {
            const int ti = first + i;
            if (ti < max_tiles) {
                map[4 + 2 * ti] = e;
                map[4 + 2 * ti + 1] = lo + i * tile_rows;
            }
        }
    }
    for (int ti = total + threadIdx.x; ti < max_tiles; ti += blockDim.x) {
        map[4 + 2 * ti] = -1;
        map[4 + 2 * ti + 1] = 0;
    }
    if (RANK) {
        // P neighbouring threads count for one expert, four counts at a time
        const int P = E <= 64 ? 8 : E <= 128 ? 4 : 2;
        const int x = threadIdx.x / P, q = threadIdx.x % P;
        int rank = 0;
        if (x < E) {
            const int mine = count[x];
#pragma unroll 2
            for (int i = 4 * q; i < E; i += 4 * P) {
                const int4 c = *reinterpret_cast<const int4*>(count + i);
                // ahead of this expert: longer ones, and among equals those with a lower index
                rank += (c.x >= mine + (i < x ? 0 : 1)) + (c.y >= mine + (i + 1 < x ? 0 : 1)) +
                        (c.z >= mine + (i + 2 < x ? 0 : 1)) + (c.w >= mine + (i + 3 < x ? 0 : 1));
            }
        }
        for (int w = 1; w < P; w *= 2) rank += __shfl_xor(rank, w, 64);
        if (x < E && q == 0) sched[rank] = x;
    }
}

int launch_tile_map(const int32_t* off, int E, int tile_rows, int max_tiles, int32_t* map, int32_t* sched, bool rank,
                    hipStream_t s) {
    const int threads = E <= 256 ? 512 : 1024;   // two per expert to count ranks
    if (rank)
        XMOE_LAUNCH(K_TILE_MAP, s, hipLaunchKernelGGL(tile_map_kernel<true>, dim3(1), dim3(threads), 0, s, off, E, tile_rows,
                                                      max_tiles, map, sched));
    else
        XMOE_LAUNCH(K_TILE_MAP, s, hipLaunchKernelGGL(tile_map_kernel<false>, dim3(1), dim3(512), 0, s, off, E, tile_rows,
                                                      max_tiles, map, sched));
    return XMOE_OK;
}

// row_grad[i] = sum_p row_part[p * B + i], p ascending, eight loads at a time in flight (B 65536, 24 parts: 12.2 -> 5.1 us)
__global__ __launch_bounds__(64) void row_grad_reduce_kernel(const float* __restrict__ row_part, int parts, int B,
                                                             float* __restrict__ row_grad) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (i >= B) return;
    float s = 0.f;
    int p = 0;
    for (; p + 8 <= parts; p += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = row_part[(size_t)(p + q) * B + i];
#pragma unroll
        for (int q = 0; q < 8; ++q) s += v[q];
    }
    for (; p < parts; ++p) s += row_part[(size_t)p * B + i];
    row_grad[i] = s;
}

int launch_row_grad_reduce(const float* row_part, int parts, int B, float* row_grad, hipStream_t s) {
    if (B <= 0) return XMOE_OK;
    XMOE_LAUNCH(K_ROW_GRAD_REDUCE, s,
                hipLaunchKernelGGL(row_grad_reduce_kernel, dim3((B + 63) / 64), dim3(64), 0, s, row_part, parts, B,
                                   row_grad));
    return XMOE_OK;
}

#define XMOE_TILE_BOUNDS __launch_bounds__(TileShape<BIG>::kThreads, 2)

// ---------------------------------------------------------------------------------------------------------
// forward 1: G = Xd Wg, U = Xd Wu, A = silu(G) * U          rows: ragged, K = d, N = f
// A block computes the same kN/2 columns of G and of U, so the rows are fetched once for both and A needs no exchange.
// ---------------------------------------------------------------------------------------------------------
template <typename T, bool BIG>
__global__ XMOE_TILE_BOUNDS void ffn_gateup_mfma_kernel(const T* __restrict__ xd,
                                                        const int32_t* __restrict__ row_index,   // or NULL
                                                        const int32_t* __restrict__ off,
                                                        const int32_t* __restrict__ map, int d, int f,
                                                        const T* __restrict__ wg, const T* __restrict__ wu,
                                                        T* __restrict__ G, T* __restrict__ U, T* __restrict__ A) {
    using S = TileShape<BIG>;
    __shared__ __align__(16) char smem[S::kLds];
    RowTile t;
    if (!t.init(off, map, (f + S::kN / 2 - 1) / (S::kN / 2), S::kM)) return;
    const int n0 = t.col * (S::kN / 2);
    RowSrc<T, S::kThreads> a;
    ColSrc<T, S::kThreads, false> b;
    a.init(row_index ? xd : xd + (size_t)t.row0 * d, d, t.rows, row_index ? row_index + t.row0 : nullptr);
    b.init(wg + (size_t)t.e * d * f + n0, wu + (size_t)t.e * d * f + n0, f, f - n0, nullptr, d);
    tile_f32x16_t acc[S::kMI][2];
    tile_zero<BIG>(acc);
    tile_mainloop<T, BIG, true, false>(acc, d, t.rows, f - n0, a, b, smem);
    if constexpr (std::is_same<T, float>::value)
        tile_finish<BIG, true>(acc, d, 1, [&](int, int ni) {
            return PlainPair{{row_index ? xd : xd + (size_t)t.row0 * d, (size_t)d, 1, row_index ? row_index + t.row0 : nullptr, nullptr, t.rows},
                             {(ni ? wu : wg) + (size_t)t.e * d * f + n0, 1, (size_t)f, nullptr, nullptr, f - n0}};
        });
    const int n = n0 + tile_col<BIG, true>(0);
    if (n >= f) return;
#pragma unroll
    for (int mi = 0; mi < S::kMI; ++mi)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = tile_row<BIG>(mi, v);
            if (r < t.rows) {
                const size_t ix = (size_t)(t.row0 + r) * f + n;
                const float g = acc[mi][0][v], u = acc[mi][1][v];
                G[ix] = from_float<T>(g);
                U[ix] = from_float<T>(u);
                A[ix] = from_float<T>(siluf_(g) * u);
            }
        }
}

// stores a block's tile: C[(row0 + r) * ld + n] for r < rows, n < N
template <typename T, bool BIG>
__device__ __forceinline__ void tile_store(const tile_f32x16_t (&acc)[TileShape<BIG>::kMI][2], T* __restrict__ C,
                                           size_t ld, int rows, int cols) {
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
        const int n = tile_col<BIG, false>(ni);
        if (n >= cols) continue;
#pragma unroll
        for (int mi = 0; mi < TileShape<BIG>::kMI; ++mi)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = tile_row<BIG>(mi, v);
                if (r < rows) C[(size_t)r * ld + n] = from_float<T>(acc[mi][ni][v]);
            }
    }
}

// ---------------------------------------------------------------------------------------------------------
// forward 2: Y = A Wd                                       rows: ragged, K = f, N = d
// ---------------------------------------------------------------------------------------------------------
template <typename T, bool BIG>
__global__ XMOE_TILE_BOUNDS void ffn_down_mfma_kernel(const T* __restrict__ A, const int32_t* __restrict__ off,
                                                      const int32_t* __restrict__ map, int d, int f,
                                                      const T* __restrict__ wd, T* __restrict__ Y) {
    using S = TileShape<BIG>;
    __shared__ __align__(16) char smem[S::kLds];
    RowTile t;
    if (!t.init(off, map, (d + S::kN - 1) / S::kN, S::kM)) return;
    const int n0 = t.col * S::kN;
    RowSrc<T, S::kThreads> a;
    ColSrc<T, S::kThreads, false> b;
    a.init(A + (size_t)t.row0 * f, f, t.rows, nullptr);
    b.init(wd + (size_t)t.e * f * d + n0, nullptr, d, d - n0, nullptr, f);
    tile_f32x16_t acc[S::kMI][2];
    tile_zero<BIG>(acc);
    tile_mainloop<T, BIG, false, false>(acc, f, t.rows, d - n0, a, b, smem);
    if constexpr (std::is_same<T, float>::value)
        tile_finish<BIG, false>(acc, f, 1, [&](int, int) {
            return PlainPair{{A + (size_t)t.row0 * f, (size_t)f, 1, nullptr, nullptr, t.rows},
                             {wd + (size_t)t.e * f * d + n0, 1, (size_t)d, nullptr, nullptr, d - n0}};
        });
    tile_store<T, BIG>(acc, Y + (size_t)t.row0 * d + n0, d, t.rows, d - n0);
}

// ---------------------------------------------------------------------------------------------------------
// backward 1: dA = dY W^T (W = Wd or W2), K = d, N = f; row r of dY is dy_scale[r] * dY[dy_index[r]], the scale follows
// in the epilogue.  EPI(i, ix, da, sc): the element ix of the [B,f] arrays from the unscaled da; it returns this
// element's share of <unscaled dY row, Y row>, whose sum over the wave's 64 columns goes to row_part (one part per
// 64 columns).
// ---------------------------------------------------------------------------------------------------------
template <typename T, bool BIG, class Prefetch, class Epi>
__device__ __forceinline__ void dact_tile(const T* __restrict__ dY, const int32_t* __restrict__ dy_index,
                                          const float* __restrict__ dy_scale, const int32_t* __restrict__ off,
                                          const int32_t* __restrict__ map, int d, int f, const T* __restrict__ w,
                                          float* __restrict__ row_part, int B, Prefetch prefetch, Epi epi) {
    using S = TileShape<BIG>;
    __shared__ __align__(16) char smem[S::kLds];
    RowTile t;
    if (!t.init(off, map, (f + S::kN - 1) / S::kN, S::kM)) return;
    const int n0 = t.col * S::kN;
    RowSrc<T, S::kThreads> a, b;
    a.init(dy_index ? dY : dY + (size_t)t.row0 * d, d, t.rows, dy_index ? dy_index + t.row0 : nullptr);
    b.init(w + ((size_t)t.e * f + n0) * d, d, f - n0, nullptr);
    tile_f32x16_t acc[S::kMI][2];
    tile_zero<BIG>(acc);
    tile_mainloop<T, BIG, false, false>(acc, d, t.rows, f - n0, a, b, smem);
    if constexpr (std::is_same<T, float>::value)
        tile_finish<BIG, false>(acc, d, 1, [&](int, int) {
            return PlainPair{{dy_index ? dY : dY + (size_t)t.row0 * d, (size_t)d, 1, dy_index ? dy_index + t.row0 : nullptr, nullptr, t.rows},
                             {w + ((size_t)t.e * f + n0) * d, (size_t)d, 1, nullptr, nullptr, f - n0}};
        });
    const bool scaled = dy_index && dy_scale;
#pragma unroll
    for (int mi = 0; mi < S::kMI; ++mi) {
        float part[16], sc[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            part[v] = 0.f;
            const int r = tile_row<BIG>(mi, v);
            sc[v] = scaled ? dy_scale[t.row0 + (r < t.rows ? r : t.rows - 1)] : 1.0f;
        }
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            const int n = n0 + tile_col<BIG, false>(ni);
            const int nc = n < f ? n : f - 1;
            // the 16 elements' inputs in one batch, at clamped addresses: no branch stands between the loads
            float in0[16], in1[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = tile_row<BIG>(mi, v);
                prefetch((size_t)(t.row0 + (r < t.rows ? r : t.rows - 1)) * f + nc, in0[v], in1[v]);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = tile_row<BIG>(mi, v);
                if (r < t.rows && n < f)
                    part[v] += epi((size_t)(t.row0 + r) * f + n, acc[mi][ni][v], sc[v], in0[v], in1[v]);
            }
        }
        const float sum = tile_sum_over_cols(part);
        const int lane = threadIdx.x & 63;
        // the lane's v is not a compile-time constant here
        const int r = tile_row<BIG>(mi, 0) + 8 * (((lane >> 1) & 15) >> 2) + (((lane >> 1) & 15) & 3);
        const int p = t.col * (S::kN / 64) + tile_col_base<BIG, false>(0) / 64;
        if (!(lane & 1) && r < t.rows && p * 64 < f) row_part[(size_t)p * B + t.row0 + r] = sum;
    }
}

// dG = dA * U * silu'(G), dU = dA * silu(G), A = silu(G) * U
template <typename T, bool BIG>
__global__ XMOE_TILE_BOUNDS void ffn_dact_mfma_kernel(const T* __restrict__ dY,
                                                      const int32_t* __restrict__ dy_index,   // or NULL
                                                      const float* __restrict__ dy_scale,     // or NULL
                                                      const int32_t* __restrict__ off,
                                                      const int32_t* __restrict__ map, int d, int f,
                                                      const T* __restrict__ wd, const T* __restrict__ G,
                                                      const T* __restrict__ U, T* __restrict__ dG,
                                                      T* __restrict__ dU, T* __restrict__ A,
                                                      float* __restrict__ row_part, int B) {
    dact_tile<T, BIG>(
        dY, dy_index, dy_scale, off, map, d, f, wd, row_part, B,
        [&](size_t ix, float& g, float& u) { g = to_float(G[ix]); u = to_float(U[ix]); },
        [&](size_t ix, float da0, float sc, float g, float u) {
            const float da = da0 * sc;
            const float sg = sigmoidf_(g);
            const float sl = g * sg;
            dG[ix] = from_float<T>(da * u * (sg * (1.0f + g * (1.0f - sg))));
            dU[ix] = from_float<T>(da * sl);
            A[ix] = from_float<T>(sl * u * sc);   // scaled: the weight gradient multiplies it with unscaled rows
            return da0 * (sl * u);
        });
}

// two-matrix expert: dH = dA * act'(H), A = act(H)
template <typename T, int ACT, bool BIG>
__global__ XMOE_TILE_BOUNDS void mlp2_dact_mfma_kernel(const T* __restrict__ dY,
                                                       const int32_t* __restrict__ dy_index,   // or NULL
                                                       const float* __restrict__ dy_scale,     // or NULL
                                                       const int32_t* __restrict__ off,
                                                       const int32_t* __restrict__ map, int d, int f,
                                                       const T* __restrict__ w2, const T* __restrict__ H,
                                                       T* __restrict__ dH, T* __restrict__ A,
                                                       float* __restrict__ row_part, int B) {
    dact_tile<T, BIG>(
        dY, dy_index, dy_scale, off, map, d, f, w2, row_part, B,
        [&](size_t ix, float& h, float& unused) { h = to_float(H[ix]); unused = 0.f; },
        [&](size_t ix, float da0, float sc, float h, float) {
            float a, g;
            act_fwd_grad<ACT>(h, a, g);
            dH[ix] = from_float<T>(da0 * sc * g);
            A[ix] = from_float<T>(a * sc);
            return da0 * a;
        });
}

// ---------------------------------------------------------------------------------------------------------
// backward 2: dXd = dG Wg^T + dU Wu^T                        rows: ragged, K = f (twice), N = d
// ---------------------------------------------------------------------------------------------------------
template <typename T, bool BIG>
__global__ XMOE_TILE_BOUNDS void ffn_dx_mfma_kernel(const T* __restrict__ dG, const T* __restrict__ dU,
                                                    const int32_t* __restrict__ off,
                                                    const int32_t* __restrict__ map, int d, int f,
                                                    const T* __restrict__ wg, const T* __restrict__ wu,
                                                    T* __restrict__ dXd) {
    using S = TileShape<BIG>;
    __shared__ __align__(16) char smem[S::kLds];
    RowTile t;
    if (!t.init(off, map, (d + S::kN - 1) / S::kN, S::kM)) return;
    const int n0 = t.col * S::kN;
    tile_f32x16_t acc[S::kMI][2];
    tile_zero<BIG>(acc);
    for (int set = 0; set < (dU ? 2 : 1); ++set) {   // the two-matrix expert has a single pair (dH, W1)
        RowSrc<T, S::kThreads> a, b;
        a.init((set ? dU : dG) + (size_t)t.row0 * f, f, t.rows, nullptr);
        b.init((set ? wu : wg) + ((size_t)t.e * d + n0) * f, f, d - n0, nullptr);
        tile_mainloop<T, BIG, false, false>(acc, f, t.rows, d - n0, a, b, smem);
    }
    if constexpr (std::is_same<T, float>::value)
        tile_finish<BIG, false>(acc, f, dU ? 2 : 1, [&](int set, int) {
            return PlainPair{{(set ? dU : dG) + (size_t)t.row0 * f, (size_t)f, 1, nullptr, nullptr, t.rows},
                             {(set ? wu : wg) + ((size_t)t.e * d + n0) * f, (size_t)f, 1, nullptr, nullptr, d - n0}};
        });
    tile_store<T, BIG>(acc, dXd + (size_t)t.row0 * d + n0, d, t.rows, d - n0);
}

// ---------------------------------------------------------------------------------------------------------
// weight gradients: dWd = A^T dY (M=f, N=d);  dWg = Xd^T dG, dWu = Xd^T dU (M=d, N=f)   (K = ragged).  Empty experts get
// zeros.
// ---------------------------------------------------------------------------------------------------------
template <typename T, bool BIG, bool GP, bool GQ>
__device__ __forceinline__ void wgrad_tile(const WgradJob<T>& j, int u, int e, int lo, int K, char* smem) {
    using S = TileShape<BIG>;
    const int tiles_m = (j.M + S::kM - 1) / S::kM, m0 = (u % tiles_m) * S::kM, n0 = (u / tiles_m) * S::kN;
    const T *P = j.P + m0 + (GP ? 0 : (size_t)lo * j.M), *Q = j.Q + n0 + (GQ ? 0 : (size_t)lo * j.N);
    const int32_t *pi = GP ? j.p_index + lo : nullptr, *qi = GQ ? j.q_index + lo : nullptr;
    T* dW = j.dW + (size_t)e * j.M * j.N + (size_t)m0 * j.N + n0;
    tile_f32x16_t acc[S::kMI][2];
    tile_zero<BIG>(acc);
    if constexpr (std::is_same<T, float>::value) {
        const PlainPair q = {{P, 1, (size_t)j.M, nullptr, pi, j.M - m0}, {Q, 1, (size_t)j.N, nullptr, qi, j.N - n0}};
        if (K <= kPlainK) {   // few rows are usual here
            tile_plain<BIG>(acc, K, q);
            tile_store<T, BIG>(acc, dW, j.N, j.M - m0, j.N - n0);
            return;
        }
    }
    ColSrc<T, S::kThreads, GP> a;
    ColSrc<T, S::kThreads, GQ> b;
    a.init(P, nullptr, j.M, j.M - m0, pi, K);
    b.init(Q, nullptr, j.N, j.N - n0, qi, K);
    tile_mainloop<T, BIG, false, true>(acc, K, j.M - m0, j.N - n0, a, b, smem);
    if constexpr (std::is_same<T, float>::value)
        tile_finish<BIG, false>(acc, K, 1, [&](int, int) {
            return PlainPair{{P, 1, (size_t)j.M, nullptr, pi, j.M - m0}, {Q, 1, (size_t)j.N, nullptr, qi, j.N - n0}};
        });
    tile_store<T, BIG>(acc, dW, j.N, j.M - m0, j.N - n0);
}

template <typename T, bool BIG>
__global__ XMOE_TILE_BOUNDS void ffn_wgrad_mfma_kernel(WgradJobs<T> jobs, int E, const int32_t* __restrict__ off,
                                                       const int32_t* __restrict__ sched) {
    __shared__ __align__(16) char smem[TileShape<BIG>::kLds];
    int m, u;
    if (!jobs.place(E, m, u)) return;
    const WgradJob<T> j = jobs.job[m % jobs.n_jobs];
    const int e = sched[m / jobs.n_jobs];
    const int lo = off[e], K = off[e + 1] - lo;
    if (j.p_index)   // gathered rows on at most one side
        wgrad_tile<T, BIG, true, false>(j, u, e, lo, K, smem);
    else if (j.q_index)
        wgrad_tile<T, BIG, false, true>(j, u, e, lo, K, smem);
    else
        wgrad_tile<T, BIG, false, false>(j, u, e, lo, K, smem);
}

// ---------------------------------------------------------------------------------------------------------
// two-matrix expert, forward 1: H = Xd W1, A = act(H)         rows: ragged, K = d, N = f
// ---------------------------------------------------------------------------------------------------------
template <typename T, int ACT, bool BIG>
__global__ XMOE_TILE_BOUNDS void mlp2_up_mfma_kernel(const T* __restrict__ xd,
                                                     const int32_t* __restrict__ row_index,   // or NULL
                                                     const int32_t* __restrict__ off,
                                                     const int32_t* __restrict__ map, int d, int f,
                                                     const T* __restrict__ w1, T* __restrict__ H,
                                                     T* __restrict__ A) {
    using S = TileShape<BIG>;
    __shared__ __align__(16) char smem[S::kLds];
    RowTile t;
    if (!t.init(off, map, (f + S::kN - 1) / S::kN, S::kM)) return;
    const int n0 = t.col * S::kN;
    RowSrc<T, S::kThreads> a;
    ColSrc<T, S::kThreads, false> b;
    a.init(row_index ? xd : xd + (size_t)t.row0 * d, d, t.rows, row_index ? row_index + t.row0 : nullptr);
    b.init(w1 + (size_t)t.e * d * f + n0, nullptr, f, f - n0, nullptr, d);
    tile_f32x16_t acc[S::kMI][2];
    tile_zero<BIG>(acc);
    tile_mainloop<T, BIG, false, false>(acc, d, t.rows, f - n0, a, b, smem);
    if constexpr (std::is_same<T, float>::value)
        tile_finish<BIG, false>(acc, d, 1, [&](int, int) {
            return PlainPair{{row_index ? xd : xd + (size_t)t.row0 * d, (size_t)d, 1, row_index ? row_index + t.row0 : nullptr, nullptr, t.rows},
                             {w1 + (size_t)t.e * d * f + n0, 1, (size_t)f, nullptr, nullptr, f - n0}};
        });
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
        const int n = n0 + tile_col<BIG, false>(ni);
        if (n >= f) continue;
#pragma unroll
        for (int mi = 0; mi < S::kMI; ++mi)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = tile_row<BIG>(mi, v);
                if (r < t.rows) {
                    const size_t ix = (size_t)(t.row0 + r) * f + n;
                    const float h = acc[mi][ni][v];
                    H[ix] = from_float<T>(h);
                    A[ix] = from_float<T>(act_fwd<ACT>(h));
                }
            }
    }
}

// ---------------------------------------------------------------------------------------------------------
// host-side drivers
// ---------------------------------------------------------------------------------------------------------
static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Tile of a call's row GEMMs (the tile map is built for it): the big one when the experts' mean row count fills most of
// it and there are enough blocks.  float32 wants a block for every CU, since its matrix products are long: whole steps
// with the big | small tile at 96 blocks (T 512 d 1024 f 704 E 16+1) 780 | 681 us, at 264 blocks (T 4096 d 512 f 512
// E 64) 1142 | 1231, at 480 (T 2048) 1665 | 1740.  bf16 gains from the big tile's fewer LDS and L2 reads earlier: 128
// blocks (T 1024 d 1000 f 1000 E 8) 289 | 321, 192 blocks (T 1000 d 1000 f 712 E 24+1) 398 | 456, 564 blocks 664 | 1009.
static inline bool big_tiles(int B, int E, int d, int f, int dt) {
    const long long blocks = (long long)ceil_div(B, 128) * ceil_div(d < f ? d : f, 128);
    return B >= 96 * E && blocks >= (dt == XMOE_F32 ? 256 : 96);
}
// Tile of the weight gradients: big when that still gives every CU two blocks (float32 and bf16: the steps above, whose
// weight gradients have 450 to 3000 big tiles, and 384 | 1536 at T 3000 d 300 f 500 E 8: 448 | 416 us).
static inline bool big_wgrad_tiles(int jobs, int E, int d, int f) {
    return (long long)jobs * E * ceil_div(d, 128) * ceil_div(f, 128) >= 512;
}

template <typename T, class Args>
static int wgrad_call(const Args& a, hipStream_t s) {
    WgradJobs<T> jobs = wgrad_jobs<T>(a);
    const bool big = big_wgrad_tiles(jobs.n_jobs, a.E, a.d, a.f);
    const dim3 grid = jobs.cut(a.E, a.d, a.f, big ? 128 : 64);
    if (big)
        XMOE_LAUNCH(K_FFN_WGRAD_MFMA, s, hipLaunchKernelGGL((ffn_wgrad_mfma_kernel<T, true>), grid, dim3(256), 0, s, jobs,
                                                            a.E, a.off, a.sched));
    else
        XMOE_LAUNCH(K_FFN_WGRAD_MFMA, s, hipLaunchKernelGGL((ffn_wgrad_mfma_kernel<T, false>), grid, dim3(128), 0, s,
                                                            jobs, a.E, a.off, a.sched));
    return XMOE_OK;
}

template <typename T, bool BIG>
static int fwd_tile(const FfnArgs& a, hipStream_t s) {
    using S = TileShape<BIG>;
    const int max_tiles = ffn_max_tiles(a.B, a.E, S::kM);
    int st = launch_tile_map(a.off, a.E, S::kM, max_tiles, a.map, a.sched, false, s);
    if (st != XMOE_OK) return st;
    const dim3 g1 = row_grid(max_tiles, ceil_div(a.f, S::kN / 2)), g2 = row_grid(max_tiles, ceil_div(a.d, S::kN));
    XMOE_LAUNCH(K_FFN_GATEUP_MFMA, s,
                hipLaunchKernelGGL((ffn_gateup_mfma_kernel<T, BIG>), g1, dim3(S::kThreads), 0, s, (const T*)a.xd,
                                   a.row_index, a.off, a.map, a.d, a.f, (const T*)a.wg, (const T*)a.wu, (T*)a.g,
                                   (T*)a.u, (T*)a.act));
    XMOE_LAUNCH(K_FFN_DOWN_MFMA, s,
                hipLaunchKernelGGL((ffn_down_mfma_kernel<T, BIG>), g2, dim3(S::kThreads), 0, s, (const T*)a.act, a.off,
                                   a.map, a.d, a.f, (const T*)a.wd, (T*)a.y));
    return XMOE_OK;
}

template <typename T, bool BIG>
static int bwd_rows_tile(const FfnArgs& a, hipStream_t s) {
    using S = TileShape<BIG>;
    const int max_tiles = ffn_max_tiles(a.B, a.E, S::kM);
    int st = launch_tile_map(a.off, a.E, S::kM, max_tiles, a.map, a.sched, true, s);
    if (st != XMOE_OK) return st;
    XMOE_LAUNCH(K_FFN_DACT_MFMA, s,
                hipLaunchKernelGGL((ffn_dact_mfma_kernel<T, BIG>), row_grid(max_tiles, ceil_div(a.f, S::kN)),
                                   dim3(S::kThreads), 0, s, (const T*)a.dy, a.dy_index, a.dy_scale, a.off, a.map, a.d,
                                   a.f, (const T*)a.wd, (const T*)a.g, (const T*)a.u, (T*)a.dg, (T*)a.du, (T*)a.act,
                                   a.row_part, a.B));
    if (a.row_grad) {
        st = launch_row_grad_reduce(a.row_part, ceil_div(a.f, 64), a.B, a.row_grad, s);
        if (st != XMOE_OK) return st;
    }
    XMOE_LAUNCH(K_FFN_DX_MFMA, s,
                hipLaunchKernelGGL((ffn_dx_mfma_kernel<T, BIG>), row_grid(max_tiles, ceil_div(a.d, S::kN)),
                                   dim3(S::kThreads), 0, s, (const T*)a.dg, (const T*)a.du, a.off, a.map, a.d, a.f,
                                   (const T*)a.wg, (const T*)a.wu, (T*)a.dxd));
    return XMOE_OK;
}

template <typename T, bool BIG>
static int mlp2_fwd_tile(const Mlp2Args& a, hipStream_t s) {
    using S = TileShape<BIG>;
    const int max_tiles = ffn_max_tiles(a.B, a.E, S::kM);
    int st = launch_tile_map(a.off, a.E, S::kM, max_tiles, a.map, a.sched, false, s);
    if (st != XMOE_OK) return st;
    const dim3 g1 = row_grid(max_tiles, ceil_div(a.f, S::kN)), g2 = row_grid(max_tiles, ceil_div(a.d, S::kN));
#define XMOE_CALL(ACT)                                                                                               \
    XMOE_LAUNCH(K_MLP2_UP_MFMA, s,                                                                                   \
                hipLaunchKernelGGL((mlp2_up_mfma_kernel<T, ACT, BIG>), g1, dim3(S::kThreads), 0, s, (const T*)a.xd,  \
                                   a.row_index, a.off, a.map, a.d, a.f, (const T*)a.w1, (T*)a.h, (T*)a.a_buf))
    XMOE_DISPATCH_ACT(a.act, XMOE_CALL);
#undef XMOE_CALL
    XMOE_LAUNCH(K_FFN_DOWN_MFMA, s,
                hipLaunchKernelGGL((ffn_down_mfma_kernel<T, BIG>), g2, dim3(S::kThreads), 0, s, (const T*)a.a_buf,
                                   a.off, a.map, a.d, a.f, (const T*)a.w2, (T*)a.y));
    return XMOE_OK;
}

template <typename T, bool BIG>
static int mlp2_bwd_rows_tile(const Mlp2Args& a, hipStream_t s) {
    using S = TileShape<BIG>;
    const int max_tiles = ffn_max_tiles(a.B, a.E, S::kM);
    int st = launch_tile_map(a.off, a.E, S::kM, max_tiles, a.map, a.sched, true, s);
    if (st != XMOE_OK) return st;
    const dim3 g1 = row_grid(max_tiles, ceil_div(a.f, S::kN));
#define XMOE_CALL(ACT)                                                                                                \
    XMOE_LAUNCH(K_MLP2_DACT_MFMA, s,                                                                                  \
                hipLaunchKernelGGL((mlp2_dact_mfma_kernel<T, ACT, BIG>), g1, dim3(S::kThreads), 0, s, (const T*)a.dy, \
                                   a.dy_index, a.dy_scale, a.off, a.map, a.d, a.f, (const T*)a.w2, (const T*)a.h,     \
                                   (T*)a.dh, (T*)a.a_buf, a.row_part, a.B))
    XMOE_DISPATCH_ACT(a.act, XMOE_CALL);
#undef XMOE_CALL
    if (a.row_grad) {
        st = launch_row_grad_reduce(a.row_part, ceil_div(a.f, 64), a.B, a.row_grad, s);
        if (st != XMOE_OK) return st;
    }
    XMOE_LAUNCH(K_FFN_DX_MFMA, s,
                hipLaunchKernelGGL((ffn_dx_mfma_kernel<T, BIG>), row_grid(max_tiles, ceil_div(a.d, S::kN)),
                                   dim3(S::kThreads), 0, s, (const T*)a.dh, (const T*)nullptr, a.off, a.map, a.d, a.f,
                                   (const T*)a.w1, (const T*)nullptr, (T*)a.dxd));
    return XMOE_OK;
}

// Widths that are multiples of 8 (bf16): the forward's row products always take the direct-to-LDS tiles, whatever the
// number of rows (staged small tiles | direct, us: E 24 d 1000 f 712, 16 rows per expert 40 | 33; E 16 d 2040 f 1480, 40
// rows 96 | 78; E 4 d 1496 f 208, 1500 rows 61 | 40), the backward's as direct_rows says.
//
// Their weight gradients take the direct-to-LDS 128 x 128 tiles as well; the staged ones where the experts have hardly any
// rows (a 64 x 64 tile of nothing but its stores).  Whole backward, us, staged | direct:
//   rows per expert             1          16          96          375         1500
//   E 24 d 1000 f 712         83 | 100   118 | 104   139 | 113   244 | 189   697 | 585
//   E 16 d 2040 f 1480       208 | 204   284 | 235   341 | 256   601 | 451  1642 | 1432
//   E 256 d 328 f 200         91 | 103   153 | 124   183 | 144   400 | 346   988 | 957 (1200 rows)
//   E 8 d 1000 f 1000         64 | 69     80 | 76     91 | 82    118 | 104   282 | 241
//   E 4 d 1496 f 208          40 | 40     52 | 43     59 | 46     72 | 57    131 | 102
// The 256-row kernels (K-strided operands only have to be whole 16-byte pieces) would take these widths too.  They are
// ahead at many rows and even loads, and far behind where one segment is long, whose few tiles then are their launch; no
// rule on the mean can tell the two.  Whole backward, us, direct | 256-row, even load, Zipf-like, one segment E/4 times as
// long:
//   E 24 d 1000 f 712,    375 rows   177 | 186     175 | 229     199 | 259
//                        1200        447 | 439     459 | 583     549 | 709
//   E 64 d 520 f 264,     375        159 | 162     157 | 253     185 | 385
//                        1200        418 | 373     431 | 737     579 | 972
//   E 64 d 1000 f 712,    375        488 | 449     505 | 524     590 | 700
//                        1200       1276 | 1120   1273 | 1371   1541 | 1945
//   E 256 d 328 f 200,    375        346 | 315     379 | 507     596 | 940
//                        1200        957 | 752    1126 | 1328   1125 | 1649
//   E 8 d 2040 f 1480,    375        206 | 221     214 | 248     219 | 236
//                        1200        519 | 502     545 | 567     621 | 597
template <class Args>
static int wgrads_any_width(const Args& a, int (*direct)(const Args&, hipStream_t), hipStream_t s) {
    if (a.dt == XMOE_F32) return wgrad_call<float>(a, s);
    return direct_supported(a) && a.B >= 12ll * a.E ? direct(a, s) : wgrad_call<bf16_t>(a, s);
}

// dAct and dX at these widths: direct where the staged 64 x 64 tiles (row tiles of a mean segment, columns of the wider
// product) are more than the 512 blocks that the chip holds at a time, and not for hardly any rows.  Whole backward, us,
// staged | direct (blocks):
//   E 16 d 1000 f 712:    45 rows   86 | 90 (256)       80 rows   92 | 92 (512)     120 rows  116 | 97 (512 to 768)
//   E 8 d 2040 f 1480:    45       138 | 147 (256)      96       142 | 148 (512)    120       176 | 151 (512 to 768)
//   E 32 d 2040 f 1480:   20       403 | 393 (1024)     64       533 | 429          160       610 | 579
//   E 8 d 1000 f 1000:    80        79 | 84 (256)      160        89 | 88 (384)     200       108 | 91 (512)
//   E 4 d 1000 f 712:    160        64 | 67 (192)      400        77 | 76 (448)     520        95 | 78 (576)
//   E 2 d 2040 f 1480:   200        92 | 101 (256)     400       108 | 109 (448)    520       135 | 111 (576)
//   E 3 d 2504 f 1000:   200        94 | 100 (480)     280       102 | 104 (600)    400       119 | 110 (840)
//   E 64 d 1000 f 712:     6       250 | 254 (1024)     45       245 | 238          90        305 | 253 (2048)
//   E 256 d 520 f 264:     6       298 | 299 (2304)     45       240 | 225          90        313 | 265 (4608)
//   E 96 d 520 f 520:      4       167 | 171 (864)      30       145 | 144          60        177 | 154
static inline bool direct_rows(int B, int E, int d, int f) {
    const long long blocks = (long long)E * ceil_div(ceil_div(B, E), 64) * ceil_div(d > f ? d : f, 64);
    return B >= 24ll * E && blocks > 512;
}

#define XMOE_TILE_CALL(CALL)                                                              \
    (a.dt == XMOE_F32 ? (big ? CALL<float, true>(a, s) : CALL<float, false>(a, s))        \
                      : (big ? CALL<bf16_t, true>(a, s) : CALL<bf16_t, false>(a, s)))

int ffn_fwd_tile(const FfnArgs& a, hipStream_t s) {
    if (direct_supported(a)) return ffn_fwd_direct(a, s);
    const bool big = big_tiles(a.B, a.E, a.d, a.f, a.dt);
    return XMOE_TILE_CALL(fwd_tile);
}
int mlp2_fwd_tile(const Mlp2Args& a, hipStream_t s) {
    if (direct_supported(a)) return mlp2_fwd_direct(a, s);
    const bool big = big_tiles(a.B, a.E, a.d, a.f, a.dt);
    return XMOE_TILE_CALL(mlp2_fwd_tile);
}
int ffn_bwd_tile(const FfnArgs& a, hipStream_t s) {
    const bool big = big_tiles(a.B, a.E, a.d, a.f, a.dt);
    const bool direct = direct_rows(a.B, a.E, a.d, a.f) && direct_supported(a);
    const int st = direct ? ffn_bwd_rows_direct(a, s) : XMOE_TILE_CALL(bwd_rows_tile);
    return st != XMOE_OK ? st : wgrads_any_width(a, ffn_bwd_wgrads_direct, s);
}
int mlp2_bwd_tile(const Mlp2Args& a, hipStream_t s) {
    const bool big = big_tiles(a.B, a.E, a.d, a.f, a.dt);
    const bool direct = direct_rows(a.B, a.E, a.d, a.f) && direct_supported(a);
    const int st = direct ? mlp2_bwd_rows_direct(a, s) : XMOE_TILE_CALL(mlp2_bwd_rows_tile);
    return st != XMOE_OK ? st : wgrads_any_width(a, mlp2_bwd_wgrads_direct, s);
}

}  // namespace xmoe
