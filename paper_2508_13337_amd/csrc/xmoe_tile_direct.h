// The 128 x 128 bf16 tile of xmoe_tile_gemm.h with its operands loaded straight into LDS, for operands whose rows are
// whole 16-byte pieces (widths that are multiples of 8, 16-byte aligned bases).
//
//   block = 256 threads = 4 waves (2 x 2), wave tile 64 x 64, 80 KiB of LDS: two blocks per CU
//
// A K-contiguous operand lies in LDS in units of [128 rows][64 k], fetched as whole 128-byte pieces of rows (half of that
// costs the address units and the L2 channels as much per request), a K-strided one in tiles of [32 k][128 columns], read
// with the transposing LDS read.  Two K-contiguous operands run a ring of five units (dir_loop_rr), one of each three
// units and four tiles (dir_loop_rc): the rings of the 256-row kernels at half size, two to three units of a block on
// their way while one is multiplied.
// A direct-to-LDS load puts lane l's 16 bytes at a wave-uniform base + 16 l, so the swizzles that keep the fragment reads
// off each other's banks choose which piece a lane fetches.  A piece past the end of K is fetched from a block of zeros;
// rows and columns past the last one repeat one that exists, what they feed is not stored.
// The matrix instruction takes the fragment of B first: a lane then owns runs of four consecutive columns of one output
// row (tile_row and tile_col do not apply).  K is added in the same ascending steps of 16 as everywhere else.
#pragma once

#include <type_traits>

#include "xmoe_ffn.h"
#include "xmoe_tile_gemm.h"

namespace xmoe {

typedef __attribute__((ext_vector_type(4))) short tile_s16x4_t;
typedef __attribute__((ext_vector_type(8))) short tile_s16x8_t;

constexpr int kDirUnit = 128 * 64 * 2, kDirTile = 32 * 128 * 2, kDirLds = 5 * kDirUnit;
__device__ __align__(16) const unsigned int kDirZero[4] = {0u, 0u, 0u, 0u};
__device__ const float kDirOne = 1.0f;

#define XMOE_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define XMOE_GLB_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

// A lane's four 16-byte pieces of a K-contiguous operand per unit.  TWO: K is the concatenation of two operand sets of
// equal length.
template <bool TWO>
struct DirRows {
    const bf16_t* p[4];             // of the unit issued next
    const bf16_t* q[TWO ? 4 : 1];   // TWO: of the second set's first unit
    int limit[2];                   // units of a set in which the pieces 0 and 2, 1 and 3 lie before the end of K
    // element (r, k) at base + row(r) * ld + k; n_valid >= 1 rows, index as in RowSrc; base2: the second set
    __device__ __forceinline__ void init(const bf16_t* base, const bf16_t* base2, size_t ld, int n_valid,
                                         const int32_t* index, int K) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int r = wave * 32 + i * 8 + (lane >> 3);
            const int c = (lane & 7) ^ ((r >> 1) & 7);
            r = r < n_valid ? r : n_valid - 1;
            if (index) r = index[r];
            p[i] = base + (size_t)r * ld + c * 8;
            if (TWO) q[TWO ? i : 0] = base2 + (size_t)r * ld + c * 8;
            if (i < 2) limit[i] = (K - c * 8 + 63) / 64;
        }
    }
    // requests unit u (units come in order); n1: units of a set
    __device__ __forceinline__ void issue(char* __restrict__ unit, int u, int n1) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int s = TWO && u >= n1 ? u - n1 : u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (TWO && u == n1) p[i] = q[TWO ? i : 0];
            const bf16_t* a = s < limit[i & 1] ? p[i] : reinterpret_cast<const bf16_t*>(kDirZero);
            __builtin_amdgcn_global_load_lds(XMOE_GLB_PTR(a), XMOE_LDS_PTR(unit + wave * 4096 + i * 1024), 16, 0, 0);
            p[i] += 64;
        }
    }
};
// A lane's two 16-byte pieces of a K-strided operand per tile: element (k, n) at p0 + k * ld + n; p1 (or NULL): the tile's
// columns 64 .. are columns 0 .. of p1; cols >= 8 columns from p0 (p1) on
struct DirCols {
    const bf16_t* p[2];   // of the tile issued next
    int limit[2];         // tiles in which the piece lies before the end of K
    size_t step;
    __device__ __forceinline__ void init(const bf16_t* p0, const bf16_t* p1, size_t ld, int cols, int K) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int kr = wave * 8 + i * 4 + (lane >> 4);
            int n = 8 * ((lane & 15) ^ ((kr & 3) << 2));
            const bf16_t* b = p0;
            if (p1 && n >= 64) {
                n -= 64;
                b = p1;
            }
            if (n >= cols) n = 0;
            p[i] = b + (size_t)kr * ld + n;
            limit[i] = (K - kr + 31) / 32;
        }
        step = 32 * ld;
    }
    __device__ __forceinline__ void issue(char* __restrict__ tile, int t) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bf16_t* a = t < limit[i] ? p[i] : reinterpret_cast<const bf16_t*>(kDirZero);
            __builtin_amdgcn_global_load_lds(XMOE_GLB_PTR(a), XMOE_LDS_PTR(tile + wave * 2048 + i * 1024), 16, 0, 0);
            p[i] += step;
        }
    }
};

// 8 bf16 (k = 16 ks + 8 (lane/32) ..) of row base + lane%32 of a unit (ks 0..3), of column base + lane%32 of a tile (ks 0..1)
__device__ __forceinline__ tile_bf16x8_t dir_frag_row(const char* unit, int base, int ks) {
    const int lane = threadIdx.x & 63, r = base + (lane & 31), c = 2 * ks + (lane >> 5);
    return *reinterpret_cast<const tile_bf16x8_t*>(unit + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
}
__device__ __forceinline__ tile_bf16x8_t dir_frag_col(const char* tile, int base, int ks) {
    // in a group G of 16 lanes, lane s addresses 4 consecutive columns (s%4) of k-row s/4, and the transposing read hands
    // every lane one column with 4 consecutive k
    const int lane = threadIdx.x & 63, G = lane >> 4, s = lane & 15, col = base + 16 * (G & 1) + 4 * (s & 3);
    tile_s16x4_t h[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int kr = 16 * ks + 8 * (G >> 1) + (s >> 2) + 4 * i;
        const char* a = tile + kr * 256 + (((col >> 3) ^ ((kr & 3) << 2)) << 4) + (col & 7) * 2;
        h[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) tile_s16x4_t*)XMOE_LDS_PTR(a));
    }
    const tile_s16x8_t v = {h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]};
    return __builtin_bit_cast(tile_bf16x8_t, v);
}

// first column of the wave's ni-th 32-column block; DUAL: the same 32 columns of two matrices of 64 columns each
template <bool DUAL>
__device__ __forceinline__ int dir_col(int ni) {
    const int wn = (threadIdx.x >> 6) & 1;
    return DUAL ? ni * 64 + wn * 32 : wn * 64 + ni * 32;
}

template <int MI>
struct DirFrags {
    tile_bf16x8_t a[MI], b[2];
};
template <int MI>
__device__ __forceinline__ void dir_clear(DirFrags<MI>& f) {
    const tile_s16x8_t z = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) f.a[mi] = __builtin_bit_cast(tile_bf16x8_t, z);
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) f.b[ni] = __builtin_bit_cast(tile_bf16x8_t, z);
}
// acc[mi][ni][v]: row 64 wm + 32 mi + lane%32, column dir_col(ni) + 8 (v/4) + 4 (lane/32) + v%4
template <int MI>
__device__ __forceinline__ void dir_mma(tile_f32x16_t (&acc)[2][2], const DirFrags<MI>& f) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[ni], f.a[mi], acc[mi][ni], 0, 0, 0);
}

// Waits until at most N of the wave's loads are on their way and its LDS reads have returned, then joins the barrier.  (As
// asm: __syncthreads() would wait for every outstanding direct-to-LDS load.)
template <int N>
__device__ __forceinline__ void dir_wait_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// ---- both operands K-contiguous: units A(0) B(0) A(1) B(1) .. in five slots
// One pass: the four 16-wide steps on A(p) = ua, B(p) = ub.  On entry both have landed, every wave has left the units of
// pass p-1 (the slots fill1, fill2), and f1 holds the last step of pass p-1.  The slots are distinct, and saying so
// matters: an LDS read that may observe a direct-to-LDS load in flight makes the compiler wait for all of them.
template <int MI>
__device__ __forceinline__ void dir_read_rr(DirFrags<MI>& f, const char* ua, const char* ub, int ks) {
    const int wm = threadIdx.x >> 7;
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) f.b[ni] = dir_frag_row(ub, dir_col<false>(ni), ks);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) f.a[mi] = dir_frag_row(ua, wm * 64 + mi * 32, ks);
}
template <bool TWO, int MI>
__device__ __forceinline__ void dir_pass_rr(tile_f32x16_t (&acc)[2][2], DirFrags<MI>& f0, DirFrags<MI>& f1, DirRows<TWO>& a,
                                            DirRows<TWO>& b, int p, int n1, char* __restrict__ fill1,
                                            char* __restrict__ fill2, const char* __restrict__ ua,
                                            const char* __restrict__ ub) {
    b.issue(fill1, p + 1, n1);
    __builtin_amdgcn_sched_barrier(0);   // the requests stay where they stand: sunk to the end of the pass they are late
    dir_read_rr<MI>(f0, ua, ub, 0);
    dir_mma<MI>(acc, f1);
    dir_read_rr<MI>(f1, ua, ub, 1);
    dir_mma<MI>(acc, f0);
    __builtin_amdgcn_sched_barrier(0);
    a.issue(fill2, p + 2, n1);
    __builtin_amdgcn_sched_barrier(0);
    dir_read_rr<MI>(f0, ua, ub, 2);
    dir_mma<MI>(acc, f1);
    dir_read_rr<MI>(f1, ua, ub, 3);
    dir_mma<MI>(acc, f0);
}
template <bool TWO, int MI>
__device__ __forceinline__ void dir_loop_rr(tile_f32x16_t (&acc)[2][2], DirRows<TWO>& a, DirRows<TWO>& b, int n, int n1,
                                            char* smem) {
    DirFrags<MI> f0, f1;
    dir_clear(f1);
    int sa = 0;   // slot of A(p) = 2p % 5
    for (int p = 0; p < n; ++p) {
        const int sb = sa + 1 < 5 ? sa + 1 : sa - 4, s3 = sa + 3 < 5 ? sa + 3 : sa - 2, s4 = sa + 4 < 5 ? sa + 4 : sa - 1;
        dir_pass_rr<TWO, MI>(acc, f0, f1, a, b, p, n1, smem + s3 * kDirUnit, smem + s4 * kDirUnit, smem + sa * kDirUnit,
                             smem + sb * kDirUnit);
        dir_wait_and_barrier<4>();
        sa = sa + 2 < 5 ? sa + 2 : sa - 3;
    }
    dir_mma<MI>(acc, f1);
}

// acc += A B over K (TWO: over both sets); rows, cols: valid ones of the tile, which may exceed it.  Every thread of the
// block calls it; smem (kDirLds bytes) is free again behind it.
template <bool TWO>
__device__ __forceinline__ void dir_mainloop_rr(tile_f32x16_t (&acc)[2][2], DirRows<TWO>& a, DirRows<TWO>& b, int K, int rows,
                                                int cols, char* smem) {
    const int n1 = (K + 63) / 64, n = TWO ? 2 * n1 : n1;
    a.issue(smem, 0, n1);
    b.issue(smem + kDirUnit, 0, n1);
    a.issue(smem + 2 * kDirUnit, 1, n1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mi_n = cols > (wave & 1) * 64 ? (rows - (wave >> 1) * 64 + 31) / 32 : 0;
    // at the top of pass p everything up to B(p) has landed for every thread, A(p+1) may be on its way
    dir_wait_and_barrier<4>();
    if (mi_n >= 2) {
        dir_loop_rr<TWO, 2>(acc, a, b, n, n1, smem);
    } else if (mi_n == 1) {
        dir_loop_rr<TWO, 1>(acc, a, b, n, n1, smem);
    } else {
        int sa = 0;
        for (int p = 0; p < n; ++p) {
            b.issue(smem + (sa + 3 < 5 ? sa + 3 : sa - 2) * kDirUnit, p + 1, n1);
            a.issue(smem + (sa + 4 < 5 ? sa + 4 : sa - 1) * kDirUnit, p + 2, n1);
            dir_wait_and_barrier<4>();
            sa = sa + 2 < 5 ? sa + 2 : sa - 3;
        }
    }
    dir_wait_and_barrier<0>();   // nothing may land in this LDS any more: it becomes the epilogue's
}

// ---- A K-contiguous, B K-strided: three units of A and behind them four tiles of B.  A pass is the two tiles of A(p): the
// first requests A(p+2) and B(2p+3), the second B(2p+4); at each barrier eight requests of a wave may be on their way (the
// two newest tiles of B and the newest unit of A).
constexpr int kDirTiles = 3 * kDirUnit;   // where B's tiles start
template <bool DUAL, int MI>
__device__ __forceinline__ void dir_read_rc(DirFrags<MI>& f, const char* ua, const char* tb, int ks_a, int ks_b) {
    const int wm = threadIdx.x >> 7;
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) f.b[ni] = dir_frag_col(tb, dir_col<DUAL>(ni), ks_b);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) f.a[mi] = dir_frag_row(ua, wm * 64 + mi * 32, ks_a);
}
template <bool DUAL, int MI, int HALF>
__device__ __forceinline__ void dir_step_rc(tile_f32x16_t (&acc)[2][2], DirFrags<MI>& f0, DirFrags<MI>& f1, DirRows<false>& a,
                                            DirCols& b, int p, int n1, char* __restrict__ fill_a,
                                            char* __restrict__ fill_b, const char* __restrict__ ua,
                                            const char* __restrict__ tb) {
    if (HALF == 0) a.issue(fill_a, p + 2, n1);
    b.issue(fill_b, 2 * p + 3 + HALF);
    dir_read_rc<DUAL, MI>(f0, ua, tb, 2 * HALF, 0);
    dir_mma<MI>(acc, f1);
    dir_read_rc<DUAL, MI>(f1, ua, tb, 2 * HALF + 1, 1);
    dir_mma<MI>(acc, f0);
}
template <bool DUAL, int MI>
__device__ __forceinline__ void dir_loop_rc(tile_f32x16_t (&acc)[2][2], DirRows<false>& a, DirCols& b, int n, char* smem) {
    DirFrags<MI> f0, f1;
    dir_clear(f1);
    char* bt = smem + kDirTiles;
    int sa = 0, sb = 0;   // slot of A(p) = p % 3, of B(2p) = 2p % 4
    for (int p = 0; p < n; ++p) {
        char* fill_a = smem + (sa + 2 < 3 ? sa + 2 : sa - 1) * kDirUnit;
        const char* ua = smem + sa * kDirUnit;
        dir_step_rc<DUAL, MI, 0>(acc, f0, f1, a, b, p, n, fill_a, bt + ((sb + 3) & 3) * kDirTile, ua, bt + sb * kDirTile);
        dir_wait_and_barrier<8>();
        dir_step_rc<DUAL, MI, 1>(acc, f0, f1, a, b, p, n, fill_a, bt + sb * kDirTile, ua, bt + (sb + 1) * kDirTile);
        dir_wait_and_barrier<8>();
        sa = sa + 1 < 3 ? sa + 1 : 0;
        sb ^= 2;
    }
    dir_mma<MI>(acc, f1);
}
// as dir_mainloop_rr; DUAL: cols of either matrix
template <bool DUAL>
__device__ __forceinline__ void dir_mainloop_rc(tile_f32x16_t (&acc)[2][2], DirRows<false>& a, DirCols& b, int K, int rows,
                                                int cols, char* smem) {
    const int n = (K + 63) / 64;
    char* bt = smem + kDirTiles;
    a.issue(smem, 0, n);
    b.issue(bt, 0);
    a.issue(smem + kDirUnit, 1, n);
    b.issue(bt + kDirTile, 1);
    b.issue(bt + 2 * kDirTile, 2);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mi_n = cols > (wave & 1) * (DUAL ? 32 : 64) ? (rows - (wave >> 1) * 64 + 31) / 32 : 0;
    dir_wait_and_barrier<8>();
    if (mi_n >= 2) {
        dir_loop_rc<DUAL, 2>(acc, a, b, n, smem);
    } else if (mi_n == 1) {
        dir_loop_rc<DUAL, 1>(acc, a, b, n, smem);
    } else {
        int sa = 0, sb = 0;
        for (int p = 0; p < n; ++p) {
            a.issue(smem + (sa + 2 < 3 ? sa + 2 : sa - 1) * kDirUnit, p + 2, n);
            b.issue(bt + ((sb + 3) & 3) * kDirTile, 2 * p + 3);
            dir_wait_and_barrier<8>();
            b.issue(bt + sb * kDirTile, 2 * p + 4);
            dir_wait_and_barrier<8>();
            sa = sa + 1 < 3 ? sa + 1 : 0;
            sb ^= 2;
        }
    }
    dir_wait_and_barrier<0>();
}

// ---- both operands K-strided (weight gradients): five stages of a tile of either, four of them on their way.
// GATHER: k-row k is row index[k] of the matrix.  The index of a piece is an ordinary load, issued with the stage four
// before the piece's own: the wait for that stage covers it, so that it never makes the ring wait.  The waits count the
// direct-to-LDS loads of three stages and not the index loads among them: right whatever the compiler makes of those.
constexpr int kDirStage = 2 * kDirTile;
template <bool GATHER>
struct DirColsK {
    const bf16_t* p[2];            // GATHER: the piece's column in row 0, else of the tile issued next
    int limit[2];
    size_t step;                   // GATHER: the leading dimension
    const int32_t* index;
    int last;                      // K - 1
    int row[GATHER ? 4 : 1][2];    // source rows of the pieces of tile t: row[t & 3]
    __device__ __forceinline__ static int k_row(int i) {
        return (int)(threadIdx.x >> 6) * 8 + i * 4 + (int)((threadIdx.x & 63) >> 4);
    }
    __device__ __forceinline__ void init(const bf16_t* p0, size_t ld, int cols, const int32_t* index_, int K) {
        index = index_;
        last = K - 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int kr = k_row(i);
            int n = 8 * ((int)(threadIdx.x & 15) ^ ((kr & 3) << 2));
            if (n >= cols) n = 0;
            p[i] = p0 + (GATHER ? 0 : (size_t)kr * ld) + n;
            limit[i] = (K - kr + 31) / 32;
        }
        step = GATHER ? ld : 32 * ld;
    }
    template <int S>
    __device__ __forceinline__ void fetch(int t) {   // the rows of tile t, t & 3 == S
        if (!GATHER) return;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = 32 * t + k_row(i);
            row[GATHER ? S : 0][i] = index[k < last ? k : last];
        }
    }
    template <int S>
    __device__ __forceinline__ void issue(char* __restrict__ tile, int t) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bf16_t* a = GATHER ? p[i] + (size_t)row[GATHER ? S : 0][i] * step : p[i];
            a = t < limit[i] ? a : reinterpret_cast<const bf16_t*>(kDirZero);
            __builtin_amdgcn_global_load_lds(XMOE_GLB_PTR(a), XMOE_LDS_PTR(tile + wave * 2048 + i * 1024), 16, 0, 0);
            if (!GATHER) p[i] += step;
        }
    }
};
template <bool GA, bool GB, int MI, int S>
__device__ __forceinline__ void dir_step_cc(tile_f32x16_t (&acc)[2][2], DirFrags<MI ? MI : 1>& f0, DirFrags<MI ? MI : 1>& f1,
                                            DirColsK<GA>& a, DirColsK<GB>& b, int i, char* __restrict__ next,
                                            const char* __restrict__ cur) {
    constexpr int M = MI ? MI : 1;
    a.template issue<S>(next, i + 4);
    b.template issue<S>(next + kDirTile, i + 4);
    a.template fetch<S>(i + 8);
    b.template fetch<S>(i + 8);
    if (MI > 0) {
        const int wm = threadIdx.x >> 7;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            DirFrags<M>& f = ks ? f1 : f0;
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) f.b[ni] = dir_frag_col(cur + kDirTile, dir_col<false>(ni), ks);
#pragma unroll
            for (int mi = 0; mi < M; ++mi) f.a[mi] = dir_frag_col(cur, wm * 64 + mi * 32, ks);
            dir_mma<M>(acc, ks ? f0 : f1);
        }
    }
    dir_wait_and_barrier<12>();
}
template <bool GA, bool GB, int MI>
__device__ __forceinline__ void dir_loop_cc(tile_f32x16_t (&acc)[2][2], DirColsK<GA>& a, DirColsK<GB>& b, int n, char* smem) {
    DirFrags<MI ? MI : 1> f0, f1;
    dir_clear(f1);
    // whole rounds of four: an exit from between the steps would cost a copy of every accumulator (stages past the end of K
    // hold zeros)
    char *cur = smem, *next = smem + 4 * kDirStage, *const end = smem + 5 * kDirStage;
    auto step = [&](auto S, int i) {
        dir_step_cc<GA, GB, MI, S.value>(acc, f0, f1, a, b, i, next, cur);
        next = cur;
        cur = cur + kDirStage < end ? cur + kDirStage : smem;
    };
    for (int i = 0; i < n; i += 4) {
        step(std::integral_constant<int, 0>{}, i);
        step(std::integral_constant<int, 1>{}, i + 1);
        step(std::integral_constant<int, 2>{}, i + 2);
        step(std::integral_constant<int, 3>{}, i + 3);
    }
    if (MI > 0) dir_mma<MI ? MI : 1>(acc, f1);
}
// acc += A B over K >= 1; rows, cols: valid ones of the tile.  At most one of the operands is gathered.
template <bool GA, bool GB>
__device__ __forceinline__ void dir_mainloop_cc(tile_f32x16_t (&acc)[2][2], DirColsK<GA>& a, DirColsK<GB>& b, int K, int rows,
                                                int cols, char* smem) {
    static_assert(!(GA && GB), "the wait counts");
    const int n = (K + 31) / 32;
    auto fetch = [&](auto S, int t) {
        a.template fetch<S.value>(t);
        b.template fetch<S.value>(t);
    };
    auto first = [&](auto S) {
        a.template issue<S.value>(smem + S.value * kDirStage, S.value);
        b.template issue<S.value>(smem + S.value * kDirStage + kDirTile, S.value);
        fetch(S, S.value + 4);
    };
    constexpr std::integral_constant<int, 0> S0{};
    constexpr std::integral_constant<int, 1> S1{};
    constexpr std::integral_constant<int, 2> S2{};
    constexpr std::integral_constant<int, 3> S3{};
    fetch(S0, 0);
    fetch(S1, 1);
    fetch(S2, 2);
    fetch(S3, 3);
    first(S0);
    first(S1);
    first(S2);
    first(S3);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mi_n = cols > (wave & 1) * 64 ? (rows - (wave >> 1) * 64 + 31) / 32 : 0;
    dir_wait_and_barrier<12>();
    if (mi_n >= 2)
        dir_loop_cc<GA, GB, 2>(acc, a, b, n, smem);
    else if (mi_n == 1)
        dir_loop_cc<GA, GB, 1>(acc, a, b, n, smem);
    else
        dir_loop_cc<GA, GB, 0>(acc, a, b, n, smem);
    dir_wait_and_barrier<0>();
}

// ---- epilogue: a wave turns 32 rows x up to 192 columns of results into whole rows through a strip of LDS of its own
// (12 KiB; behind it 4 KiB for what it reads).  Rows of 384 bytes; the 8-byte pieces of 128 bytes are XOR-swizzled with
// row / 2, so that neither a column of 32 rows nor a row falls twice on a bank.
constexpr int kDirStripBytes = 32 * 384, kDirWaveBytes = 16384;
__device__ __forceinline__ char* dir_strip(char* smem) { return smem + (threadIdx.x >> 6) * kDirWaveBytes; }
__device__ __forceinline__ int dir_strip_at(int row, int piece) { return row * 384 + ((piece ^ ((row >> 1) & 15)) << 3); }
// a wave's LDS operations execute in order: no barrier is needed, only that the compiler keeps the order
__device__ __forceinline__ void dir_strip_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// this lane's values 4q .. 4q+3 of a 32 x 32 accumulator whose columns start at piece0
__device__ __forceinline__ void dir_put4(char* strip, int piece0, int q, float a, float b, float c, float d) {
    const int lane = threadIdx.x & 63;
    *reinterpret_cast<uint2*>(strip + dir_strip_at(lane & 31, piece0 + 2 * q + (lane >> 5))) =
        make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
}
// writes NC (32 or 64) columns from piece0 on of 32 rows to C; MASK = false: the caller knows all of them to be valid.
// NT: streaming stores (whole lines that this launch does not read)
template <int NC, bool MASK, bool NT>
__device__ __forceinline__ void dir_flush(const char* strip, int piece0, bf16_t* C, size_t ldc, int rows, int cols) {
    const int lane = threadIdx.x & 63;
    constexpr int kPerRow = NC / 4, kRows = 64 / kPerRow;
    const int c = lane % kPerRow;
#pragma unroll
    for (int it = 0; it < 32 / kRows; ++it) {
        const int r = it * kRows + lane / kPerRow;
        if (!MASK || (r < rows && c * 4 < cols)) {
            typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;
            const u32x2_t v = *reinterpret_cast<const u32x2_t*>(strip + dir_strip_at(r, piece0 + c));
            u32x2_t* dst = reinterpret_cast<u32x2_t*>(C + (size_t)r * ldc + c * 4);
            if (NT)
                __builtin_nontemporal_store(v, dst);
            else
                *dst = v;
        }
    }
}

// C[r * ldc + n] of the block's tile (C at its first element)
__device__ __forceinline__ void dir_store(const tile_f32x16_t (&acc)[2][2], char* smem, bf16_t* C, size_t ldc, int rows,
                                          int cols) {
    char* strip = dir_strip(smem);
    const int wm = threadIdx.x >> 7, wn = (threadIdx.x >> 6) & 1;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                dir_put4(strip, 8 * ni, q, acc[mi][ni][4 * q], acc[mi][ni][4 * q + 1], acc[mi][ni][4 * q + 2],
                         acc[mi][ni][4 * q + 3]);
        dir_strip_sync();
        const int r0 = wm * 64 + mi * 32;
        dir_flush<64, true, true>(strip, 0, C + (size_t)r0 * ldc + wn * 64, ldc, rows - r0, cols - wn * 64);
        dir_strip_sync();
    }
}

// The epilogue of dA = dY W^T: NIN arrays of the forward are read, NOUT written, all [B, f], at the tile's first element.
// EPI(pa, sc, in, out): one element from the unscaled product pa, the row's scale sc and in[NIN]; fills out[NOUT] and
// returns the unscaled activation, whose product with pa is summed over the wave's 64 columns into row_part (one part
// per 64 columns; part: the tile's first row of the wave's part).  row_scale: of the tile's first row, or NULL.
// CHAIN: the order of that sum.  A call's row count selects between these tiles and the 256-row ones (CHAIN: a lane's 16
// columns of a 32-column block in turn) or the register-staged ones (otherwise: columns n and n + 32, then halving over the
// 32), and a row's gradient has the same bits from either.
// The inputs of a 32 x 32 block are fetched as whole 64-byte pieces of rows, one block ahead, and turned into the
// accumulators' layout through LDS.  FULL: the wave's 64 x 64 block is entirely valid, and no load or store stands inside
// a branch: the compiler then leaves them outstanding where it would otherwise wait for all of them.
template <bool FULL, bool CHAIN, int NIN, int NOUT, class Epi>
__device__ __forceinline__ void dir_dact_rounds(const tile_f32x16_t (&acc)[2][2], char* smem, const bf16_t* const (&in)[NIN],
                                                bf16_t* const (&out)[NOUT], size_t f, const float* row_scale, float* part,
                                                int rows, int cols, Epi epi) {
    char* strip = dir_strip(smem);
    char* inbuf = strip + kDirStripBytes;
    const int lane = threadIdx.x & 63, wm = threadIdx.x >> 7, wn = (threadIdx.x >> 6) & 1, m = lane & 31;
    const int frow = lane >> 2, fchunk = lane & 3;
    rows -= wm * 64;
    cols -= wn * 64;
    const size_t base = (size_t)(wm * 64) * f + wn * 64;
    // the scales ahead of every other request; without scales every lane reads a 1
    float sc[2];
    {
        typedef const __attribute__((address_space(1))) char* gchar_p;
        typedef const __attribute__((address_space(1))) float* gfloat_p;
        const float* s0 = row_scale ? row_scale + wm * 64 : &kDirOne;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            int r = mi * 32 + m;
            if (!FULL) r = r < rows ? r : 0;
            if (!FULL && rows <= 0) r = -wm * 64;   // the wave's rows lie past the segment: its first row's scale
            sc[mi] = *(gfloat_p)((gchar_p)XMOE_GLB_PTR(s0) + (long)(row_scale ? r : 0) * 4);
        }
    }
    uint4 w[2][NIN][2];
    auto fetch = [&](int r, uint4 (&x)[NIN][2]) {
        const int mi = r >> 1, ni = r & 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = mi * 32 + 16 * i + frow, col = ni * 32 + fchunk * 8;
#pragma unroll
            for (int a = 0; a < NIN; ++a) {
                x[a][i] = make_uint4(0, 0, 0, 0);
                if (FULL || (row < rows && col < cols))
                    x[a][i] = *reinterpret_cast<const uint4*>(in[a] + base + (size_t)row * f + col);
            }
        }
    };
    fetch(0, w[0]);
    float rowpart = 0.f, pcol[16];   // pcol: not CHAIN, this lane's columns n and n + 32
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int mi = r >> 1, ni = r & 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = 16 * i + frow, pos = (fchunk ^ ((row >> 2) & 3)) << 4;
#pragma unroll
            for (int a = 0; a < NIN; ++a) *reinterpret_cast<uint4*>(inbuf + a * 2048 + row * 64 + pos) = w[r & 1][a][i];
        }
        if (r < 3) fetch(r + 1, w[(r + 1) & 1]);
        dir_strip_sync();
        float p = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t iw[NIN][2];
#pragma unroll
            for (int a = 0; a < NIN; ++a) {
                const uint2 v = *reinterpret_cast<const uint2*>(inbuf + a * 2048 + m * 64 + ((q ^ ((m >> 2) & 3)) << 4) +
                                                                8 * (lane >> 5));
                iw[a][0] = v.x;
                iw[a][1] = v.y;
            }
            float o[NOUT][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float x[NIN], y[NOUT];
#pragma unroll
                for (int a = 0; a < NIN; ++a)
                    x[a] = __uint_as_float((j & 1) ? (iw[a][j >> 1] & 0xffff0000u) : (iw[a][j >> 1] << 16));
                const float pa = acc[mi][ni][4 * q + j], a = epi(pa, sc[mi], x, y);
                if (CHAIN) {
                    p = fmaf(pa, a, p);
                } else {   // a column past the last one holds a copy of another's product, which may be infinite
                    const float c = ni == 0 ? 0.f : pcol[4 * q + j];
                    pcol[4 * q + j] = FULL || ni * 32 + 8 * q + 4 * (lane >> 5) + j < cols ? fmaf(pa, a, c) : c;
                }
#pragma unroll
                for (int b = 0; b < NOUT; ++b) o[b][j] = y[b];
            }
#pragma unroll
            for (int b = 0; b < NOUT; ++b) dir_put4(strip, 16 * b + 8 * ni, q, o[b][0], o[b][1], o[b][2], o[b][3]);
        }
        if (CHAIN) rowpart = ni == 0 ? p : rowpart + p;
        if (ni == 1) {
            float tot;
            if (CHAIN) {
                tot = rowpart + __shfl_xor(rowpart, 32, 64);
            } else {   // the halving of tile_sum_over_cols: columns 16, 8, 4 (the other half of the wave), 2 and 1 apart
                float h[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    h[j] = (pcol[j] + pcol[8 + j]) + (pcol[4 + j] + pcol[12 + j]);
                    h[j] += __shfl_xor(h[j], 32, 64);
                }
                tot = (h[0] + h[2]) + (h[1] + h[3]);
            }
            if (FULL || (lane < 32 && mi * 32 + m < rows && cols > 0)) part[wm * 64 + mi * 32 + m] = tot;
            dir_strip_sync();
#pragma unroll
            for (int b = 0; b < NOUT; ++b)
                dir_flush<64, !FULL, false>(strip, 16 * b, out[b] + base + (size_t)(mi * 32) * f, f, rows - mi * 32, cols);
            dir_strip_sync();
        }
    }
}

}  // namespace xmoe

#undef XMOE_LDS_PTR
#undef XMOE_GLB_PTR
