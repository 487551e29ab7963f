// A GEMM tile on the matrix cores for any shape, stride and alignment, in float32 (v_mfma_f32_32x32x2_f32: float32
// products and sums, nothing is split or rounded to fewer bits) and in bf16 (v_mfma_f32_32x32x16_bf16, float32
// accumulators).  It serves the float32 workloads and the bf16 shapes whose d or f is no multiple of 64, for which
// the direct-to-LDS kernels have no loads.
//
//   BIG:   128 x 128 outputs, 256 threads = 4 waves (2 x 2), wave tile 64 x 64, 64 KiB of LDS: two blocks per CU
//   small:  64 x  64 outputs, 128 threads = 2 waves (2 x 1), wave tile 32 x 64, 32 KiB of LDS
//
// K is stepped by 128 bytes (32 floats or 64 bf16).  Both operand tiles lie in LDS as [row or column][128 bytes of k],
// so one 16-byte LDS read is a fragment for either type: four consecutive k for four float32 MFMAs, eight for one
// bf16 MFMA.  The next step's operands travel global -> registers while the matrix instructions run and are written to
// the other half of the LDS buffer behind them, one barrier per step.  An operand that is K-strided in memory is
// transposed in registers on the way (4 x 4 floats are renamed, 8 x 4 bf16 take 16 byte permutes).  Loads are declared
// with the alignment of one element; the hardware takes unaligned 16-byte loads at the rate of aligned ones but for the
// lines they straddle, so an odd leading dimension costs no scalar path.  Only a vector that crosses the end of K or
// of the columns is fetched element by element.
//
// Bound: float32 by the matrix cores (a K-step is 4096 clocks of them per wave, against about 2000 for the latency of
// its loads), busy 52 to 64 % of a launch whose blocks fill 1.2 to 1.7 of two waves per SIMD on average (dAct, with the
// activation's loads and stores behind it, 39 %); bf16 by that latency (512 clocks of matrix work per step and wave): 39 to
// 53 % of a wave's time is waits, the matrix cores are busy 9 to 15 %.
#pragma once

#include "xmoe_internal.h"

namespace xmoe {

typedef __attribute__((ext_vector_type(16))) float tile_f32x16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 tile_bf16x8_t;

template <bool BIG>
struct TileShape {
    static constexpr int kM = BIG ? 128 : 64, kN = BIG ? 128 : 64;
    static constexpr int kThreads = BIG ? 256 : 128;
    static constexpr int kMI = BIG ? 2 : 1;                     // 32-row blocks per wave
    static constexpr int kBufBytes = (kM + kN) * 128;
    static constexpr int kLds = 2 * kBufBytes;
};

template <typename T>
struct TileElem;
template <>
struct TileElem<float> {
    static constexpr int kV = 4, kK = 32;                       // elements per 16 bytes, k per step
};
template <>
struct TileElem<bf16_t> {
    static constexpr int kV = 8, kK = 64;
};

// 16 (8) bytes from an address that is aligned to one element only
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) Packed16 {
    uint32_t v[4];
};
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) Packed8 {
    uint32_t v[2];
};

__device__ __forceinline__ uint32_t elem_bits(const float* p) { return __float_as_uint(*p); }
__device__ __forceinline__ uint32_t elem_bits(const bf16_t* p) { return p->bits; }

// byte address of 16-byte chunk c (0..7) of row (or column) r in a tile: eight consecutive rows at one chunk and eight
// rows four apart at one chunk (the fragment reads, and the writes of a transposed operand) fall on all banks
__device__ __forceinline__ int tile_addr(int r, int c) { return r * 128 + ((c ^ ((r ^ (r >> 3)) & 7)) << 4); }

// ---- K-contiguous operand: element (r, k) at base + row(r)*ld + k; rows past the last valid one repeat it (the outputs
// they feed are never stored), k past K reads zero
template <typename T, int NT>
struct RowSrc {
    static constexpr int kV = TileElem<T>::kV, kK = TileElem<T>::kK;
    const T* p[4];
    uint32_t s[4][4];
    // n_valid >= 1 rows; index: row r of the tile is row index[r] of the matrix (index points at the tile's first row)
    __device__ __forceinline__ void init(const T* base, size_t ld, int n_valid, const int32_t* index) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int r = (int)(threadIdx.x >> 3) + (NT / 8) * i;
            r = r < n_valid ? r : n_valid - 1;
            if (index) r = index[r];
            p[i] = base + (size_t)r * ld + (threadIdx.x & 7) * kV;
        }
    }
    __device__ __forceinline__ bool wide() const { return true; }
    __device__ __forceinline__ void load_full(int k0, int) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Packed16<T> q = *reinterpret_cast<const Packed16<T>*>(p[i] + k0);
#pragma unroll
            for (int j = 0; j < 4; ++j) s[i][j] = q.v[j];
        }
    }
    __device__ __forceinline__ void load_tail(int k0, int K) {
        const int n = K - k0 - (int)(threadIdx.x & 7) * kV;   // valid elements of this thread's chunks
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) s[i][j] = 0;
            if (n >= kV) {
                const Packed16<T> q = *reinterpret_cast<const Packed16<T>*>(p[i] + k0);
#pragma unroll
                for (int j = 0; j < 4; ++j) s[i][j] = q.v[j];
            } else {
#pragma unroll
                for (int j = 0; j < kV - 1; ++j)
                    if (j < n) s[i][j * 4 / kV] |= elem_bits(p[i] + k0 + j) << (kV == 8 ? 16 * (j & 1) : 0);
            }
        }
    }
    __device__ __forceinline__ void store(char* tile) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = (threadIdx.x >> 3) + (NT / 8) * i;
            *reinterpret_cast<uint4*>(tile + tile_addr(r, threadIdx.x & 7)) =
                make_uint4(s[i][0], s[i][1], s[i][2], s[i][3]);
        }
    }
};

// ---- K-strided operand: element (k, n) at base + row(k)*ld + n, ld columns in all.  A thread owns kV k-rows x 4
// columns; k past K reads zero.  Columns past the last one feed outputs that are never stored, so what they read only
// has to lie in the matrix: a thread whose four columns straddle the end reads the last four and moves them down before
// they go to LDS, one that lies past it reads the tile's first columns.
template <typename T, int NT, bool GATHER>
struct ColSrc {
    static constexpr int kV = TileElem<T>::kV, kK = TileElem<T>::kK;
    static constexpr int kNB = NT == 256 ? 32 : 16;   // 4-column blocks of the tile
    const T* base;       // already at this thread's columns
    size_t ld;
    const int32_t* index;   // GATHER: k-row k is row index[k] of the matrix
    int shift;           // columns the loaded four lie before the thread's own
    int n_valid;         // of this thread's four columns (used where ld < 4 only)
    int row[GATHER ? kV : 1];   // GATHER: the source rows of the next load
    uint32_t s[16];
    // cols >= 1: columns from p0 on.  Two matrices side by side (p1 != NULL): columns [0, TN/2) from p0, the others from p1
    __device__ __forceinline__ void init(const T* p0, const T* p1, size_t ld_, int cols, const int32_t* index_, int K) {
        int n = (int)(threadIdx.x % kNB) * 4;
        base = p0;
        if (p1 && n >= 2 * kNB) {
            n -= 2 * kNB;
            base = p1;
        }
        n_valid = cols - n;
        ld = ld_;
        if (n_valid <= 0 && wide()) {
            n = 0;
            n_valid = cols;
        }
        shift = n_valid < 4 && wide() ? 4 - n_valid : 0;
        base += n - shift;
        index = index_;
        if (GATHER && K > 0) fetch_rows(0, K);
    }
    __device__ __forceinline__ bool wide() const { return ld >= 4; }   // block-uniform
    __device__ __forceinline__ void fetch_rows(int k0, int K) {
        const int k = k0 + (int)(threadIdx.x / kNB) * kV;
#pragma unroll
        for (int q = 0; q < kV; ++q) row[q] = index[k + q < K ? k + q : K - 1];
    }
    __device__ __forceinline__ void load4(int q, const T* p) {
        if (kV == 4) {
            const Packed16<T> v = *reinterpret_cast<const Packed16<T>*>(p);
#pragma unroll
            for (int c = 0; c < 4; ++c) s[q * 4 + c] = v.v[c];
        } else {
            const Packed8<T> v = *reinterpret_cast<const Packed8<T>*>(p);
            s[q * 2] = v.v[0];
            s[q * 2 + 1] = v.v[1];
        }
    }
    // a whole step of a wide matrix: no branch, so all of a step's loads are in flight together
    __device__ __forceinline__ void load_full(int k0, int K) {
        const T* p = base + (size_t)(k0 + (int)(threadIdx.x / kNB) * kV) * ld;
#pragma unroll
        for (int q = 0; q < kV; ++q) load4(q, GATHER ? base + (size_t)row[GATHER ? q : 0] * ld : p + q * ld);
        if (GATHER) fetch_rows(k0 + kK, K);
    }
    __device__ __forceinline__ void load_tail(int k0, int K) {
        const int k = k0 + (int)(threadIdx.x / kNB) * kV;
        const T* p = base + (size_t)k * ld;
#pragma unroll
        for (int j = 0; j < 16; ++j) s[j] = 0;
#pragma unroll
        for (int q = 0; q < kV; ++q) {
            if (k + q >= K) continue;
            const T* pr = GATHER ? base + (size_t)row[GATHER ? q : 0] * ld : p + q * ld;
            if (wide()) {
                load4(q, pr);
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (c < n_valid)
                        s[kV == 4 ? q * 4 + c : q * 2 + (c >> 1)] |= elem_bits(pr + c) << (kV == 8 ? 16 * (c & 1) : 0);
            }
        }
        if (GATHER) fetch_rows(k0 + kK, K);
    }
    __device__ __forceinline__ void unshift() {
        if (shift == 0) return;
        // two steps of constant moves: a choice by `shift` itself would index the registers and put them in memory
        const bool by1 = shift & 1, by2 = shift & 2;
#pragma unroll
        for (int q = 0; q < kV; ++q) {
            if (kV == 4) {
                s[q * 4] = by1 ? s[q * 4 + 1] : s[q * 4];
                s[q * 4 + 1] = by1 ? s[q * 4 + 2] : s[q * 4 + 1];
                s[q * 4 + 2] = by1 ? s[q * 4 + 3] : s[q * 4 + 2];
                s[q * 4] = by2 ? s[q * 4 + 2] : s[q * 4];
                s[q * 4 + 1] = by2 ? s[q * 4 + 3] : s[q * 4 + 1];
            } else {
                const uint64_t v = (((uint64_t)s[q * 2 + 1] << 32) | s[q * 2]) >> (16 * shift);
                s[q * 2] = (uint32_t)v;
                s[q * 2 + 1] = (uint32_t)(v >> 32);
            }
        }
    }
    __device__ __forceinline__ void store(char* tile) {
        unshift();
        const int c = threadIdx.x / kNB, n = (threadIdx.x % kNB) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t v[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                if (kV == 4)
                    v[a] = s[a * 4 + j];
                else   // the low (even column) or high halves of k-rows 2a and 2a+1
                    v[a] = __builtin_amdgcn_perm(s[(2 * a + 1) * 2 + (j >> 1)], s[2 * a * 2 + (j >> 1)],
                                                 (j & 1) ? 0x07060302u : 0x05040100u);
            }
            *reinterpret_cast<uint4*>(tile + tile_addr(n + j, c)) = make_uint4(v[0], v[1], v[2], v[3]);
        }
    }
};

// acc[mi][ni] += a[mi] b[ni] over the fragments' k.  Consecutive matrix instructions go to different accumulators.
template <int MI, int N>
__device__ __forceinline__ void tile_mma(tile_f32x16_t (&acc)[N][2], const uint4 (&a)[MI], const uint4 (&b)[2],
                                         const float*) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) {
                const uint32_t av[4] = {a[mi].x, a[mi].y, a[mi].z, a[mi].w};
                const uint32_t bv[4] = {b[ni].x, b[ni].y, b[ni].z, b[ni].w};
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av[j]), __uint_as_float(bv[j]),
                                                                   acc[mi][ni], 0, 0, 0);
            }
}
template <int MI, int N>
__device__ __forceinline__ void tile_mma(tile_f32x16_t (&acc)[N][2], const uint4 (&a)[MI], const uint4 (&b)[2],
                                         const bf16_t*) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(tile_bf16x8_t, a[mi]),
                                                                  __builtin_bit_cast(tile_bf16x8_t, b[ni]),
                                                                  acc[mi][ni], 0, 0, 0);
}

// Where a lane's accumulators lie: acc[mi][ni][v] is output (tile_row(mi, v), tile_col(ni)) of the block's tile.
// DUAL: the wave's two column blocks are the same columns of two matrices side by side, tile_col<true>(0) of either.
template <bool BIG>
__device__ __forceinline__ int tile_row(int mi, int v) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    return (BIG ? (wave >> 1) * 64 : wave * 32) + mi * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
}
template <bool BIG, bool DUAL>
__device__ __forceinline__ int tile_col_base(int ni) {
    const int wn = BIG ? (threadIdx.x >> 6) & 1 : 0;
    return DUAL ? ni * (TileShape<BIG>::kN / 2) + wn * 32 : wn * 64 + ni * 32;
}
template <bool BIG, bool DUAL>
__device__ __forceinline__ int tile_col(int ni) { return tile_col_base<BIG, DUAL>(ni) + (int)(threadIdx.x & 31); }

// one K-step of the first MI 32-row blocks of the wave; k: valid k of the step, behind which there are zeros only
template <typename T, bool BIG, bool DUAL, int MI, int N>
__device__ __forceinline__ void tile_compute(tile_f32x16_t (&acc)[N][2], const char* ta, const char* tb,
                                             int k = TileElem<T>::kK) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ra = (BIG ? (wave >> 1) * 64 : wave * 32) + (lane & 31);
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        if (st * 2 * TileElem<T>::kV >= k) break;
        const int c = 2 * st + (lane >> 5);
        uint4 fa[MI], fb[2];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) fa[mi] = *reinterpret_cast<const uint4*>(ta + tile_addr(ra + mi * 32, c));
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
            fb[ni] = *reinterpret_cast<const uint4*>(tb + tile_addr(tile_col<BIG, DUAL>(ni), c));
        tile_mma<MI, N>(acc, fa, fb, (const T*)nullptr);
    }
}

// acc += A B over K; smem holds TileShape<BIG>::kLds bytes; rows, cols: valid ones of the tile (may exceed it).  Every
// thread of the block calls it.  A wave multiplies only its 32-row blocks that hold a valid row, and nothing if no
// column of its is valid: a partly filled tile then costs the matrix cores what it holds.  RAGGED: K is a row count, and
// the last step multiplies only what there is of it (float32, 1 row per expert, d 1024 f 704 E 17: the whole backward
// 149 -> 138 us; the row products, whose K is a width, are 1 to 2 % slower with it).
template <typename T, bool BIG, bool DUAL, bool RAGGED, class SrcA, class SrcB>
__device__ __forceinline__ void tile_mainloop(tile_f32x16_t (&acc)[TileShape<BIG>::kMI][2], int K, int rows, int cols,
                                              SrcA& a, SrcB& b, char* smem) {
    constexpr int MI = TileShape<BIG>::kMI, kK = TileElem<T>::kK, kBuf = TileShape<BIG>::kBufBytes;
    constexpr int kBOff = TileShape<BIG>::kM * 128;
    if (K <= 0) return;   // block-uniform
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wcol = BIG ? (wave & 1) * (DUAL ? 32 : 64) : 0;
    const int mi_n = cols > wcol ? (rows - (BIG ? (wave >> 1) * 64 : wave * 32) + 31) / 32 : 0;
    auto compute = [&](int i, int k) {
        const char* t = smem + (i & 1) * kBuf;
        if (mi_n >= MI)
            tile_compute<T, BIG, DUAL, MI>(acc, t, t + kBOff, k);
        else if (MI == 2 && mi_n == 1)
            tile_compute<T, BIG, DUAL, 1>(acc, t, t + kBOff, k);
    };
    auto store = [&](int i) {   // into the half that was last read before the previous step's barrier
        a.store(smem + (i & 1) * kBuf);
        b.store(smem + (i & 1) * kBuf + kBOff);
        __syncthreads();
    };
    const int n = (K + kK - 1) / kK, n_full = a.wide() && b.wide() ? K / kK : 0;
    if (n_full > 0) {
        a.load_full(0, K);
        b.load_full(0, K);
    } else {
        a.load_tail(0, K);
        b.load_tail(0, K);
    }
    __syncthreads();      // a previous loop's last reads of the buffer
    store(0);
    int i = 0;
    for (; i + 1 < n_full; ++i) {
        a.load_full((i + 1) * kK, K);
        b.load_full((i + 1) * kK, K);
        compute(i, kK);
        store(i + 1);
    }
    for (; i + 1 < n; ++i) {
        a.load_tail((i + 1) * kK, K);
        b.load_tail((i + 1) * kK, K);
        compute(i, kK);
        store(i + 1);
    }
    compute(i, RAGGED ? K - i * kK : kK);
}

template <bool BIG>
__device__ __forceinline__ void tile_zero(tile_f32x16_t (&acc)[TileShape<BIG>::kMI][2]) {
#pragma unroll
    for (int mi = 0; mi < TileShape<BIG>::kMI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
}

// Sums part[v] over the 32 lanes of each half-wave by halving (a fixed order); lane l then holds the sum of
// v = (l/2) % 16.  One call per step: a loop over the halving width is left rolled by the compiler, and its indexing
// puts the array in memory (16 KiB of LDS per 256-thread block).
template <int W>
__device__ __forceinline__ void tile_fold(float (&part)[16]) {
    const bool upper = (threadIdx.x & (2 * W)) != 0;
#pragma unroll
    for (int v = 0; v < W; ++v) {
        const float send = upper ? part[v] : part[v + W];
        const float keep = upper ? part[v + W] : part[v];
        part[v] = keep + __shfl_xor(send, 2 * W, 64);
    }
}
__device__ __forceinline__ float tile_sum_over_cols(float (&part)[16]) {
    tile_fold<8>(part);
    tile_fold<4>(part);
    tile_fold<2>(part);
    tile_fold<1>(part);
    return part[0] + __shfl_xor(part[0], 1, 64);
}

}  // namespace xmoe
