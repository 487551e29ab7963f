// A GEMM tile on the matrix cores for any shape, stride and alignment, in float32 and in bf16, with float32 accumulators.
// It serves the float32 workloads and the bf16 shapes for which the direct-to-LDS kernels have no loads (d or f no multiple
// of 8, operands not 16-byte aligned) or are the slower ones (weight gradients of few rows per expert).
//
//   BIG:   128 x 128 outputs, 256 threads = 4 waves (2 x 2), wave tile 64 x 64, 64 KiB of LDS: two blocks per CU
//   small:  64 x  64 outputs, 128 threads = 2 waves (2 x 1), wave tile 32 x 64, 32 KiB of LDS
//
// The matrix instruction is v_mfma_f32_32x32x16_bf16 for both types.  A float is the exact sum of three bf16 numbers (hi +
// mid + lo, 8 bits each; the splitting of G. Henry, P. Tang, A. Heinecke, "Leveraging the bfloat16 artificial intelligence
// datatype for higher-precision computations", 2019), a product of two floats the sum of nine products of bf16 numbers, each
// exact in float32.  Six of them take 192 clocks of the matrix cores per 16 k, where the float32 instruction
// (v_mfma_f32_32x32x2_f32) takes 512.  Left out are lo x lo, at most 2^-32 of the whole, and mid x lo and lo x mid, 2^-23
// each at worst and 2^-26 on average: up to four times what a float32 product rounds off.  What makes up for it is that a sum
// has an eighth of a float32 chain's roundings: per 16 k, hi x hi is added to it once and the five small products once,
// summed among themselves before (added one by one they would each be cut off at the sum's last bit: this instruction
// truncates).  Sums of up to kPlainK terms, which would lose by it, are the float32 instruction's.  Error against float64,
// rms in 2^-24 of the sum of the terms' magnitudes, float32 instruction | this, for normal operands and for operands just
// above 1 whose mid and lo are the largest: K 10 0.46 | 0.29 and 0.93 | 0.68, K 17 0.47 | 0.30 and 1.11 | 0.85, K 64 0.47 |
// 0.21 and 1.81 | 1.07, K 1024 0.47 | 0.19 and 30.8 | 1.98; training steps 1.2e-6 -> 0.5e-6 and 4.0e-7 -> 2.5e-7.
// The parts are taken of 2^24 times each operand, so that the bits of the smallest floats too are parts in bf16's normal
// range, and a sum is multiplied by 2^-48 at its end: both exact but for results below 2^-126.  What is not finite then (an
// infinity or an operand from 2^104 on has no finite parts, a sum from 2^80 on overflows) is computed again from the floats
// themselves (tile_finish).
//
// K is stepped by 64 bf16 (both operand tiles lie in LDS as [row or column][128 bytes of k]) or 16 floats ([row or
// column][three parts of 32 bytes]), so that one 16-byte LDS read is a fragment of a matrix instruction.  The operands
// travel global -> registers, two steps ahead for float32 and one for bf16 (whose steps are four times as many
// registers), while the matrix instructions run, and are written to the other half of the LDS buffer behind them (float32:
// split on the way, once per element of the tile), one barrier per step.  An operand that is K-strided in memory is
// transposed in registers on the way.  Loads are declared with the alignment of one element; the hardware takes unaligned
// 16-byte loads at the rate of aligned ones but for the lines they straddle, so an odd leading dimension costs no scalar
// path.  Only a vector that crosses the end of K or of the columns is fetched element by element.
//
// Bound: float32 by the matrix cores and the vector instructions of the split and of the small products' sums between them
// (gate/up of T 2048, d 1024, f 704, 16 experts + 1: 344 -> 201 us, the matrix cores busy 40 % of it); float32 with few tiles
// and K up to 256 by the chain of a step (T 256 d 128 f 64, 8 experts, whole step: 89 us with the float32 instruction, 94
// now); bf16 by latency (512 clocks of matrix work per step and wave, 44 % of a wave's time is waits, the matrix cores are
// busy 15 %).
#pragma once

#include <type_traits>

#include "xmoe_internal.h"

namespace xmoe {

typedef __attribute__((ext_vector_type(16))) float tile_f32x16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 tile_bf16x8_t;

template <bool BIG>
struct TileShape {
    static constexpr int kM = BIG ? 128 : 64, kN = BIG ? 128 : 64;
    static constexpr int kThreads = BIG ? 256 : 128;
    static constexpr int kMI = BIG ? 2 : 1;                     // 32-row blocks per wave
    static constexpr int kLds = 2 * (kM + kN) * 128;
};

template <typename T>
struct TileElem;
template <>
struct TileElem<float> {
    static constexpr int kV = 4, kK = 16;                       // elements per 16 bytes, k per step
    static constexpr int kRowBytes = 96;                        // of a tile row in LDS
    static constexpr int kColK = 4, kColN = 2;                  // a thread's k-rows and columns of a K-strided operand
    static constexpr int kSets = 2;                             // steps on their way in registers
};
template <>
struct TileElem<bf16_t> {
    static constexpr int kV = 8, kK = 64;
    static constexpr int kRowBytes = 128;
    static constexpr int kColK = 8, kColN = 4;
    static constexpr int kSets = 1;
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

// bf16: byte address of 16-byte chunk c (0..7) of row (or column) r in a tile: eight consecutive rows at one chunk and
// eight rows four apart at one chunk (the fragment reads, and the writes of a transposed operand) fall on all banks
__device__ __forceinline__ int tile_addr(int r, int c) { return r * 128 + ((c ^ ((r ^ (r >> 3)) & 7)) << 4); }
// float32: byte address of chunk c (0..1: eight k) of part p (0..2) of row r
__device__ __forceinline__ int split_addr(int r, int p, int c) {
    return r * 96 + p * 32 + ((c ^ (((r >> 2) ^ (r >> 3)) & 1)) << 4);
}

// The three bf16 parts of four floats, x kPartScale = hi + mid + lo exactly (8 bits each; hi is cut off, mid and lo are
// rounded to nearest); kUnscale takes the scales of a product's operands off
constexpr float kPartScale = 0x1p24f, kUnscale = 0x1p-48f;
__device__ __forceinline__ void split4(const uint32_t (&x)[4], uint2 (&part)[3]) {
    uint32_t h[2], m[2], l[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t a = __float_as_uint(__uint_as_float(x[2 * i]) * kPartScale);
        const uint32_t b = __float_as_uint(__uint_as_float(x[2 * i + 1]) * kPartScale);
        h[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);
        const float ra = __uint_as_float(a) - __uint_as_float(a & 0xffff0000u);
        const float rb = __uint_as_float(b) - __uint_as_float(b & 0xffff0000u);
        m[i] = pack_bf16x2(ra, rb);
        l[i] = pack_bf16x2(ra - __uint_as_float(m[i] << 16), rb - __uint_as_float(m[i] & 0xffff0000u));
    }
    part[0] = make_uint2(h[0], h[1]);
    part[1] = make_uint2(m[0], m[1]);
    part[2] = make_uint2(l[0], l[1]);
}

// ---- K-contiguous operand: element (r, k) at base + row(r)*ld + k; rows past the last valid one repeat it (the outputs
// they feed are never stored), k past K reads zero.  Two sets of registers: two steps of the operand are on their way.
template <typename T, int NT>
struct RowSrc {
    static constexpr int kV = TileElem<T>::kV, kK = TileElem<T>::kK;
    static constexpr int kC = kK / kV;                           // chunks of a row
    static constexpr int kP = (NT == 256 ? 128 : 64) * kC / NT;  // rows per thread
    const T* p[kP];
    uint32_t s[TileElem<T>::kSets][kP][4];
    // n_valid >= 1 rows; index: row r of the tile is row index[r] of the matrix (index points at the tile's first row)
    __device__ __forceinline__ void init(const T* base, size_t ld, int n_valid, const int32_t* index) {
#pragma unroll
        for (int i = 0; i < kP; ++i) {
            int r = (int)(threadIdx.x / kC) + (NT / kC) * i;
            r = r < n_valid ? r : n_valid - 1;
            if (index) r = index[r];
            p[i] = base + (size_t)r * ld + (threadIdx.x % kC) * kV;
        }
    }
    __device__ __forceinline__ bool wide() const { return true; }
    __device__ __forceinline__ void advance(int, int) {}
    template <int S>
    __device__ __forceinline__ void load_full(int k0) {
#pragma unroll
        for (int i = 0; i < kP; ++i) {
            const Packed16<T> q = *reinterpret_cast<const Packed16<T>*>(p[i] + k0);
#pragma unroll
            for (int j = 0; j < 4; ++j) s[S][i][j] = q.v[j];
        }
    }
    template <int S>
    __device__ __forceinline__ void load_tail(int k0, int K) {
        const int n = K - k0 - (int)(threadIdx.x % kC) * kV;   // valid elements of this thread's chunks
#pragma unroll
        for (int i = 0; i < kP; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) s[S][i][j] = 0;
            if (n >= kV) {
                const Packed16<T> q = *reinterpret_cast<const Packed16<T>*>(p[i] + k0);
#pragma unroll
                for (int j = 0; j < 4; ++j) s[S][i][j] = q.v[j];
            } else {
#pragma unroll
                for (int j = 0; j < kV - 1; ++j)
                    if (j < n) s[S][i][j * 4 / kV] |= elem_bits(p[i] + k0 + j) << (kV == 8 ? 16 * (j & 1) : 0);
            }
        }
    }
    template <int S>
    __device__ __forceinline__ void store(char* tile) {
#pragma unroll
        for (int i = 0; i < kP; ++i) {
            const int r = threadIdx.x / kC + (NT / kC) * i, c = threadIdx.x % kC;
            if (kV == 8) {
                *reinterpret_cast<uint4*>(tile + tile_addr(r, c)) =
                    make_uint4(s[S][i][0], s[S][i][1], s[S][i][2], s[S][i][3]);
            } else {
                uint2 part[3];
                split4(s[S][i], part);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uint2*>(tile + split_addr(r, q, c >> 1) + (c & 1) * 8) = part[q];
            }
        }
    }
};

// ---- K-strided operand: element (k, n) at base + row(k)*ld + n, ld columns in all.  A thread owns kColK k-rows x kColN
// columns (8 bytes of a row); k past K reads zero.  Columns past the last one feed outputs that are never stored, so what
// they read only has to lie in the matrix: a thread whose columns straddle the end reads the last kColN and moves them
// down before they go to LDS, one that lies past it reads the tile's first columns.
template <typename T, int NT, bool GATHER>
struct ColSrc {
    static constexpr int kQ = TileElem<T>::kColK, kC = TileElem<T>::kColN, kK = TileElem<T>::kK;
    static constexpr int kNB = (NT == 256 ? 128 : 64) / kC;   // column blocks of the tile
    const T* base;       // already at this thread's columns
    size_t ld;
    const int32_t* index;   // GATHER: k-row k is row index[k] of the matrix
    int shift;           // columns the loaded ones lie before the thread's own
    int n_valid;         // of this thread's columns (used where ld < kC only)
    int row[GATHER ? kQ : 1], next_row[GATHER ? kQ : 1];   // GATHER: the source rows of this load and of the next one
    uint32_t s[TileElem<T>::kSets][2 * kQ];
    // The thread's column block and group of k-rows.  bf16: consecutive threads take consecutive blocks.  float32: the
    // two groups of a 16-byte chunk alternate between eight blocks, so that 16 lanes' 8-byte writes fall on all banks.
    static __device__ __forceinline__ int block() {
        const int t = threadIdx.x;
        if (kC == 4) return t % kNB;
        return (t & 7) | (t >> 1 & (kNB - 8));
    }
    static __device__ __forceinline__ int group() {
        const int t = threadIdx.x;
        if (kC == 4) return t / kNB;
        return (t >> 3 & 1) | (t / (2 * kNB)) << 1;
    }
    // cols >= 1: columns from p0 on.  Two matrices side by side (p1 != NULL): columns [0, TN/2) from p0, the others from p1
    __device__ __forceinline__ void init(const T* p0, const T* p1, size_t ld_, int cols, const int32_t* index_, int K) {
        int n = block() * kC;
        base = p0;
        if (p1 && n >= kNB * kC / 2) {
            n -= kNB * kC / 2;
            base = p1;
        }
        n_valid = cols - n;
        ld = ld_;
        if (n_valid <= 0 && wide()) {
            n = 0;
            n_valid = cols;
        }
        shift = n_valid < kC && wide() ? kC - n_valid : 0;
        base += n - shift;
        index = index_;
        if (GATHER && K > 0) fetch_rows(0, K);
    }
    // before the load of the step at k0: its source rows have arrived, the next step's are requested, ahead of the step's
    // own loads (the next step then waits for these and no newer ones before it forms its addresses)
    __device__ __forceinline__ void advance(int k0, int K) {
        if (!GATHER) return;
#pragma unroll
        for (int q = 0; q < kQ; ++q) row[GATHER ? q : 0] = next_row[GATHER ? q : 0];
        fetch_rows(k0 + kK, K);
    }
    __device__ __forceinline__ bool wide() const { return ld >= kC; }   // block-uniform
    __device__ __forceinline__ void fetch_rows(int k0, int K) {
        const int k = k0 + group() * kQ;
#pragma unroll
        for (int q = 0; q < kQ; ++q) next_row[GATHER ? q : 0] = index[k + q < K ? k + q : K - 1];
    }
    template <int S>
    __device__ __forceinline__ void load_row(int q, const T* p) {
        const Packed8<T> v = *reinterpret_cast<const Packed8<T>*>(p);
        s[S][q * 2] = v.v[0];
        s[S][q * 2 + 1] = v.v[1];
    }
    // a whole step of a wide matrix: no branch, so all of a step's loads are in flight together
    template <int S>
    __device__ __forceinline__ void load_full(int k0) {
        const T* p = base + (size_t)(k0 + group() * kQ) * ld;
#pragma unroll
        for (int q = 0; q < kQ; ++q) load_row<S>(q, GATHER ? base + (size_t)row[GATHER ? q : 0] * ld : p + q * ld);
    }
    template <int S>
    __device__ __forceinline__ void load_tail(int k0, int K) {
        const int k = k0 + group() * kQ;
        const T* p = base + (size_t)k * ld;
#pragma unroll
        for (int j = 0; j < 2 * kQ; ++j) s[S][j] = 0;
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            if (k + q >= K) continue;
            const T* pr = GATHER ? base + (size_t)row[GATHER ? q : 0] * ld : p + q * ld;
            if (wide()) {
                load_row<S>(q, pr);
            } else {
#pragma unroll
                for (int c = 0; c < kC - 1; ++c)
                    if (c < n_valid) s[S][q * 2 + c * 2 / kC] |= elem_bits(pr + c) << (kC == 4 ? 16 * (c & 1) : 0);
            }
        }
    }
    template <int S>
    __device__ __forceinline__ void store(char* tile) {
        if (shift != 0) {
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const uint64_t v = (((uint64_t)s[S][q * 2 + 1] << 32) | s[S][q * 2]) >> (8 * sizeof(T) * shift);
                s[S][q * 2] = (uint32_t)v;
                s[S][q * 2 + 1] = (uint32_t)(v >> 32);
            }
        }
        const int c = group(), n = block() * kC;
#pragma unroll
        for (int j = 0; j < kC; ++j) {
            uint32_t v[4];
            if (kC == 4) {   // the low (even column) or high halves of k-rows 2a and 2a+1
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    v[a] = __builtin_amdgcn_perm(s[S][((2 * a + 1) * 2 + (j >> 1)) % (2 * kQ)],
                                                 s[S][(2 * a * 2 + (j >> 1)) % (2 * kQ)],
                                                 (j & 1) ? 0x07060302u : 0x05040100u);
                *reinterpret_cast<uint4*>(tile + tile_addr(n + j, c)) = make_uint4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int a = 0; a < 4; ++a) v[a] = s[S][a * 2 + j];
                uint2 part[3];
                split4(v, part);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uint2*>(tile + split_addr(n + j, q, c >> 1) + (c & 1) * 8) = part[q];
            }
        }
    }
};

__device__ __forceinline__ tile_f32x16_t tile_mfma(const uint4& a, const uint4& b, const tile_f32x16_t& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(tile_bf16x8_t, a),
                                                   __builtin_bit_cast(tile_bf16x8_t, b), c, 0, 0, 0);
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

// One K-step of the first MI 32-row blocks of the wave; k: valid k of the step, behind which there are zeros only.
// Consecutive matrix instructions go to different accumulators.
template <bool BIG, bool DUAL, int MI, int N>
__device__ __forceinline__ void tile_compute(tile_f32x16_t (&acc)[N][2], const char* ta, const char* tb, int k) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ra = (BIG ? (wave >> 1) * 64 : wave * 32) + (lane & 31);
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        if (st * 16 >= k) break;
        const int c = 2 * st + (lane >> 5);
        uint4 fa[MI], fb[2];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) fa[mi] = *reinterpret_cast<const uint4*>(ta + tile_addr(ra + mi * 32, c));
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
            fb[ni] = *reinterpret_cast<const uint4*>(tb + tile_addr(tile_col<BIG, DUAL>(ni), c));
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = tile_mfma(fa[mi], fb[ni], acc[mi][ni]);
    }
}
// float32: six products of the parts in ascending size, hi x hi into the sum, the others among themselves and then into the
// sum
template <bool BIG, bool DUAL, int MI, int N>
__device__ __forceinline__ void tile_compute_split(tile_f32x16_t (&acc)[N][2], const char* ta, const char* tb) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane >> 5;
    const int ra = (BIG ? (wave >> 1) * 64 : wave * 32) + (lane & 31);
    uint4 fb[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
            fb[ni][p] = *reinterpret_cast<const uint4*>(tb + split_addr(tile_col<BIG, DUAL>(ni), p, c));
    constexpr int kPa[5] = {0, 2, 1, 0, 1}, kPb[5] = {2, 0, 1, 1, 0};
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        uint4 fa[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) fa[p] = *reinterpret_cast<const uint4*>(ta + split_addr(ra + mi * 32, p, c));
        tile_f32x16_t x[2];
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) x[ni][v] = 0.f;
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) x[ni] = tile_mfma(fa[kPa[t]], fb[ni][kPb[t]], x[ni]);
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = tile_mfma(fa[0], fb[ni][0], acc[mi][ni]);
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] += x[ni][v];
    }
}

// Sums of up to this many terms are float32's own: in them the products that are left out weigh as much as the roundings
constexpr int kPlainK = 8;

// acc += A B over K; smem holds TileShape<BIG>::kLds bytes; rows, cols: valid ones of the tile (may exceed it).  Every
// thread of the block calls it.  A wave multiplies only its 32-row blocks that hold a valid row, and nothing if no
// column of its is valid: a partly filled tile then costs the matrix cores what it holds.  RAGGED: K is a row count, and
// the last step multiplies only what there is of it.
template <typename T, bool BIG, bool DUAL, bool RAGGED, class SrcA, class SrcB>
__device__ __forceinline__ void tile_mainloop(tile_f32x16_t (&acc)[TileShape<BIG>::kMI][2], int K, int rows, int cols,
                                              SrcA& a, SrcB& b, char* smem) {
    constexpr int MI = TileShape<BIG>::kMI, kK = TileElem<T>::kK;
    constexpr int kBOff = TileShape<BIG>::kM * TileElem<T>::kRowBytes;
    constexpr int kBuf = kBOff + TileShape<BIG>::kN * TileElem<T>::kRowBytes;
    static_assert(2 * kBuf <= TileShape<BIG>::kLds, "two buffers");
    if (K <= (std::is_same<T, float>::value ? kPlainK : 0)) return;   // block-uniform; float32: tile_finish's sums
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wcol = BIG ? (wave & 1) * (DUAL ? 32 : 64) : 0;
    const int mi_n = cols > wcol ? (rows - (BIG ? (wave >> 1) * 64 : wave * 32) + 31) / 32 : 0;
    const int n = (K + kK - 1) / kK, n_full = a.wide() && b.wide() ? K / kK : 0;
    auto compute = [&](auto P, int k) {
        const char* t = smem + P.value * kBuf;
        auto blocks = [&](auto M) {
            if constexpr (std::is_same<T, float>::value)
                tile_compute_split<BIG, DUAL, M.value>(acc, t, t + kBOff);
            else
                tile_compute<BIG, DUAL, M.value>(acc, t, t + kBOff, k);
        };
        if (mi_n >= MI)
            blocks(std::integral_constant<int, MI>{});
        else if (MI == 2 && mi_n == 1)
            blocks(std::integral_constant<int, 1>{});
    };
    auto load_whole = [&](auto S, int i) {
        a.advance(i * kK, K);
        b.advance(i * kK, K);
        a.template load_full<S.value>(i * kK);
        b.template load_full<S.value>(i * kK);
    };
    auto load = [&](auto P, int i) {
        a.advance(i * kK, K);
        b.advance(i * kK, K);
        if (i < n_full) {
            a.template load_full<P.value>(i * kK);
            b.template load_full<P.value>(i * kK);
        } else {
            a.template load_tail<P.value>(i * kK, K);
            b.template load_tail<P.value>(i * kK, K);
        }
    };
    // register set S into buffer P, which was last read before the barrier of the step before
    auto store = [&](auto S, auto P) {
        a.template store<S.value>(smem + P.value * kBuf);
        b.template store<S.value>(smem + P.value * kBuf + kBOff);
        __syncthreads();
    };
    constexpr int kS1 = TileElem<T>::kSets - 1;   // the odd steps' register set
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, 1> P1{};
    constexpr std::integral_constant<int, kS1> S1{};
    load(P0, 0);
    if (kS1 && n > 1) load(S1, 1);
    __syncthreads();      // a previous loop's last reads of the buffers
    store(P0, P0);
    int i = 0;
    // Before step i its operands lie in buffer i % 2; with two sets those of step i + 1 are on their way to registers.
    // The loop over whole steps has no branch: the compiler then waits for the older of the two sets only.
    for (; i + 2 + kS1 < n_full; i += 2) {
        load_whole(P0, i + 1 + kS1);
        compute(P0, kK);
        store(S1, P1);
        load_whole(S1, i + 2 + kS1);
        compute(P1, kK);
        store(P0, P0);
    }
    for (; i < n; i += 2) {
        if (i + 1 + kS1 < n) load(P0, i + 1 + kS1);
        compute(P0, RAGGED ? K - i * kK : kK);
        if (i + 1 >= n) break;
        store(S1, P1);
        if (i + 2 + kS1 < n) load(S1, i + 2 + kS1);
        compute(P1, RAGGED ? K - (i + 1) * kK : kK);
        if (i + 2 < n) store(P0, P0);
    }
}

// float32: what stands between the sums of products of parts and the results: the parts' scale, the results that the parts
// lose, and sums of at most kPlainK terms.  The accumulators of a wave that holds an infinity or a NaN are summed again with
// the float32 instruction, straight from memory, and what is not finite takes what comes out: an infinity where the floats
// give one, NaN where they do.  Diverged data pays for it: the training step of T 2048, d 1024, f 704, 16 experts + 1 takes
// 1.15 ms, with one infinite weight 1.55, with a NaN for every gradient 3.2, for every weight 4.0 (with the float32
// instruction throughout 1.62 on any data).
// One operand: element (i, k) of the tile, i its row (of A) or column (of B), n of them valid.
struct PlainOp {
    const float* p;
    size_t stride_i, stride_k;
    const int32_t* index_i;
    const int32_t* index_k;
    int n;
    __device__ __forceinline__ float at(int i, int k) const {
        i = i < n ? i : n - 1;
        return p[(size_t)(index_i ? index_i[i] : i) * stride_i + (size_t)(index_k ? index_k[k] : k) * stride_k];
    }
    // k .. k + 3, zeros from K on
    __device__ __forceinline__ void four(int i, int k, int K, float (&v)[4]) const {
        if (stride_k == 1 && k + 4 <= K) {
            i = i < n ? i : n - 1;
            const Packed16<float> q =
                *reinterpret_cast<const Packed16<float>*>(p + (size_t)(index_i ? index_i[i] : i) * stride_i + k);
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = __uint_as_float(q.v[t]);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = k + t < K ? at(i, k + t) : 0.f;
        }
    }
};
struct PlainPair {
    PlainOp a, b;
};
// K <= kPlainK: acc += the product of the pair, its loads in flight together
template <bool BIG>
__device__ __forceinline__ void tile_plain(tile_f32x16_t (&acc)[TileShape<BIG>::kMI][2], int K, const PlainPair& q) {
    constexpr int MI = TileShape<BIG>::kMI, NT = kPlainK / 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float a[MI][NT], b[2][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int k = 2 * t + (lane >> 5);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) a[mi][t] = 0.f;
        b[0][t] = b[1][t] = 0.f;
        if (k >= K) continue;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            a[mi][t] = q.a.at((BIG ? (wave >> 1) * 64 : wave * 32) + mi * 32 + (lane & 31), k);
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) b[ni][t] = q.b.at(tile_col<BIG, false>(ni), k);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (2 * t >= K) break;   // both halves of the wave go on together
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mi][t], b[ni][t], acc[mi][ni], 0, 0, 0);
    }
}
// pairs(set, ni): the operands of product `set` of the sum; DUAL: b is the matrix of column block ni
template <bool BIG, bool DUAL, class Pairs>
__device__ __forceinline__ void tile_finish(tile_f32x16_t (&acc)[TileShape<BIG>::kMI][2], int K, int sets, Pairs&& pairs) {
    constexpr int MI = TileShape<BIG>::kMI;
    bool lost = K <= kPlainK;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) lost |= !(fabsf(acc[mi][ni][v]) < INFINITY);
    if (!__any(lost)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mi][ni][v] *= kUnscale;
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    tile_f32x16_t x[MI][2];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) x[mi][ni][v] = 0.f;
    for (int set = 0; set < sets; ++set)
        for (int k0 = 0; k0 < K; k0 += 8) {   // both halves of the wave go round together
            const int k = k0 + 4 * (lane >> 5);
            float a[MI][4], b[2][4];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                pairs(set, 0).a.four((BIG ? (wave >> 1) * 64 : wave * 32) + mi * 32 + (lane & 31), k, K, a[mi]);
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) pairs(set, ni).b.four(tile_col<BIG, DUAL>(DUAL ? 0 : ni), k, K, b[ni]);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni)
                        x[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mi][t], b[ni][t], x[mi][ni], 0, 0, 0);
        }
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float c = acc[mi][ni][v];
                acc[mi][ni][v] = K > kPlainK && fabsf(c) < INFINITY ? c * kUnscale : x[mi][ni][v];
            }
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

// A row GEMM's block: its row tile (expert and rows from the tile map) and column tile.  Blocks go to the XCDs in turn
// (block b to XCD b % 8); each XCD takes an eighth of the tiles there are, in one run.  An expert's tiles are numbered in
// bands of eight row tiles, down the rows of a band first: the blocks of an XCD then work on few experts at a time, and its
// L2 fetches a panel of weights once for the rows of a band and the rows once for all columns.
constexpr int kTileBand = 8;
struct RowTile {
    int e, row0, rows, col;   // rows: valid rows of the tile, may exceed the tile
    __device__ __forceinline__ bool init(const int32_t* __restrict__ off, const int32_t* __restrict__ map, int cols,
                                         int tile_rows) {
        const int total = map[0] * cols, per = (total + 7) / 8, s = blockIdx.x >> 3;
        const int t = (blockIdx.x & 7) * per + s;
        if (s >= per || t >= total) return false;
        const int i = t / cols;
        e = map[4 + 2 * i];
        const int lo = off[e], hi = off[e + 1];
        const int first = i - (map[4 + 2 * i + 1] - lo) / tile_rows;   // the expert's first row tile
        const int tiles = (hi - lo + tile_rows - 1) / tile_rows;
        const int u = t - first * cols, band = u / (kTileBand * cols), v = u - band * kTileBand * cols;
        const int in_band = tiles - band * kTileBand < kTileBand ? tiles - band * kTileBand : kTileBand;
        col = v / in_band;
        row0 = lo + (band * kTileBand + v - col * in_band) * tile_rows;
        rows = hi - row0;
        return true;
    }
};
static inline dim3 row_grid(int max_tiles, int cols) { return dim3((unsigned)(((long long)max_tiles * cols + 7) / 8 * 8)); }

}  // namespace xmoe
