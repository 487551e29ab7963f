// Forward products of the expert MLP where the experts have few rows (bf16, d and f multiples of 64, 16-byte aligned
// operands): a decoding step, the prompt of one request, a small micro-batch.  The weights of every expert with rows
// have to come from memory once and that is the bound; the 256 x 256 tiles of the direct-to-LDS kernels leave one
// block and at most three 16 KiB pieces of weights in flight per CU, and cut the work into so few tiles that the last
// wave of them is nearly empty (the down product of 36 experts at d 2048: 288 tiles for 256 CUs).
//
//   block = 4 waves = 64 rows x 128 columns (gate/up: the same 64 columns of both matrices), two blocks per CU.  The
//   waves split K, 32 at a time, and their sums are added through LDS in a fixed order at the end, so a wave streams its
//   part of the weights into registers with no barrier: 8 KiB of loads per wave and piece of K, one piece ahead (two
//   where the tile holds at most 32 rows).
//
// A lane fetches 8 bytes (4 columns) of 8 consecutive k-rows, which is after 16 byte permutes its share of four matrix
// instructions (v_mfma_f32_32x32x16_bf16, weights first): instruction j multiplies the columns 4c + j, c = 0..31.  So
// every load covers 256 contiguous bytes of a weight row, nothing passes through LDS on the way in, and a lane ends up
// with runs of consecutive columns of one row.
//
// Measured (MI355X, d 2048, f 1408, 64 experts + 2 shared, one decoding step of 8 tokens with 36 experts active): gate/up
// 95 -> 87 us (4.8 TB/s), down 64 -> 44 (4.7 TB/s); 8 experts with 8 rows each: both together 119 -> 36.
#include "xmoe_ffn.h"

namespace xmoe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 few_bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float few_f32x16_t;
typedef __attribute__((ext_vector_type(2))) uint32_t few_u32x2_t;
typedef __attribute__((ext_vector_type(4))) uint32_t few_u32x4_t;

constexpr int kFewRows = 64, kFewCols = 128, kFewK = 32;
__device__ __align__(16) const unsigned int kFewZero[4] = {0u, 0u, 0u, 0u};

// Explicitly global addresses: through a pointer that may be the block of zeros the compiler makes flat loads, which
// count as LDS accesses too and are waited for all at once.
typedef const __attribute__((address_space(1))) char* few_gptr;
template <typename V>
__device__ __forceinline__ V few_load(few_gptr p) {
    return *reinterpret_cast<const __attribute__((address_space(1))) V*>(p);
}

// what becomes of a product
enum FewMode { FEW_PLAIN = 0, FEW_GATEUP = 1, FEW_MLP2 = 2 };

struct FewOut {
    bf16_t *o0, *o1, *o2;   // PLAIN: C; GATEUP: G, U, A; MLP2: H, A
};

// the operands of one piece of K in flight
template <int MB>
struct FewPiece {
    few_u32x2_t w[2][8];
    few_u32x4_t x[MB][2];
};

// MB 32-row blocks of rows; w: this lane's columns of k-row 0 of the wave's K range, x: its rows at k 0 of it
template <int MB, int NB>
__device__ __forceinline__ void few_mainloop(few_f32x16_t (&acc)[MB][4], const bf16_t* w, size_t ldw,
                                             const bf16_t* const (&x)[MB], int n) {
    FewPiece<MB> p[NB];
    const few_gptr zero = (few_gptr)(const char*)kFewZero;
    const few_gptr wl = (few_gptr)(const char*)(w + 8 * ((threadIdx.x >> 5) & 1) * ldw);
    auto load = [&](FewPiece<MB>& q, int c) {   // past the end: zeros, so that no load depends on a branch
        const bool in = c < n;
        const size_t ld = in ? 2 * ldw : 0;
        const few_gptr wp = in ? wl + (size_t)c * kFewK * ld : zero;
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int k = 0; k < 8; ++k) q.w[st][k] = few_load<few_u32x2_t>(wp + (16 * st + k) * ld);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const few_gptr xl = in ? (few_gptr)(const char*)x[mb] + c * kFewK * 2 : zero;
#pragma unroll
            for (int st = 0; st < 2; ++st) q.x[mb][st] = few_load<few_u32x4_t>(xl + (in ? 32 * st : 0));
        }
    };
    auto multiply = [&](const FewPiece<MB>& q) {
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t f[4];
#pragma unroll
                for (int a = 0; a < 4; ++a) {   // the low (even column) or high halves of k-rows 2a and 2a+1
                    const few_u32x2_t lo = q.w[st][2 * a], hi = q.w[st][2 * a + 1];
                    f[a] = __builtin_amdgcn_perm(j < 2 ? hi.x : hi.y, j < 2 ? lo.x : lo.y,
                                                 (j & 1) ? 0x07060302u : 0x05040100u);
                }
                const few_bf16x8_t wf = __builtin_bit_cast(few_bf16x8_t, make_uint4(f[0], f[1], f[2], f[3]));
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[mb][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        wf, __builtin_bit_cast(few_bf16x8_t, q.x[mb][st]), acc[mb][j], 0, 0, 0);
            }
    };
#pragma unroll
    for (int b = 0; b < NB - 1; ++b) load(p[b], b);
    for (int c = 0; c < n; c += NB)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            load(p[(b + NB - 1) % NB], c + b + NB - 1);
            multiply(p[b]);
        }
}

// red: 64 KiB.  Lane (h, r) of wave w adds up, for row r, the columns it stores: PLAIN, MLP2 16 consecutive ones
// (registers 4w .. 4w+3 of the four accumulators), GATEUP 8 of either matrix (registers 2w, 2w+1 and 8 above them).
template <int MODE, int ACT, int MB, int NB>
__device__ __forceinline__ void few_tile(float* red, const bf16_t* w, size_t ldw, const bf16_t* x, size_t ldx,
                                         const int32_t* row_index, int row0, int rows, int k0, int n, FewOut out, int N,
                                         int n0) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, r = lane & 31;
    const bf16_t* xp[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {   // rows past the last one repeat it; what they give is not stored
        int rr = mb * 32 + r;
        rr = row0 + (rr < rows ? rr : rows - 1);
        xp[mb] = x + (size_t)(row_index ? row_index[rr] : rr) * ldx + k0 + 8 * h;
    }
    few_f32x16_t acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][j][v] = 0.f;
    few_mainloop<MB, NB>(acc, w + (size_t)k0 * ldw, ldw, xp, n);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (mb) __syncthreads();
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[((wave * 16 + v) * 4 + j) * 64 + lane] = acc[mb][j][v];
        __syncthreads();
        float s[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = MODE == FEW_GATEUP ? 2 * wave + (q & 1) + 8 * (q >> 1) : 4 * wave + q;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float* p = red + (v * 4 + j) * 64 + lane;
                s[q * 4 + j] = ((p[0] + p[4096]) + p[8192]) + p[12288];
            }
        }
        if (mb * 32 + r >= rows) continue;
        // accumulator register v holds c = 8 (v/4) + 4 h + v%4, columns 4c .. 4c+3 (GATEUP: c < 16 gate, then up)
        const int c = MODE == FEW_GATEUP ? 8 * (wave >> 1) + 4 * h + 2 * (wave & 1) : 8 * wave + 4 * h;
        const int col = n0 + 4 * c;
        if (col >= N) continue;
        const size_t ix = (size_t)(row0 + mb * 32 + r) * N + col;
        auto store8 = [&](bf16_t* o, const float* t) {
            *reinterpret_cast<uint4*>(o + ix) = make_uint4(pack_bf16x2(t[0], t[1]), pack_bf16x2(t[2], t[3]),
                                                           pack_bf16x2(t[4], t[5]), pack_bf16x2(t[6], t[7]));
        };
        if (MODE == FEW_GATEUP) {
            float a[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) a[i] = siluf_(s[i]) * s[8 + i];
            store8(out.o0, s);
            store8(out.o1, s + 8);
            store8(out.o2, a);
        } else {
            store8(out.o0, s);
            store8(out.o0 + 8, s + 8);
            if (MODE == FEW_MLP2) {
                float a[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) a[i] = act_fwd<ACT>(s[i]);
                store8(out.o1, a);
                store8(out.o1 + 8, a + 8);
            }
        }
    }
}

// C[rows of the tile, n0 ..] = X W;  K x N weights per expert (w1: the second matrix of GATEUP)
template <int MODE, int ACT>
__device__ __forceinline__ void few_block(const bf16_t* __restrict__ x, const int32_t* __restrict__ row_index,   // or NULL
                                          const int32_t* __restrict__ off, const int32_t* __restrict__ map, int K, int N,
                                          const bf16_t* __restrict__ w0, const bf16_t* __restrict__ w1, FewOut out) {
    __shared__ __align__(16) float red[4 * 64 * 64];
    constexpr int kCols = MODE == FEW_GATEUP ? kFewCols / 2 : kFewCols;
    const int e = map[4 + 2 * blockIdx.y], n0 = blockIdx.x * kCols;
    if (e < 0 || n0 >= N) return;
    const int row0 = map[4 + 2 * blockIdx.y + 1], rows = off[e + 1] - row0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = threadIdx.x & 31;
    const bf16_t* w = w0;
    int col = n0 + 4 * c;
    if (MODE == FEW_GATEUP && c >= 16) {
        w = w1;
        col -= 64;
    }
    if (col >= N) col = n0;   // the second half of a tile at the edge: not stored
    w += (size_t)e * K * N + col;
    const int pieces = K / kFewK, p0 = pieces * wave / 4, n = pieces * (wave + 1) / 4 - p0;
    if (rows <= 32)
        few_tile<MODE, ACT, 1, 3>(red, w, N, x, K, row_index, row0, rows, p0 * kFewK, n, out, N, n0);
    else
        few_tile<MODE, ACT, 2, 2>(red, w, N, x, K, row_index, row0, rows, p0 * kFewK, n, out, N, n0);
}

__global__ __launch_bounds__(256, 2) void ffn_gateup_few_kernel(const bf16_t* __restrict__ xd,
                                                                const int32_t* __restrict__ row_index,
                                                                const int32_t* __restrict__ off,
                                                                const int32_t* __restrict__ map, int d, int f,
                                                                const bf16_t* __restrict__ wg,
                                                                const bf16_t* __restrict__ wu, FewOut out) {
    few_block<FEW_GATEUP, XMOE_ACT_IDENTITY>(xd, row_index, off, map, d, f, wg, wu, out);
}
__global__ __launch_bounds__(256, 2) void ffn_down_few_kernel(const bf16_t* __restrict__ A,
                                                              const int32_t* __restrict__ off,
                                                              const int32_t* __restrict__ map, int f, int d,
                                                              const bf16_t* __restrict__ w, FewOut out) {
    few_block<FEW_PLAIN, XMOE_ACT_IDENTITY>(A, nullptr, off, map, f, d, w, nullptr, out);
}
template <int ACT>
__global__ __launch_bounds__(256, 2) void mlp2_up_few_kernel(const bf16_t* __restrict__ xd,
                                                             const int32_t* __restrict__ row_index,
                                                             const int32_t* __restrict__ off,
                                                             const int32_t* __restrict__ map, int d, int f,
                                                             const bf16_t* __restrict__ w1, FewOut out) {
    few_block<FEW_MLP2, ACT>(xd, row_index, off, map, d, f, w1, nullptr, out);
}

// columns padded to a multiple of the XCD count: the row tiles of an expert that read the same weights meet in one L2
inline dim3 few_grid(int N, int cols, int max_tiles) { return dim3(((N + cols - 1) / cols + 7) / 8 * 8, max_tiles); }

}  // namespace

// Where these kernels are the faster ones (gate/up and down together, us, 256-row tiles | these): mean rows 1: 173 | 154,
// 8: 228 | 212, 16: 231 | 221, 32: 236 | 248 (64 experts, d 2048, f 1408); 8: 181 | 164, 32: 177 | 183 (32 experts,
// d 4096, f 1024).  Fewer 256-row tiles than CUs leave most of the chip idle, and the line lies higher: mean rows 8:
// 119 | 36, 32: 120 | 43 (8 experts, d 2048, f 1408); 32: 247 | 115 (4 experts, d 7168, f 2048).
bool few_rows(int B, int E, int f) {
    return B <= 16ll * E || (B <= 32ll * E && (long long)E * ((f + 127) / 128) < 256);
}

int ffn_fwd_few(const FfnArgs& a, hipStream_t s) {
    const int max_tiles = ffn_max_tiles(a.B, a.E, kFewRows);
    int st = launch_tile_map(a.off, a.E, kFewRows, max_tiles, a.map, a.sched, s);
    if (st != XMOE_OK) return st;
    const FewOut o1 = {(bf16_t*)a.g, (bf16_t*)a.u, (bf16_t*)a.act}, o2 = {(bf16_t*)a.y, nullptr, nullptr};
    XMOE_LAUNCH(K_FFN_GATEUP_FEW, s,
                hipLaunchKernelGGL(ffn_gateup_few_kernel, few_grid(a.f, kFewCols / 2, max_tiles), dim3(256), 0, s,
                                   (const bf16_t*)a.xd, a.row_index, a.off, a.map, a.d, a.f, (const bf16_t*)a.wg,
                                   (const bf16_t*)a.wu, o1));
    XMOE_LAUNCH(K_FFN_DOWN_FEW, s,
                hipLaunchKernelGGL(ffn_down_few_kernel, few_grid(a.d, kFewCols, max_tiles), dim3(256), 0, s,
                                   (const bf16_t*)a.act, a.off, a.map, a.f, a.d, (const bf16_t*)a.wd, o2));
    return XMOE_OK;
}

int mlp2_fwd_few(const Mlp2Args& a, hipStream_t s) {
    const int max_tiles = ffn_max_tiles(a.B, a.E, kFewRows);
    int st = launch_tile_map(a.off, a.E, kFewRows, max_tiles, a.map, a.sched, s);
    if (st != XMOE_OK) return st;
    const FewOut o1 = {(bf16_t*)a.h, (bf16_t*)a.a_buf, nullptr}, o2 = {(bf16_t*)a.y, nullptr, nullptr};
#define XMOE_CALL(ACT)                                                                                               \
    XMOE_LAUNCH(K_MLP2_UP_FEW, s,                                                                                    \
                hipLaunchKernelGGL((mlp2_up_few_kernel<ACT>), few_grid(a.f, kFewCols, max_tiles), dim3(256), 0, s,    \
                                   (const bf16_t*)a.xd, a.row_index, a.off, a.map, a.d, a.f, (const bf16_t*)a.w1, o1))
    XMOE_DISPATCH_ACT(a.act, XMOE_CALL);
#undef XMOE_CALL
    XMOE_LAUNCH(K_FFN_DOWN_FEW, s,
                hipLaunchKernelGGL(ffn_down_few_kernel, few_grid(a.d, kFewCols, max_tiles), dim3(256), 0, s,
                                   (const bf16_t*)a.a_buf, a.off, a.map, a.f, a.d, (const bf16_t*)a.w2, o2));
    return XMOE_OK;
}

}  // namespace xmoe
