// Forward products of the expert MLP where the experts have few rows (bf16, d and f multiples of 64, 16-byte aligned
// operands): a decoding step, the prompt of one request, a small micro-batch.  The weights of every expert with rows
// have to come from memory once and that is the bound; the 256 x 256 tiles of the direct-to-LDS kernels keep at most
// three 16 KiB pieces of weights in flight per CU, and cut the work into so few tiles that the last wave of them is nearly
// empty (the down product of 36 experts at d 2048: 288 tiles for 256 CUs).
//
//   block = 4 waves = 64 rows x 128 columns (gate/up: the same 64 columns of both matrices), two blocks per CU.  A ring
//   of kFewStages stages of 32 k (8 KiB of weights, 4 KiB of rows) is filled by direct-to-LDS loads, three per wave and
//   stage, so a block keeps all but one stage in flight; one barrier per stage.  A wave owns 32 columns over all of K.
//
// Measured (MI355X, d 2048, f 1408, 64 experts + 2 shared, one decoding step of 8 tokens with 36 experts active, 256-row
// tiles | these): gate/up 96 | 85 us (4.9 TB/s), down 63 | 46 (4.5 TB/s); 8 experts with 8 rows each 70 | 18 and 48 | 12.
// Four stages and three blocks per CU: 2 to 8 % faster for narrow f, 15 % slower for a Zipf load on 32 experts of
// d 4096; twelve stages and one block: 3 to 15 % slower.
//
// Every output is one accumulator that takes K in ascending steps of 16, as in the 256 x 256 kernels, with the same
// operands in the same slots of the same instruction and the same activation: a row's result has the same bits whichever
// of the two families a call's row count selects.
#include "xmoe_ffn.h"

namespace xmoe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 few_bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float few_f32x16_t;
typedef __attribute__((ext_vector_type(4))) short few_s16x4_t;
typedef __attribute__((ext_vector_type(8))) short few_s16x8_t;

constexpr int kFewRows = 64, kFewCols = 128, kFewK = 32, kFewStages = 6;
constexpr int kFewWBytes = kFewK * kFewCols * 2;              // [32 k][128 columns]
constexpr int kFewStageBytes = kFewWBytes + kFewRows * kFewK * 2;   // and [64 rows][32 k]
constexpr int kFewLoads = 3;                                  // per wave and stage: two of weights, one of rows
__device__ __align__(16) const unsigned int kFewZero[4] = {0u, 0u, 0u, 0u};

// what becomes of a product
enum FewMode { FEW_PLAIN = 0, FEW_GATEUP = 1, FEW_MLP2 = 2 };

struct FewOut {
    bf16_t *o0, *o1, *o2;   // PLAIN: C; GATEUP: G, U, A; MLP2: H, A
};

__device__ __forceinline__ void few_load16(const bf16_t* p, char* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                     (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// A lane's share of the loads: 16 bytes of k-rows kr and kr + 4 of the weights and of one row of X per stage.
struct FewLoader {
    const bf16_t *w[2], *x;   // of the stage issued next
    size_t step;              // elements between the weights of two stages
    int left;                 // stages of K not yet issued; behind them the block of zeros, so that the counts stay uniform
    __device__ __forceinline__ void issue(char* __restrict__ stage) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const bool in = left > 0;
        const bf16_t* z = reinterpret_cast<const bf16_t*>(kFewZero);
        few_load16(in ? w[0] : z, stage + wave * 2048);
        few_load16(in ? w[1] : z, stage + wave * 2048 + 1024);
        few_load16(in ? x : z, stage + kFewWBytes + wave * 1024);
        w[0] += step;
        w[1] += step;
        x += kFewK;
        --left;
    }
};

// LDS layout: k-rows of 256 bytes whose 16-byte pieces are XOR-swizzled with 4 * (k-row % 4), rows of X of 64 bytes with
// pieces XOR-swizzled with (row / 4) % 4: the fragment reads fall on all banks.
// Columns of the wave, 8 k (16 ks + 8 (lane/32) ..): in a group of 16 lanes, lane s addresses 4 consecutive columns (s%4)
// of k-row s/4, and the transposing read hands every lane one column with 4 consecutive k.
template <int MODE>
__device__ __forceinline__ few_bf16x8_t few_frag_w(const char* stage, int ks) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, G = lane >> 4, s = lane & 15;
    const int col = (MODE == FEW_GATEUP ? 64 * (G & 1) + 16 * wave : 32 * wave + 16 * (G & 1)) + 4 * (s & 3);
    few_s16x4_t h[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int kr = 16 * ks + 8 * (G >> 1) + (s >> 2) + 4 * q;
        const char* a = stage + kr * 256 + (((col >> 3) ^ ((kr & 3) << 2)) << 4) + (col & 7) * 2;
        h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) few_s16x4_t*)(
            (__attribute__((address_space(3))) void*)a));
    }
    const few_s16x8_t v = {h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]};
    return __builtin_bit_cast(few_bf16x8_t, v);
}
__device__ __forceinline__ few_bf16x8_t few_frag_x(const char* stage, int mb, int ks) {
    const int lane = threadIdx.x & 63, r = mb * 32 + (lane & 31), c = 2 * ks + (lane >> 5);
    return *reinterpret_cast<const few_bf16x8_t*>(stage + kFewWBytes + r * 64 + ((c ^ ((r >> 2) & 3)) << 4));
}

// Refills the stage read before the last barrier and multiplies `cur`.  The two are distinct, and saying so matters: an
// LDS read that may observe a direct-to-LDS load in flight makes the compiler wait for all of them.
template <int MODE, int MB>
__device__ __forceinline__ void few_step(few_f32x16_t (&acc)[MB], FewLoader& ld, char* __restrict__ next,
                                         const char* __restrict__ cur) {
    ld.issue(next);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const few_bf16x8_t w = few_frag_w<MODE>(cur, ks);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, few_frag_x(cur, mb, ks), acc[mb], 0, 0, 0);
    }
}

// One tile: rows [row0, row0 + min(rows, 32 MB)), the block's columns.
template <int MODE, int ACT, int MB>
__device__ __forceinline__ void few_tile(FewLoader& ld, char* smem, int n, int row0, int rows, FewOut out, int N, int n0) {
    few_f32x16_t acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[mb][v] = 0.f;
#pragma unroll
    for (int s = 0; s < kFewStages - 1; ++s) ld.issue(smem + s * kFewStageBytes);
    int cur = 0, next = kFewStages - 1;
    for (int i = 0; i < n; ++i) {
        // stage i has landed for every thread, and every wave is done with stage i - 1, which is refilled now
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kFewLoads * (kFewStages - 2)) : "memory");
        few_step<MODE, MB>(acc, ld, smem + next * kFewStageBytes, smem + cur * kFewStageBytes);
        next = cur;
        cur = cur + 1 < kFewStages ? cur + 1 : 0;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may land in this LDS once the block has left it
    // accumulator register v of row r: column 8 (v/4) + 4 (lane/32) + v%4 of the wave's 32 (GATEUP: 16 gate, then 16 up)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31;
    const int col = n0 + (MODE == FEW_GATEUP ? 16 : 32) * wave + 4 * (lane >> 5);
    if (col >= N) return;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (mb * 32 + r >= rows) continue;
        const size_t ix = (size_t)(row0 + mb * 32 + r) * N + col;
        auto store4 = [&](bf16_t* o, int q, float a, float b, float c, float d) {
            *reinterpret_cast<uint2*>(o + ix + 8 * q) = make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
        };
#pragma unroll
        for (int q = 0; q < (MODE == FEW_GATEUP ? 2 : 4); ++q) {
            float s[4], a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = acc[mb][4 * q + i];
            store4(out.o0, q, s[0], s[1], s[2], s[3]);
            if (MODE == FEW_GATEUP) {
                float u[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    u[i] = acc[mb][8 + ((4 * q + i) & 7)];
                    a[i] = s[i] * fast_sigmoid(s[i]) * u[i];
                }
                store4(out.o1, q, u[0], u[1], u[2], u[3]);
                store4(out.o2, q, a[0], a[1], a[2], a[3]);
            }
            if (MODE == FEW_MLP2) {
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = act_fast<ACT>(s[i]);
                store4(out.o1, q, a[0], a[1], a[2], a[3]);
            }
        }
    }
}

// C[rows of the tile, n0 ..] = X W;  K x N weights per expert (w1: the second matrix of GATEUP).
// The tiles (row tile, then column tile) are dealt to the XCDs in eight runs of equal length, workgroup L going to XCD
// L % 8: every XCD gets its share whatever the number of column tiles, and row tiles that read the same weights meet in
// one L2.
template <int MODE, int ACT>
__device__ __forceinline__ void few_block(const bf16_t* __restrict__ x, const int32_t* __restrict__ row_index,   // or NULL
                                          const int32_t* __restrict__ off, const int32_t* __restrict__ map, int K, int N,
                                          const bf16_t* __restrict__ w0, const bf16_t* __restrict__ w1, FewOut out) {
    __shared__ __align__(16) char smem[kFewStages * kFewStageBytes];
    constexpr int kCols = MODE == FEW_GATEUP ? kFewCols / 2 : kFewCols;
    const int nt = (N + kCols - 1) / kCols, total = map[0] * nt, run = (total + 7) / 8;
    const int slot = blockIdx.x >> 3, t = (blockIdx.x & 7) * run + slot;
    if (slot >= run || t >= total) return;
    const int tile = t / nt, n0 = (t - tile * nt) * kCols;
    const int e = map[4 + 2 * tile], row0 = map[4 + 2 * tile + 1], rows = off[e + 1] - row0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    FewLoader ld;
    {
        int r = wave * 16 + (lane >> 2);   // rows past the last one repeat it; what they give is not stored
        const int c = (lane & 3) ^ ((r >> 2) & 3);
        r = row0 + (r < rows ? r : rows - 1);
        ld.x = x + (size_t)(row_index ? row_index[r] : r) * K + 8 * c;
    }
    const int c = (lane & 15) ^ ((lane >> 4) << 2);
    const bf16_t* w = MODE == FEW_GATEUP && c >= 8 ? w1 : w0;
    int col = n0 + 8 * (MODE == FEW_GATEUP ? c & 7 : c);
    if (col >= N) col = n0;   // the second half of a tile at the edge: not stored
    w += ((size_t)e * K + wave * 8 + (lane >> 4)) * N + col;
    ld.w[0] = w;
    ld.w[1] = w + (size_t)4 * N;
    ld.step = (size_t)kFewK * N;
    ld.left = K / kFewK;
    if (rows <= 32)
        few_tile<MODE, ACT, 1>(ld, smem, K / kFewK, row0, rows, out, N, n0);
    else
        few_tile<MODE, ACT, 2>(ld, smem, K / kFewK, row0, rows, out, N, n0);
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

inline dim3 few_grid(int N, int cols, int max_tiles) {
    const long long tiles = (long long)max_tiles * ((N + cols - 1) / cols);
    return dim3((unsigned)((tiles + 7) / 8 * 8));
}

}  // namespace

// Where these kernels are the faster ones: up to 32 rows per expert on average.  Measured (MI355X, gate/up and down
// together, us, 256-row tiles | these; Zipf: the experts' loads follow rank^-1.2):
//     mean rows                         1           8          16          32          48          64
//     64 experts, d 2048, f 1408    240 | 203   234 | 211   241 | 224   247 | 239   251 | 255   254 | 270
//       Zipf                                    222 | 202   241 | 225   258 | 258   280 | 281   306 | 314
//     256 experts, d 2048, f 512    347 | 295   342 | 317   360 | 336   367 | 359   377 | 391   388 | 404
//     32 experts, d 4096, f 1024    183 | 165   179 | 165   183 | 168   181 | 174   183 | 184   185 | 191
//       Zipf                                    182 | 174   188 | 177   244 | 193   237 | 230   269 | 244
//     512 experts, d 1024, f 256    228 | 172   229 | 186   238 | 199   246 | 218   257 | 229   262 | 249
//     64 experts, d 7168, f 256     207 | 146   202 | 153   195 | 158   200 | 175
//     8 experts, d 2048, f 1408     117 | 29    118 | 29    118 | 30    116 | 30
// With all rows on one expert they are the faster ones too (64 experts, d 2048, f 1408, mean 16: 96 | 51), but for 8192
// rows and more (256 experts, d 2048, f 512, mean 32: 106 | 112).  Above 32 rows the 64-row tiles read the weights more
// often than the 256-row ones wait for them.
bool few_rows(int B, int E) { return B <= 32ll * E; }

int ffn_fwd_few(const FfnArgs& a, hipStream_t s) {
    const int max_tiles = ffn_max_tiles(a.B, a.E, kFewRows);
    int st = launch_tile_map(a.off, a.E, kFewRows, max_tiles, a.map, a.sched, false, s);
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
    int st = launch_tile_map(a.off, a.E, kFewRows, max_tiles, a.map, a.sched, false, s);
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
