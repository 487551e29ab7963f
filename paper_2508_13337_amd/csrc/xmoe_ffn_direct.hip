// Products of the expert MLP on 128 x 128 bf16 tiles with direct-to-LDS loads (xmoe_tile_direct.h):
//   - widths that are multiples of 8 but not of 64, in place of the register-staged tiles;
//   - widths that are multiples of 64 where the 256 x 256 tiles of the direct-to-LDS kernels are too few for the chip, or
//     half empty (direct_fwd, direct_bwd, direct_wgrads below).
//
// Measured (MI355X): T 3001 d 1000 f 712, 24 experts + 1 shared, register-staged | these: gate/up 96 | 72 us, dAct 82 | 58,
// down 51 | 47, dX 78 | 75; 509 tokens, 64 experts + 2 shared, d 2048 f 1408, 256-row tiles | these: gate/up 180 | 172,
// down 120 | 86; 8 experts of 200 rows, d 2048 f 1408: forward 119 | 57; weight gradients of the first of these 166 | 103.
//
// Bound: a 128 x 128 tile takes in 64 bytes per clock and CU at the full rate of the matrix cores, about what a CU's load
// path delivers at best; they reach 15 to 30 % of it where K is long, a third less than the 256 x 256 tiles, which is why
// those keep every call that fills the chip with them.
#include "xmoe_ffn.h"
#include "xmoe_tile_direct.h"

namespace xmoe {
namespace {

#define XMOE_DIRECT_KERNEL __global__ __launch_bounds__(256, 2) void

// FAST (widths that are multiples of 64): the activations of the 256-row kernels, so that a row's result does not depend on
// which of the two a call's row count selects; otherwise those of the register-staged tiles, for the same reason.
template <bool FAST>
__device__ __forceinline__ float dir_sigmoid(float g) { return FAST ? fast_sigmoid(g) : sigmoidf_(g); }

// G = Xd Wg, U = Xd Wu, A = silu(G) * U: 64 columns of both matrices
template <bool FAST>
XMOE_DIRECT_KERNEL ffn_gateup_direct_kernel(const bf16_t* __restrict__ xd, const int32_t* __restrict__ row_index,   // or NULL
                                            const int32_t* __restrict__ off, const int32_t* __restrict__ map, int d, int f,
                                            const bf16_t* __restrict__ wg, const bf16_t* __restrict__ wu,
                                            bf16_t* __restrict__ G, bf16_t* __restrict__ U, bf16_t* __restrict__ A) {
    __shared__ __align__(16) char smem[kDirLds];
    RowTile t;
    if (!t.init(off, map, (f + 63) / 64, 128)) return;
    const int n0 = t.col * 64;
    DirRows<false> a;
    DirCols b;
    a.init(row_index ? xd : xd + (size_t)t.row0 * d, nullptr, d, t.rows, row_index ? row_index + t.row0 : nullptr, d);
    b.init(wg + (size_t)t.e * d * f + n0, wu + (size_t)t.e * d * f + n0, f, f - n0, d);
    tile_f32x16_t acc[2][2];
    tile_zero<true>(acc);
    dir_mainloop_rc<true>(acc, a, b, d, t.rows, f - n0, smem);
    char* strip = dir_strip(smem);
    const int wm = threadIdx.x >> 7, wn = (threadIdx.x >> 6) & 1, cols = f - n0 - wn * 32;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float g[4], u[4], s[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                g[j] = acc[mi][0][4 * q + j];
                u[j] = acc[mi][1][4 * q + j];
                s[j] = g[j] * dir_sigmoid<FAST>(g[j]) * u[j];
            }
            dir_put4(strip, 0, q, g[0], g[1], g[2], g[3]);
            dir_put4(strip, 16, q, u[0], u[1], u[2], u[3]);
            dir_put4(strip, 32, q, s[0], s[1], s[2], s[3]);
        }
        dir_strip_sync();
        const int r0 = wm * 64 + mi * 32;
        const size_t ix = (size_t)(t.row0 + r0) * f + n0 + wn * 32;
        dir_flush<32, true, false>(strip, 0, G + ix, f, t.rows - r0, cols);
        dir_flush<32, true, false>(strip, 16, U + ix, f, t.rows - r0, cols);
        dir_flush<32, true, false>(strip, 32, A + ix, f, t.rows - r0, cols);
        dir_strip_sync();
    }
}

// Y = A Wd
XMOE_DIRECT_KERNEL ffn_down_direct_kernel(const bf16_t* __restrict__ A, const int32_t* __restrict__ off,
                                          const int32_t* __restrict__ map, int d, int f, const bf16_t* __restrict__ wd,
                                          bf16_t* __restrict__ Y) {
    __shared__ __align__(16) char smem[kDirLds];
    RowTile t;
    if (!t.init(off, map, (d + 127) / 128, 128)) return;
    const int n0 = t.col * 128;
    DirRows<false> a;
    DirCols b;
    a.init(A + (size_t)t.row0 * f, nullptr, f, t.rows, nullptr, f);
    b.init(wd + (size_t)t.e * f * d + n0, nullptr, d, d - n0, f);
    tile_f32x16_t acc[2][2];
    tile_zero<true>(acc);
    dir_mainloop_rc<false>(acc, a, b, f, t.rows, d - n0, smem);
    dir_store(acc, smem, Y + (size_t)t.row0 * d + n0, d, t.rows, d - n0);
}

// two-matrix expert: H = Xd W1, A = act(H)
template <int ACT, bool FAST>
XMOE_DIRECT_KERNEL mlp2_up_direct_kernel(const bf16_t* __restrict__ xd, const int32_t* __restrict__ row_index,   // or NULL
                                         const int32_t* __restrict__ off, const int32_t* __restrict__ map, int d, int f,
                                         const bf16_t* __restrict__ w1, bf16_t* __restrict__ H, bf16_t* __restrict__ A) {
    __shared__ __align__(16) char smem[kDirLds];
    RowTile t;
    if (!t.init(off, map, (f + 127) / 128, 128)) return;
    const int n0 = t.col * 128;
    DirRows<false> a;
    DirCols b;
    a.init(row_index ? xd : xd + (size_t)t.row0 * d, nullptr, d, t.rows, row_index ? row_index + t.row0 : nullptr, d);
    b.init(w1 + (size_t)t.e * d * f + n0, nullptr, f, f - n0, d);
    tile_f32x16_t acc[2][2];
    tile_zero<true>(acc);
    dir_mainloop_rc<false>(acc, a, b, d, t.rows, f - n0, smem);
    char* strip = dir_strip(smem);
    const int wm = threadIdx.x >> 7, wn = (threadIdx.x >> 6) & 1, cols = f - n0 - wn * 64;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float h[4], s[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    h[j] = acc[mi][ni][4 * q + j];
                    s[j] = FAST ? act_fast<ACT>(h[j]) : act_fwd<ACT>(h[j]);
                }
                dir_put4(strip, 8 * ni, q, h[0], h[1], h[2], h[3]);
                dir_put4(strip, 16 + 8 * ni, q, s[0], s[1], s[2], s[3]);
            }
        dir_strip_sync();
        const int r0 = wm * 64 + mi * 32;
        const size_t ix = (size_t)(t.row0 + r0) * f + n0 + wn * 64;
        dir_flush<64, true, false>(strip, 0, H + ix, f, t.rows - r0, cols);
        dir_flush<64, true, false>(strip, 16, A + ix, f, t.rows - r0, cols);
        dir_strip_sync();
    }
}

// dA = dY W^T (W = Wd or W2) and what follows from it; in, out: arrays [B, f], CHAIN and EPI as in dir_dact_rounds
template <bool CHAIN, int NIN, int NOUT, class Epi>
__device__ __forceinline__ void dact_direct(const bf16_t* __restrict__ dY, const int32_t* __restrict__ dy_index,
                                            const float* __restrict__ dy_scale, const int32_t* __restrict__ off,
                                            const int32_t* __restrict__ map, int d, int f, const bf16_t* __restrict__ w,
                                            float* __restrict__ row_part, int B, const bf16_t* const (&in)[NIN],
                                            bf16_t* const (&out)[NOUT], Epi epi) {
    __shared__ __align__(16) char smem[kDirLds];
    RowTile t;
    if (!t.init(off, map, (f + 127) / 128, 128)) return;
    const int n0 = t.col * 128;
    DirRows<false> a, b;
    a.init(dy_index ? dY : dY + (size_t)t.row0 * d, nullptr, d, t.rows, dy_index ? dy_index + t.row0 : nullptr, d);
    b.init(w + ((size_t)t.e * f + n0) * d, nullptr, d, f - n0, nullptr, d);
    tile_f32x16_t acc[2][2];
    tile_zero<true>(acc);
    dir_mainloop_rr<false>(acc, a, b, d, t.rows, f - n0, smem);
    const size_t base = (size_t)t.row0 * f + n0;
    const bf16_t* tin[NIN];
    bf16_t* tout[NOUT];
#pragma unroll
    for (int i = 0; i < NIN; ++i) tin[i] = in[i] + base;
#pragma unroll
    for (int i = 0; i < NOUT; ++i) tout[i] = out[i] + base;
    const int wm = threadIdx.x >> 7, wn = (threadIdx.x >> 6) & 1;
    float* part = row_part + (size_t)(t.col * 2 + wn) * B + t.row0;
    const float* scale = dy_index && dy_scale ? dy_scale + t.row0 : nullptr;
    if (t.rows >= wm * 64 + 64 && f - n0 >= wn * 64 + 64)
        dir_dact_rounds<true, CHAIN, NIN, NOUT>(acc, smem, tin, tout, f, scale, part, t.rows, f - n0, epi);
    else
        dir_dact_rounds<false, CHAIN, NIN, NOUT>(acc, smem, tin, tout, f, scale, part, t.rows, f - n0, epi);
}

// dG = dA * U * silu'(G), dU = dA * silu(G), A = silu(G) * U
template <bool FAST>
XMOE_DIRECT_KERNEL ffn_dact_direct_kernel(const bf16_t* __restrict__ dY, const int32_t* __restrict__ dy_index,   // or NULL
                                          const float* __restrict__ dy_scale,                                   // or NULL
                                          const int32_t* __restrict__ off, const int32_t* __restrict__ map, int d, int f,
                                          const bf16_t* __restrict__ wd, const bf16_t* __restrict__ G,
                                          const bf16_t* __restrict__ U, bf16_t* __restrict__ dG, bf16_t* __restrict__ dU,
                                          bf16_t* __restrict__ A, float* __restrict__ row_part, int B) {
    const bf16_t* in[2] = {G, U};
    bf16_t* out[3] = {dG, dU, A};
    dact_direct<FAST, 2, 3>(dY, dy_index, dy_scale, off, map, d, f, wd, row_part, B, in, out,
                      [](float da0, float sc, const float(&x)[2], float(&y)[3]) {
                          const float g = x[0], u = x[1], da = da0 * sc, sg = dir_sigmoid<FAST>(g), sl = g * sg;
                          const float a1 = sl * u;
                          y[0] = da * u * (sg * (1.0f + g * (1.0f - sg)));
                          y[1] = da * sl;
                          y[2] = a1 * sc;   // scaled: the weight gradient multiplies it with unscaled rows
                          return a1;
                      });
}

// two-matrix expert: dH = dA * act'(H), A = act(H)
template <int ACT, bool FAST>
XMOE_DIRECT_KERNEL mlp2_dact_direct_kernel(const bf16_t* __restrict__ dY, const int32_t* __restrict__ dy_index,   // or NULL
                                           const float* __restrict__ dy_scale,                                   // or NULL
                                           const int32_t* __restrict__ off, const int32_t* __restrict__ map, int d, int f,
                                           const bf16_t* __restrict__ w2, const bf16_t* __restrict__ H,
                                           bf16_t* __restrict__ dH, bf16_t* __restrict__ A, float* __restrict__ row_part,
                                           int B) {
    const bf16_t* in[1] = {H};
    bf16_t* out[2] = {dH, A};
    dact_direct<FAST, 1, 2>(dY, dy_index, dy_scale, off, map, d, f, w2, row_part, B, in, out,
                      [](float da0, float sc, const float(&x)[1], float(&y)[2]) {
                          float a, g;
                          if (FAST)
                              act_fast_grad<ACT>(x[0], a, g);
                          else
                              act_fwd_grad<ACT>(x[0], a, g);
                          y[0] = da0 * sc * g;
                          y[1] = a * sc;
                          return a;
                      });
}

// dXd = dG Wg^T + dU Wu^T; TWO = false: a single pair (the two-matrix expert: dXd = dH W1^T)
template <bool TWO>
XMOE_DIRECT_KERNEL ffn_dx_direct_kernel(const bf16_t* __restrict__ dG, const bf16_t* __restrict__ dU,
                                        const int32_t* __restrict__ off, const int32_t* __restrict__ map, int d, int f,
                                        const bf16_t* __restrict__ wg, const bf16_t* __restrict__ wu,
                                        bf16_t* __restrict__ dXd) {
    __shared__ __align__(16) char smem[kDirLds];
    RowTile t;
    if (!t.init(off, map, (d + 127) / 128, 128)) return;
    const int n0 = t.col * 128;
    DirRows<TWO> a, b;
    const size_t r = (size_t)t.row0 * f, c = ((size_t)t.e * d + n0) * f;
    a.init(dG + r, TWO ? dU + r : nullptr, f, t.rows, nullptr, f);
    b.init(wg + c, TWO ? wu + c : nullptr, f, d - n0, nullptr, f);
    tile_f32x16_t acc[2][2];
    tile_zero<true>(acc);
    dir_mainloop_rr<TWO>(acc, a, b, f, t.rows, d - n0, smem);
    dir_store(acc, smem, dXd + (size_t)t.row0 * d + n0, d, t.rows, d - n0);
}

// Weight gradients
template <bool GP, bool GQ>
__device__ __forceinline__ void wgrad_direct_tile(const WgradJob<bf16_t>& j, int u, int e, int lo, int K, char* smem) {
    const int tiles_m = (j.M + 127) / 128, m0 = (u % tiles_m) * 128, n0 = (u / tiles_m) * 128;
    tile_f32x16_t acc[2][2];
    tile_zero<true>(acc);
    if (K > 0) {
        DirColsK<GP> a;
        DirColsK<GQ> b;
        a.init(j.P + m0 + (GP ? 0 : (size_t)lo * j.M), j.M, j.M - m0, GP ? j.p_index + lo : nullptr, K);
        b.init(j.Q + n0 + (GQ ? 0 : (size_t)lo * j.N), j.N, j.N - n0, GQ ? j.q_index + lo : nullptr, K);
        dir_mainloop_cc<GP, GQ>(acc, a, b, K, j.M - m0, j.N - n0, smem);
    }
    dir_store(acc, smem, j.dW + (size_t)e * j.M * j.N + (size_t)m0 * j.N + n0, j.N, j.M - m0, j.N - n0);
}
XMOE_DIRECT_KERNEL ffn_wgrad_direct_kernel(WgradJobs<bf16_t> jobs, int E, const int32_t* __restrict__ off,
                                           const int32_t* __restrict__ sched) {
    __shared__ __align__(16) char smem[kDirLds];
    int m, u;
    if (!jobs.place(E, m, u)) return;
    const WgradJob<bf16_t> j = jobs.job[m % jobs.n_jobs];
    const int e = sched[m / jobs.n_jobs], lo = off[e], K = off[e + 1] - lo;
    if (j.p_index)
        wgrad_direct_tile<true, false>(j, u, e, lo, K, smem);
    else if (j.q_index)
        wgrad_direct_tile<false, true>(j, u, e, lo, K, smem);
    else
        wgrad_direct_tile<false, false>(j, u, e, lo, K, smem);
}

template <class Args>
inline int tile_map_direct(const Args& a, bool rank, hipStream_t s) {
    return launch_tile_map(a.off, a.E, 128, ffn_max_tiles(a.B, a.E, 128), a.map, a.sched, rank, s);
}
template <class Args>
inline dim3 grid_direct(const Args& a, int n, int cols) {
    return row_grid(ffn_max_tiles(a.B, a.E, 128), (n + cols - 1) / cols);
}
inline bool fast_act(int d, int f) { return d % 64 == 0 && f % 64 == 0; }

}  // namespace

// Where these are faster than the 256-row kernels.  Measured (MI355X, gate/up and down together, us, 256-row | these; the
// tiles are those of the 256-row kernels for both products):
//   few tiles (a launch of up to one or two rounds of 256 CUs runs as long as its longest tile, whatever it holds):
//     rows per expert         100          400          800          1600         3200
//     4 experts, 2048 x 1408  117 | 43     121 | 58     136 | 93     185 | 146    262 | 268     (304, 532, 988 tiles from 800)
//     8 experts, 2048 x 1408   92 | 45     144 | 87     158 | 148    264 | 268    472 | 539     (304, 608, 1064 from 400)
//     8 experts, 4096 x 1024  147 | 56     143 | 113    188 | 204    354 | 386                  (384, 768 from 400)
//    16 experts, 1024 x 704    65 | 30      95 | 53     102 | 88     161 | 157                  (320, 640, 1120 from 400)
//    32 experts, 2048 x 704   103 | 78     185 | 183    294 | 318                               (896, 1792 from 400)
//   one half-empty tile per expert (Z: Zipf-like load of the mean above it):
//     rows per expert              34           48           64           80           96           120
//    48 experts, 2048 x 1024   163 | 137    161 | 141    160 | 146    165 | 151    168 | 155    178 | 169   Z 48: 162 | 148
//   256 experts,  512 x 768    184 | 144    200 | 152    200 | 159    212 | 166    215 | 174    218 | 194   Z 48: 204 | 167
//    64 experts, 1536 x 1536   212 | 193    219 | 200    221 | 208    227 | 216    231 | 224    241 | 252   Z 48: 235 | 220
//   300 experts,  512 x 1024   267 | 219    274 | 242    277 | 242    283 | 248    300 | 267    323 | 287   Z 48: 274 | 250
//                                                                      72
//    32 experts, 2048 x 2560   220 | 219    223 | 225    229 | 233    235 | 235                             Z 64: 268 | 267
//    96 experts, 1024 x 1792   260 | 232    262 | 235    264 | 249    271 | 254                             Z 64: 275 | 272
//    16 experts, 4096 x 2816   243 | 221    250 | 224    248 | 228    255 | 228                             Z 64: 259 | 278
//    64 experts, 2048 x 1408   244 | 217    244 | 229    245 | 238    250 | 244    (128: 268 | 313)         Z 64: 259 | 263
//    80 experts, 2048 x 1152   241 | 220    243 | 225    249 | 235    253 | 239                             Z 64: 255 | 262
//   512 experts,  512 x 704    315 | 247    335 | 263    334 | 274    335 | 285                             Z 64: 346 | 298
//                                                                      80
//    64 experts, 2048 x 1792   292 | 278    299 | 290    299 | 307    304 | 310    309 | 320    318 | 370   Z 48: 308 | 318
//   128 experts, 2048 x 1024   338 | 330    341 | 345    351 | 350    361 | 364    362 | 372    374 | 409   Z 48: 368 | 368
//    32 experts, 4096 x 2048   311 | 320    313 | 329    312 | 336    322 | 346    323 | 356    336 | 404   Z 48: 364 | 349
//    96 experts, 2048 x 2048   470 | 478    473 | 503    478 | 517    488 | 531    497 | 550    521 | 614   Z 48: 519 | 531
//   256 experts, 2048 x 1408   830 | 874    853 | 907    865 | 952    876 | 993    900 | 1003   964 | 1100  Z 48: 915 | 985
//   128 experts, 5120 x 1536  1143 | 1216              1166 | 1289                            1214 | 1383  (128: 1367 | 1600)
// Many weights keep the chip full and their stream long, and then the larger tile's fewer requests count: from 235 million
// elements of a matrix on (E d f) the two are level at best.  Below 256 columns the products are launch-bound either way.
bool direct_fwd(int B, int E, int d, int f) {
    if (d < 256 || f < 256) return false;
    const long long row_tiles = E * ((B + 256ll * E - 1) / (256ll * E)), weights = (long long)E * d * f;
    if (row_tiles * ((f + 127) / 128 + (d + 255) / 256) <= 640) return true;
    return weights <= 200000000 && B <= (weights <= 160000000 ? 96ll : 72ll) * E;
}
// The backward.  Its weight gradients take the 128 x 128 tiles where the 256-row kernels have few tiles of them and the
// experts are not long; dAct and dX do with them, and where a launch of theirs has few or half-empty tiles of 256 rows (the
// weight gradients are then a launch of the 256-row kernels without dX).  Whole backward, us, all 256-row | dAct and dX
// 128-row | all 128-row (- : not measured):
//     rows per expert                        40                100               400                  1600
//     4 experts, 512 x 256 (24 tiles)     79 | 55 | 34      82 | 60 | 35     104 | 72 | 39      161 | 132 | 56
//     4 experts, 2048 x 1408 (544)       167 | 141 | 93    175 | 149 | 98    212 | 162 | 123    340 | 347 | 314
//     8 experts, 1024 x 704 (288)        139 | 112 | 59    136 | 111 | 62    163 | 130 | 79     237 | 232 | 184
//     8 experts, 2048 x 1408 (1088)      172 | 146 | 115   175 | 151 | 120   205 | 214 | 196    535 | 579 | 578
//     8 experts, 4096 x 1024 (1536)      233 | 162 | 141   246 | 169 | 147   368 | 273 | 267    746 | 767 | 813
//    16 experts, 1024 x 704 (576)        146 | 126 | 72    139 | 118 | 75    134 | 147 | 120    335 | 344 | 339
//    16 experts, 2048 x 1408 (2176)      234 | 206 | 183   196 | 210 | 193   380 | 375 | 388   1000 | 1086 | 1183
//    64 experts, 1024 x 704 (2304)       215 | 169 | 173   204 | 194 | 195   369 | - | 432
//    64 experts, 2048 x 1408 (8704)      542 | 520 | 676   601 | 589 | 738  1171 | - | 1540
//   256 experts, 1024 x 256 (3072)       253 | 238 | 264   280 | 270 | 312
//    32 experts, 7168 x 2048 (14336)    1166 | 1090 | -   1297 | 1246 | -
//   256 experts, 2048 x 512             810 | 812 | -      907 | 902 | -
// dAct and dX by rows per expert: 64 experts, 2048 x 1408: 4 rows 504 | 471, 64 rows 562 | 541, 96 of routed and 2 x 1021
// rows 679 | 757; 16 experts, 2048 x 1408: 64 rows 225 | 190, 96 rows 192 | 202.
bool direct_wgrads(int B, int E, int d, int f, int matrices) {
    const long long td = (d + 255) / 256;   // n: tiles of the 256-row weight-gradient kernels
    const long long n = E * td * ((f + 255) / 256 + (matrices == 3 ? (f + 127) / 128 : (f + 255) / 256));
    return n <= 2200 && n * B <= 600000ll * E;
}
bool direct_bwd(int B, int E, int d, int f, int matrices) {
    if (d < 256 || f < 256) return false;
    const long long row_tiles = E * ((B + 256ll * E - 1) / (256ll * E));
    return B <= 80ll * E || row_tiles * ((f + 255) / 256) <= 64 || direct_wgrads(B, E, d, f, matrices);
}

bool direct_supported(const FfnArgs& a) {
    if (a.dt != XMOE_BF16 || a.d % 8 != 0 || a.f % 8 != 0) return false;
    const void* ptrs[] = {a.xd, a.wg, a.wu, a.wd, a.g, a.u, a.y, a.dy, a.dxd, a.dwg, a.dwu, a.dwd, a.act, a.dg, a.du};
    for (const void* p : ptrs)
        if (!aligned16(p)) return false;
    return true;
}
bool direct_supported(const Mlp2Args& a) {
    if (a.dt != XMOE_BF16 || a.d % 8 != 0 || a.f % 8 != 0) return false;
    const void* ptrs[] = {a.xd, a.w1, a.w2, a.h, a.y, a.dy, a.dxd, a.dw1, a.dw2, a.a_buf, a.dh};
    for (const void* p : ptrs)
        if (!aligned16(p)) return false;
    return true;
}

template <bool FAST>
static int fwd_direct(const FfnArgs& a, hipStream_t s) {
    int st = tile_map_direct(a, false, s);
    if (st != XMOE_OK) return st;
    XMOE_LAUNCH(K_FFN_GATEUP_DIRECT, s,
                hipLaunchKernelGGL((ffn_gateup_direct_kernel<FAST>), grid_direct(a, a.f, 64), dim3(256), 0, s,
                                   (const bf16_t*)a.xd, a.row_index, a.off, a.map, a.d, a.f, (const bf16_t*)a.wg,
                                   (const bf16_t*)a.wu, (bf16_t*)a.g, (bf16_t*)a.u, (bf16_t*)a.act));
    XMOE_LAUNCH(K_FFN_DOWN_DIRECT, s,
                hipLaunchKernelGGL(ffn_down_direct_kernel, grid_direct(a, a.d, 128), dim3(256), 0, s, (const bf16_t*)a.act,
                                   a.off, a.map, a.d, a.f, (const bf16_t*)a.wd, (bf16_t*)a.y));
    return XMOE_OK;
}
int ffn_fwd_direct(const FfnArgs& a, hipStream_t s) {
    return fast_act(a.d, a.f) ? fwd_direct<true>(a, s) : fwd_direct<false>(a, s);
}

template <bool FAST>
static int bwd_rows_direct(const FfnArgs& a, hipStream_t s) {
    int st = tile_map_direct(a, true, s);
    if (st != XMOE_OK) return st;
    XMOE_LAUNCH(K_FFN_DACT_DIRECT, s,
                hipLaunchKernelGGL((ffn_dact_direct_kernel<FAST>), grid_direct(a, a.f, 128), dim3(256), 0, s,
                                   (const bf16_t*)a.dy, a.dy_index, a.dy_scale, a.off, a.map, a.d, a.f, (const bf16_t*)a.wd,
                                   (const bf16_t*)a.g, (const bf16_t*)a.u, (bf16_t*)a.dg, (bf16_t*)a.du, (bf16_t*)a.act,
                                   a.row_part, a.B));
    if (a.row_grad) {
        st = launch_row_grad_reduce(a.row_part, (a.f + 63) / 64, a.B, a.row_grad, s);
        if (st != XMOE_OK) return st;
    }
    XMOE_LAUNCH(K_FFN_DX_DIRECT, s,
                hipLaunchKernelGGL((ffn_dx_direct_kernel<true>), grid_direct(a, a.d, 128), dim3(256), 0, s,
                                   (const bf16_t*)a.dg, (const bf16_t*)a.du, a.off, a.map, a.d, a.f, (const bf16_t*)a.wg,
                                   (const bf16_t*)a.wu, (bf16_t*)a.dxd));
    return XMOE_OK;
}
int ffn_bwd_rows_direct(const FfnArgs& a, hipStream_t s) {
    return fast_act(a.d, a.f) ? bwd_rows_direct<true>(a, s) : bwd_rows_direct<false>(a, s);
}

template <class Args>
static int bwd_wgrads(const Args& a, hipStream_t s) {
    WgradJobs<bf16_t> jobs = wgrad_jobs<bf16_t>(a);
    const dim3 grid = jobs.cut(a.E, a.d, a.f, 128);
    XMOE_LAUNCH(K_FFN_WGRAD_DIRECT, s,
                hipLaunchKernelGGL(ffn_wgrad_direct_kernel, grid, dim3(256), 0, s, jobs, a.E, a.off, a.sched));
    return XMOE_OK;
}
int ffn_bwd_wgrads_direct(const FfnArgs& a, hipStream_t s) { return bwd_wgrads(a, s); }
int mlp2_bwd_wgrads_direct(const Mlp2Args& a, hipStream_t s) { return bwd_wgrads(a, s); }

template <bool FAST>
static int mlp2_fwd_direct_as(const Mlp2Args& a, hipStream_t s) {
    int st = tile_map_direct(a, false, s);
    if (st != XMOE_OK) return st;
#define XMOE_CALL(ACT)                                                                                                    \
    XMOE_LAUNCH(K_MLP2_UP_DIRECT, s,                                                              \
                hipLaunchKernelGGL((mlp2_up_direct_kernel<ACT, FAST>), grid_direct(a, a.f, 128), dim3(256), 0, s,          \
                                   (const bf16_t*)a.xd, a.row_index, a.off, a.map, a.d, a.f, (const bf16_t*)a.w1,          \
                                   (bf16_t*)a.h, (bf16_t*)a.a_buf))
    XMOE_DISPATCH_ACT(a.act, XMOE_CALL);
#undef XMOE_CALL
    XMOE_LAUNCH(K_FFN_DOWN_DIRECT, s,
                hipLaunchKernelGGL(ffn_down_direct_kernel, grid_direct(a, a.d, 128), dim3(256), 0, s,
                                   (const bf16_t*)a.a_buf, a.off, a.map, a.d, a.f, (const bf16_t*)a.w2, (bf16_t*)a.y));
    return XMOE_OK;
}
int mlp2_fwd_direct(const Mlp2Args& a, hipStream_t s) {
    return fast_act(a.d, a.f) ? mlp2_fwd_direct_as<true>(a, s) : mlp2_fwd_direct_as<false>(a, s);
}

template <bool FAST>
static int mlp2_bwd_rows_direct_as(const Mlp2Args& a, hipStream_t s) {
    int st = tile_map_direct(a, true, s);
    if (st != XMOE_OK) return st;
#define XMOE_CALL(ACT)                                                                                                    \
    XMOE_LAUNCH(K_MLP2_DACT_DIRECT, s,                                                          \
                hipLaunchKernelGGL((mlp2_dact_direct_kernel<ACT, FAST>), grid_direct(a, a.f, 128), dim3(256), 0, s,        \
                                   (const bf16_t*)a.dy, a.dy_index, a.dy_scale, a.off, a.map, a.d, a.f,                    \
                                   (const bf16_t*)a.w2, (const bf16_t*)a.h, (bf16_t*)a.dh, (bf16_t*)a.a_buf, a.row_part,   \
                                   a.B))
    XMOE_DISPATCH_ACT(a.act, XMOE_CALL);
#undef XMOE_CALL
    if (a.row_grad) {
        st = launch_row_grad_reduce(a.row_part, (a.f + 63) / 64, a.B, a.row_grad, s);
        if (st != XMOE_OK) return st;
    }
    XMOE_LAUNCH(K_FFN_DX_DIRECT, s,
                hipLaunchKernelGGL((ffn_dx_direct_kernel<false>), grid_direct(a, a.d, 128), dim3(256), 0, s,
                                   (const bf16_t*)a.dh, (const bf16_t*)nullptr, a.off, a.map, a.d, a.f,
                                   (const bf16_t*)a.w1, (const bf16_t*)nullptr, (bf16_t*)a.dxd));
    return XMOE_OK;
}
int mlp2_bwd_rows_direct(const Mlp2Args& a, hipStream_t s) {
    return fast_act(a.d, a.f) ? mlp2_bwd_rows_direct_as<true>(a, s) : mlp2_bwd_rows_direct_as<false>(a, s);
}

}  // namespace xmoe
