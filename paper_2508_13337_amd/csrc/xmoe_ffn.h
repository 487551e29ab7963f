// Internal interface between the expert-MLP entry points and their two kernel families.
#pragma once

#include "xmoe_internal.h"
#include "xmoe_sizes.h"

namespace xmoe {

struct FfnArgs {
    int B, E, d, f, dt;
    const int32_t* off;          // expert_offsets [E+1], device
    const void *xd, *wg, *wu, *wd;
    const int32_t* row_index;    // NULL, or: xd is the token matrix and row i of the expert input is xd[row_index[i]]
    // forward: outputs g, u, y; backward: inputs g, u, dy and outputs dxd, dwg, dwu, dwd
    void *g, *u, *y;
    const void* dy;
    // backward: NULL, or dy is the [T,d] gradient of the layer's output and row i of dY is dy_scale[i] * dy[dy_index[i]]
    const int32_t* dy_index;
    const float* dy_scale;       // NULL = 1
    void *dxd, *dwg, *dwu, *dwd;
    // workspace carve-up
    int32_t* map;                // tile map
    int32_t* sched;              // experts by descending row count [E], then kSchedCounters counters
    void *act, *dg, *du;         // A = silu(G)*U, dG, dU   [B,f]
    // backward, optional: row_grad [B] (caller's) receives <unscaled row of dY, Y[row]> for every row; row_part is
    // the workspace for its partial sums, row_grad_parts(f) x B floats laid out [part][row]
    float* row_grad;
    float* row_part;
};

// the two-matrix expert (xmoe_expert_mlp2_fwd / _bwd)
struct Mlp2Args {
    int B, E, d, f, dt, act;
    const int32_t* off;          // expert_offsets [E+1], device
    const void *xd, *w1, *w2;
    const int32_t* row_index;    // as in FfnArgs
    void *h, *y;                 // forward: outputs; backward: h is an input
    const void* dy;
    const int32_t* dy_index;     // as in FfnArgs
    const float* dy_scale;
    void *dxd, *dw1, *dw2;
    int32_t* map;
    int32_t* sched;
    void *a_buf, *dh;            // A = act(H), dH   [B,f]
    float* row_grad;             // as in FfnArgs
    float* row_part;
};

// Weight gradients of the 128- and 64-row kernels: dW_e[m, n] = sum over the expert's rows r of P[r, m] * Q[r, n].  All of a
// call's are one launch, the experts with the most rows first (sched), so the long sums start early and only one tail of idle
// CUs is left.  A matrix's tiles are cut into at most eight runs, dealt to the XCDs in turn (block b runs on XCD b % 8): the
// tiles of a run share operand panels in one L2.
template <typename T>
struct WgradJob {
    const T *P, *Q;
    const int32_t *p_index, *q_index;   // or NULL; at most one
    int M, N;
    T* dW;
};
template <typename T>
struct WgradJobs {
    WgradJob<T> job[3];
    int n_jobs, tiles, run, runs;   // tiles of a matrix, tiles of a run, runs of a matrix
    // matrix m of all (jobs of the first expert in sched's order, of the second ...) and its tile u for this block
    __device__ __forceinline__ bool place(int E, int& m, int& u) const {
        const int s = blockIdx.x >> 3, r = (s / run) * 8 + (blockIdx.x & 7);   // run r of all
        m = r / runs;
        u = (r - m * runs) * run + s % run;
        return m < n_jobs * E && u < tiles;
    }
    // tile x tile outputs per block; the launch's grid
    dim3 cut(int E, int d, int f, int tile) {
        tiles = ((d + tile - 1) / tile) * ((f + tile - 1) / tile);
        run = (tiles + 7) / 8;
        runs = (tiles + run - 1) / run;
        return dim3((unsigned)(((long long)n_jobs * E * runs + 7) / 8 * 8 * run));
    }
};
template <typename T>
WgradJobs<T> wgrad_jobs(const FfnArgs& a) {
    return {{{(const T*)a.act, (const T*)a.dy, nullptr, a.dy_index, a.f, a.d, (T*)a.dwd},
             {(const T*)a.xd, (const T*)a.dg, a.row_index, nullptr, a.d, a.f, (T*)a.dwg},
             {(const T*)a.xd, (const T*)a.du, a.row_index, nullptr, a.d, a.f, (T*)a.dwu}},
            3};
}
template <typename T>
WgradJobs<T> wgrad_jobs(const Mlp2Args& a) {
    return {{{(const T*)a.a_buf, (const T*)a.dy, nullptr, a.dy_index, a.f, a.d, (T*)a.dw2},
             {(const T*)a.xd, (const T*)a.dh, a.row_index, nullptr, a.d, a.f, (T*)a.dw1}},
            2};
}

// sigmoid with the hardware exp2 and reciprocal (each good to about 1 ulp): the results are rounded to bf16, and
// the library-grade expf and IEEE division cost as much as a quarter of a tile's main loop in the fused epilogues.
__device__ __forceinline__ float fast_sigmoid(float g) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * g));
}

// activation of the matrix-core epilogues: silu takes the hardware exp2 / reciprocal like the SwiGLU epilogues
// and gelu takes the error function from the rational approximation 7.1.26 of Abramowitz and Stegun
//   erf(x) = 1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-x^2),  t = 1 / (1 + p x),  x >= 0,  |error| <= 1.5e-7,
// far below half a bf16 unit of the stored result; its exp(-x^2) with x = h / sqrt(2) is also the Gaussian density
// that the derivative needs.
__device__ __forceinline__ void fast_gelu_parts(float h, float& Phi, float& phi) {
    const float x = fabsf(h) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * x);
    const float e = __builtin_amdgcn_exp2f(-1.44269504088896341f * x * x);
    const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
    const float erf_abs = 1.0f - poly * e;
    Phi = 0.5f * (1.0f + copysignf(erf_abs, h));
    phi = 0.39894228040143268f * e;
}
template <int ACT>
__device__ __forceinline__ float act_fast(float h) {
    if (ACT == XMOE_ACT_SILU) return h * fast_sigmoid(h);
    if (ACT == XMOE_ACT_GELU) {
        float Phi, phi;
        fast_gelu_parts(h, Phi, phi);
        return h * Phi;
    }
    return h;
}
template <int ACT>
__device__ __forceinline__ void act_fast_grad(float h, float& a, float& g) {
    if (ACT == XMOE_ACT_SILU) {
        const float sg = fast_sigmoid(h);
        a = h * sg;
        g = sg * (1.0f + h * (1.0f - sg));
    } else if (ACT == XMOE_ACT_GELU) {
        float Phi, phi;
        fast_gelu_parts(h, Phi, phi);
        a = h * Phi;
        g = Phi + h * phi;
    } else {
        a = h;
        g = 1.0f;
    }
}

// rank: the experts' order too (the backward's weight gradients)
int launch_tile_map(const int32_t* off, int E, int tile_rows, int max_tiles, int32_t* map, int32_t* sched, bool rank,
                    hipStream_t s);

// row_grad[i] = sum over p < parts of row_part[p * B + i], p ascending (fixed order: the result is reproducible)
int launch_row_grad_reduce(const float* row_part, int parts, int B, float* row_grad, hipStream_t s);

int ffn_fwd_tile(const FfnArgs& a, hipStream_t s);
int ffn_bwd_tile(const FfnArgs& a, hipStream_t s);

// bf16 MFMA family (needs d % 64 == 0, f % 64 == 0 and 16-byte aligned operands): 256x256 tiles, operands streamed
// global -> LDS directly, transposing LDS reads
bool ffn_dma_supported(const FfnArgs& a);
int ffn_fwd_dma(const FfnArgs& a, hipStream_t s);
int ffn_bwd_dma(const FfnArgs& a, hipStream_t s);
int ffn_bwd_wgrads_dma(const FfnArgs& a, hipStream_t s);   // the weight gradients only, once dG, dU and A exist

// forward products of experts with few rows (the same operands as the direct-to-LDS kernels)
bool few_rows(int B, int E);
int ffn_fwd_few(const FfnArgs& a, hipStream_t s);
int mlp2_fwd_few(const Mlp2Args& a, hipStream_t s);

// 128-row tiles with direct-to-LDS loads (bf16, d % 8 == 0, f % 8 == 0 and 16-byte aligned operands): the whole forward, and
// the backward's row products (tile map, dAct with the row scales' gradient, dX) without the weight gradients
bool direct_fwd(int B, int E, int d, int f);   // whether they take a call's row products from the 256-row kernels
bool direct_bwd(int B, int E, int d, int f, int matrices);       // matrices of an expert: 3, or 2 (mlp2)
bool direct_wgrads(int B, int E, int d, int f, int matrices);    // and, behind direct_bwd, its weight gradients
bool direct_supported(const FfnArgs& a);
bool direct_supported(const Mlp2Args& a);
int ffn_fwd_direct(const FfnArgs& a, hipStream_t s);
int ffn_bwd_rows_direct(const FfnArgs& a, hipStream_t s);
int ffn_bwd_wgrads_direct(const FfnArgs& a, hipStream_t s);   // the weight gradients, behind the row products
int mlp2_fwd_direct(const Mlp2Args& a, hipStream_t s);
int mlp2_bwd_rows_direct(const Mlp2Args& a, hipStream_t s);
int mlp2_bwd_wgrads_direct(const Mlp2Args& a, hipStream_t s);

int mlp2_fwd_tile(const Mlp2Args& a, hipStream_t s);
int mlp2_bwd_tile(const Mlp2Args& a, hipStream_t s);
bool mlp2_dma_supported(const Mlp2Args& a);
int mlp2_fwd_dma(const Mlp2Args& a, hipStream_t s);
int mlp2_bwd_dma(const Mlp2Args& a, hipStream_t s);
int mlp2_bwd_wgrads_dma(const Mlp2Args& a, hipStream_t s);

}  // namespace xmoe
