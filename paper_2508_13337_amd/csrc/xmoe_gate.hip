// Gating of the padding-free MoE layer (paper: Listing 1 gating(); Appendix B.3 "Padding-free Gating"):
// gate projection in a fixed float32 order, softmax + top-k routing, and their backward.
#include <type_traits>

#include "xmoe_internal.h"
#include "xmoe_sizes.h"

namespace xmoe {

// =========================================================================================================
// gate projection, fixed summation order
// =========================================================================================================
// The contract: partial l (0..63) of a (token, expert) pair absorbs i = l, l+64, ... in ascending order, one fused
// multiply-add each; the 64 partials are folded by halving.  For one l that is a [tokens x d/64] x [d/64 x experts]
// product whose terms are added one at a time, which is what the matrix instructions with K = 1 compute: one fused
// multiply-add per output and instruction, with several independent blocks per instruction (v_mfma_f32_32x32x1_2b_f32,
// v_mfma_f32_16x16x1_4b_f32).  The blocks take l, l+32 (TL = 32) or l, l+16, l+32, l+48 (TL = 16).  Same bits as the
// plain loop, at twice the rate of the float32 ALUs without packed instructions.
//
//   block = 8 waves, TL tokens x TL experts.  Wave w owns the pairs l = 2(w%4) + {0, 1} + 8(w/4) (+ the blocks' offsets,
//   + 16 for TL = 32), so that one LDS read of x serves two instructions; offsets 32 and 16 of the fold stay in
//   registers, 8 to 1 go through LDS.  A stage is 16 KiB of either operand, 512 bytes (TL = 32) or 1 KiB (TL = 16) of
//   i per token, fetched one stage ahead through registers.  x past d reads +0 and w past d -0: their product -0 leaves
//   every sum as it is, -0 included.
//
// Bound: TL = 32 by the barriers between its stages: about 180 registers leave one block of 8 waves per CU, and nothing
// runs over them (61 to 72 TFLOP/s, the matrix cores busy 36 %); TL = 16 (few tokens) by the latency of its stages.
// Measured (MI355X, bf16, 64 experts, d 2048; float32 ALUs, operands staged through LDS a 64-wide chunk at a time | this):
// T 8: 19 | 9 us, T 509: 19 | 10, T 8192: 52 | 35, T 65536: 334 | 238; d 1000, 24 experts, T 3001: 12 | 8.
typedef __attribute__((ext_vector_type(32))) float gate_f32x32_t;
template <int TL>
struct GateMma;
template <>
struct GateMma<32> {
    typedef gate_f32x32_t Acc;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x1f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int v) { return 8 * (v >> 2) + 4 * ((threadIdx.x >> 5) & 1) + (v & 3); }
};
template <>
struct GateMma<16> {
    typedef __attribute__((ext_vector_type(16))) float Acc;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int v) { return 4 * ((threadIdx.x >> 4) & 3) + v; }
};

// 16 bytes from an address that is aligned to one element only
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) GateVec {
    uint32_t v[4];
};
__device__ __forceinline__ uint32_t gate_bits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t gate_bits(bf16_t v) { return v.bits; }
// the vector at p of which the first n elements exist; `fill` stands for the others
template <typename T>
__device__ __forceinline__ uint4 gate_load(const T* __restrict__ p, int n, uint32_t fill) {
    constexpr int EV = 16 / sizeof(T);
    if (n >= EV) {
        const GateVec<T> q = *reinterpret_cast<const GateVec<T>*>(p);
        return make_uint4(q.v[0], q.v[1], q.v[2], q.v[3]);
    }
    uint32_t s[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < EV; ++j) s[j * 4 / EV] |= (j < n ? gate_bits(p[j]) : fill) << (EV == 8 ? 16 * (j & 1) : 0);
    return make_uint4(s[0], s[1], s[2], s[3]);
}

// what stands past d: +0 for x, -0 for w in bf16 and in float32
__device__ __align__(16) const uint32_t kGatePad[12] = {0, 0, 0, 0, 0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u,
                                                        0x80000000u, 0x80000000u, 0x80000000u, 0x80000000u};
// explicitly global, whichever of the two a lane reads: a flat load would count as an LDS access as well
typedef const __attribute__((address_space(1))) char* gate_gptr;
template <typename T>
__device__ __forceinline__ uint4 gate_load16(gate_gptr p) {
    const auto* q = reinterpret_cast<const __attribute__((address_space(1))) GateVec<T>*>(p);
    return make_uint4(q->v[0], q->v[1], q->v[2], q->v[3]);
}

__device__ __forceinline__ void gate_pair(const bf16_t* p, float& a, float& b) {
    const uint32_t u = *reinterpret_cast<const uint32_t*>(p);
    a = __uint_as_float(u << 16);
    b = __uint_as_float(u & 0xffff0000u);
}
__device__ __forceinline__ void gate_pair(const float* p, float& a, float& b) {
    const float2 v = *reinterpret_cast<const float2*>(p);
    a = v.x;
    b = v.y;
}

// TL = 32 from this many of its blocks on (one per CU) and from 17 experts on.  Below, tiles of a quarter of the size
// spread over more of the chip, and a stage is twice as deep; up to 16 experts the larger tile would spend half of its
// matrix work or more on columns that do not exist (bf16 d 2048, T 8192 | 32768, us at TL = 32, at 16: 8 experts 18 | 62,
// 12 | 39; 4 experts d 512, T 32768: 33, 18).
constexpr long kGateBigBlocks = 256;

template <typename T, int TL, bool VECX, bool VECW>
__global__ __launch_bounds__(512, 2) void gate_logits_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                             const float* __restrict__ bias,
                                                             float* __restrict__ logits, int Tn, int d, int E) {
    using M = GateMma<TL>;
    constexpr int EV = 16 / sizeof(T);
    constexpr int NBLK = 64 / TL, NJ = TL / 16;            // blocks per instruction; values of l per wave and parity
    constexpr int CH = 16384 / (TL * 64 * (int)sizeof(T)); // 64-wide chunks of i per stage
    constexpr int KI = CH * 64;
    constexpr int VX = KI / EV, VW = TL / EV;              // vectors per row of x, of w
    constexpr int XS = KI + EV;                            // elements per staged token
    static_assert(TL * VX == 1024 && KI * VW == 1024, "two vectors of either operand per thread");
    constexpr int kXBytes = TL * XS * (int)sizeof(T);
    constexpr int kStage = kXBytes + 16384;
    __shared__ __align__(16) char smem[2 * kStage];
    static_assert(2 * kStage >= 16 * TL * TL * 4, "the fold reuses the stages");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.x * TL, e0 = blockIdx.y * TL;
    const int b = lane / TL, c = lane % TL;

    uint4 rx[2], rw[2];
    auto fetch = [&](int i0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int v = tid + 512 * q;
            int t = t0 + v / VX;
            t = t < Tn ? t : Tn - 1;      // rows past the last one repeat it; what they give is not stored
            const int ix = i0 + (v % VX) * EV, iw = i0 + v / VW, e = e0 + (v % VW) * EV;
            if (VECX) {   // no vector straddles an end: those past it come from the pad
                const gate_gptr px = (gate_gptr)(const char*)(x + (size_t)t * d + ix);
                rx[q] = gate_load16<T>(ix < d ? px : (gate_gptr)(const char*)kGatePad);
            } else {
                rx[q] = gate_load(x + (size_t)t * d + ix, d - ix, 0u);
            }
            if (VECW) {
                const gate_gptr pw = (gate_gptr)(const char*)(w + (size_t)iw * E + (e < E ? e : 0));
                rw[q] = gate_load16<T>(iw < d ? pw : (gate_gptr)(const char*)(kGatePad + (sizeof(T) == 2 ? 4 : 8)));
            } else {
                rw[q] = gate_load(w + (size_t)iw * E + e, iw < d ? E - e : 0, sizeof(T) == 2 ? 0x8000u : 0x80000000u);
            }
        }
    };
    auto stage = [&](int buf) {
        T* sx = reinterpret_cast<T*>(smem + buf * kStage);
        T* sw = reinterpret_cast<T*>(smem + buf * kStage + kXBytes);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int v = tid + 512 * q;
            *reinterpret_cast<uint4*>(sx + (v / VX) * XS + (v % VX) * EV) = rx[q];
            *reinterpret_cast<uint4*>(sw + v * EV) = rw[q];
        }
    };

    typename M::Acc acc[NJ][2];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int v = 0; v < 16 * NJ; ++v) acc[j][s][v] = 0.f;

    const int l0 = 2 * (wave & 3) + 8 * (wave >> 2);
    auto multiply = [&](int g) {
        const T* sx = reinterpret_cast<const T*>(smem + (g & 1) * kStage) + c * XS + TL * b + l0;
        const T* sw = reinterpret_cast<const T*>(smem + (g & 1) * kStage + kXBytes) + (TL * b + l0) * TL + c;
        auto chunk = [&](int q) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                float a[2];
                gate_pair(sx + q * 64 + 16 * j, a[0], a[1]);
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    acc[j][s] = M::mma(a[s], to_float(sw[(q * 64 + 16 * j + s) * TL]), acc[j][s]);
            }
        };
        // unrolled: the reads of later chunks run under the matrix instructions of earlier ones
#pragma unroll
        for (int q = 0; q < CH; ++q) chunk(q);
    };
    const int stages = (d + KI - 1) / KI;
    fetch(0);
    stage(0);
    __syncthreads();
    for (int g = 0; g + 1 < stages; ++g) {
        fetch((g + 1) * KI);
        __builtin_amdgcn_sched_barrier(0);   // the loads stay in front of the matrix instructions they run under
        multiply(g);
        stage((g + 1) & 1);
        // the stage written above is read after this barrier; its buffer was last read before the previous one
        __syncthreads();
    }
    multiply(stages - 1);
    __syncthreads();

    // fold: offset 32 between the blocks, 16 between the blocks (TL = 16) or the j (TL = 32), then 8, 4, 2, 1 over the
    // waves' sums red[l][token][expert], l = 0..15
    float* red = reinterpret_cast<float*>(smem);
    constexpr int NV = TL * TL / 64;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            float p;
            if (TL == 32)
                p = (acc[0][s][v] + acc[0][s][NV + v]) + (acc[NJ - 1][s][v] + acc[NJ - 1][s][NV + v]);
            else
                p = (acc[0][s][v] + acc[0][s][2 * NV + v]) + (acc[0][s][NV + v] + acc[0][s][(3 * NV + v) & (16 * NJ - 1)]);
            red[((l0 + s) * TL + M::row(v)) * TL + c] = p;
        }
    __syncthreads();
    for (int o = tid; o < TL * TL; o += 512) {
        float p[16];
#pragma unroll
        for (int l = 0; l < 16; ++l) p[l] = red[l * TL * TL + o];
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
            for (int l = 0; l < off; ++l) p[l] = p[l] + p[l + off];
        const int t = t0 + o / TL, e = e0 + o % TL;
        if (t < Tn && e < E) logits[(size_t)t * E + e] = bias ? p[0] + bias[e] : p[0];
    }
}

// =========================================================================================================
// softmax + top-k: one wave per token
// =========================================================================================================
// Bound by the chain of k wave-wide maxima: on the vector ALU's lane moves (six 32-bit maxima, then ballots for the lane)
// instead of 64-bit exchanges through LDS.  E 64, k 6, T 8192: 10.4 -> 5.1 us.
constexpr int kMaxPerLane = XMOE_MAX_EXPERTS / 64;   // 8

// order-preserving bit pattern of a float; -0.0 and +0.0 compare equal as numbers, so both map to +0.0's key and
// the lower expert index decides between them like any other tie
__device__ __forceinline__ uint32_t order_key(float v) {
    uint32_t u = __float_as_uint(v);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
// the largest of the wave's values, wave-uniform: lane moves of the vector ALU, which cost no LDS traffic
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    auto step = [&](auto ctrl, auto rows) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xf,
                                                                 false);
        v = o > v ? o : v;
    };
    typedef std::integral_constant<int, 0xf> all;
    step(std::integral_constant<int, 0x111>{}, all{});   // row_shr 1, 2, 4, 8: lane 15 of a row holds the row's maximum
    step(std::integral_constant<int, 0x112>{}, all{});
    step(std::integral_constant<int, 0x114>{}, all{});
    step(std::integral_constant<int, 0x118>{}, all{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast 15 into rows 1 and 3
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});   // row_bcast 31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

template <int PER_LANE>
__global__ __launch_bounds__(256) void route_kernel(const float* __restrict__ logits, int Tn, int E, int k,
                                                    int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= Tn) return;
    const float* row = logits + (size_t)t * E;
    float l[PER_LANE];
    // order-preserving bits of the logits; 0 stands for a column that does not exist or has been selected, and is the key of
    // one logit, the NaN of all ones.  The largest key wins, and among equal ones the lowest expert, i.e. the first lane of
    // the first j.
    uint32_t key[PER_LANE];
#pragma unroll
    for (int j = 0; j < PER_LANE; ++j) {
        const int e = lane + 64 * j;
        l[j] = e < E ? row[e] : -INFINITY;
        key[j] = e < E ? order_key(l[j]) : 0u;
    }
    auto wave_best = [&] {
        uint32_t best = 0u;
#pragma unroll
        for (int j = 0; j < PER_LANE; ++j) best = key[j] > best ? key[j] : best;
        return wave_max_u32(best);
    };
    auto logit_of = [](uint32_t ob) { return __uint_as_float((ob & 0x80000000u) ? (ob & 0x7fffffffu) : ~ob); };
    uint32_t best = wave_best();
    const float m = logit_of(best);
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < PER_LANE; ++j) s += (lane + 64 * j < E) ? expf(l[j] - m) : 0.f;
    s = wave_sum(s);
    const float inv = 1.0f / s;

    int my_idx = 0;
    float my_w = 0.f;
    int slot = 0;
    for (; slot < k; ++slot) {
        if (best == 0u) break;   // wave-uniform, as `best` is
        int e = 0;
        bool found = false;
#pragma unroll
        for (int j = 0; j < PER_LANE; ++j) {
            const unsigned long long who = __ballot(key[j] == best);
            if (!found && who) {   // wave-uniform
                found = true;
                const int winner = __ffsll((long long)who) - 1;
                e = winner + 64 * j;
                if (lane == winner) key[j] = 0u;   // retired
            }
        }
        if (lane == slot) {
            my_idx = e;
            my_w = expf(logit_of(best) - m) * inv;
        }
        if (slot + 1 < k) best = wave_best();
    }
    // only NaNs of all ones are left: by ascending expert
    for (int last = -1; slot < k; ++slot) {
        int e = E;
#pragma unroll
        for (int j = PER_LANE - 1; j >= 0; --j) {
            const unsigned long long who = __ballot(__float_as_uint(l[j]) == 0xffffffffu && lane + 64 * j > last);
            if (who) e = __ffsll((long long)who) - 1 + 64 * j;
        }
        last = e;
        if (lane == slot) {
            my_idx = e;
            my_w = logit_of(0u);
        }
    }
    if (lane < k) {
        topk_idx[(size_t)t * k + lane] = my_idx;
        topk_w[(size_t)t * k + lane] = my_w;
    }
}

// backward of softmax + top-k (indices constant): one wave per token.  ROWS: the combine weights' gradient comes row by row
// (grad[row_of_slot], 0 for a dropped entry) and goes out slot by slot (dw) on the way; otherwise grad is dw itself.
template <int PER_LANE, bool ROWS>
__global__ __launch_bounds__(256) void route_bwd_kernel(const float* __restrict__ logits,
                                                        const int32_t* __restrict__ topk_idx,
                                                        const float* __restrict__ grad,
                                                        const int32_t* __restrict__ row_of_slot, int Tn, int E, int k,
                                                        float* __restrict__ dw, float* __restrict__ dlogits) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= Tn) return;
    const float* row = logits + (size_t)t * E;
    // slot `lane`'s expert and gradient
    int my_e = 0;
    float my_g = 0.f;
    if (lane < k) {
        const size_t n = (size_t)t * k + lane;
        my_e = topk_idx[n];
        if (ROWS) {
            const int r = row_of_slot[n];
            my_g = r >= 0 ? grad[r] : 0.f;
            dw[n] = my_g;
        } else {
            my_g = grad[n];
        }
    }
    float p[PER_LANE], dp[PER_LANE];
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < PER_LANE; ++j) {
        int e = lane + 64 * j;
        p[j] = e < E ? row[e] : -INFINITY;
        dp[j] = 0.f;
        m = fmaxf(m, p[j]);
    }
    m = wave_max(m);
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < PER_LANE; ++j) {
        p[j] = (lane + 64 * j < E) ? expf(p[j] - m) : 0.f;
        s += p[j];
    }
    s = wave_sum(s);
    const float inv = 1.0f / s;
#pragma unroll
    for (int j = 0; j < PER_LANE; ++j) p[j] *= inv;
    for (int slot = 0; slot < k; ++slot) {
        const int e = __shfl(my_e, slot, 64);
        const float g = __shfl(my_g, slot, 64);
#pragma unroll
        for (int j = 0; j < PER_LANE; ++j)
            if (lane + 64 * j == e) dp[j] += g;
    }
    float inner = 0.f;
#pragma unroll
    for (int j = 0; j < PER_LANE; ++j) inner += p[j] * dp[j];
    inner = wave_sum(inner);
#pragma unroll
    for (int j = 0; j < PER_LANE; ++j) {
        int e = lane + 64 * j;
        if (e < E) dlogits[(size_t)t * E + e] = p[j] * (dp[j] - inner);
    }
}

// =========================================================================================================
// backward of the gate projection
// =========================================================================================================
// Both GEMMs of the gate projection's backward run on the float32 matrix instruction v_mfma_f32_32x32x2_f32 (the
// operands are dlogits, float32, and x / w_router widened exactly to float32, so nothing is rounded before the
// float32 accumulation).  A lane supplies one element of each operand per instruction: lane l holds
// A[row l%32][k = l/32] and B[k = l/32][column l%32], and ends up with 16 results
// D[row 8*(v/4) + 4*(l/32) + v%4][column l%32], v = 0..15.
typedef __attribute__((ext_vector_type(16))) float gate_f32x16_t;

// An element, or two consecutive ones, of a row as float32, zero where !ok.  The address is what depends on ok: with a
// branch around each load the compiler waits for one load before it issues the next.
__device__ __forceinline__ float load_or_zero(const bf16_t* p, bool ok) {
    const gate_gptr a = ok ? (gate_gptr)(const char*)p : (gate_gptr)(const char*)kGatePad;
    return bf16_bits_to_float(*reinterpret_cast<const __attribute__((address_space(1))) uint16_t*>(a));
}
__device__ __forceinline__ float load_or_zero(const float* p, bool ok) {
    const gate_gptr a = ok ? (gate_gptr)(const char*)p : (gate_gptr)(const char*)kGatePad;
    return *reinterpret_cast<const __attribute__((address_space(1))) float*>(a);
}
// VEC: one 4-byte (bf16) / 8-byte (float) load, ok0 standing for both
template <bool VEC>
__device__ __forceinline__ void load_pair(const bf16_t* p, bool ok0, bool ok1, float& a, float& b) {
    if (VEC) {
        const gate_gptr q = ok0 ? (gate_gptr)(const char*)p : (gate_gptr)(const char*)kGatePad;
        const uint32_t u = *reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(q);
        a = __uint_as_float(u << 16);
        b = __uint_as_float(u & 0xffff0000u);
    } else {
        a = load_or_zero(p, ok0);
        b = load_or_zero(p + 1, ok1);
    }
}
template <bool VEC>
__device__ __forceinline__ void load_pair(const float* p, bool ok0, bool ok1, float& a, float& b) {
    if (VEC) {
        const gate_gptr q = ok0 ? (gate_gptr)(const char*)p : (gate_gptr)(const char*)kGatePad;
        const uint64_t u = *reinterpret_cast<const __attribute__((address_space(1))) uint64_t*>(q);
        a = __uint_as_float((uint32_t)u);
        b = __uint_as_float((uint32_t)(u >> 32));
    } else {
        a = load_or_zero(p, ok0);
        b = load_or_zero(p + 1, ok1);
    }
}

// The same from an address that is always readable (p[0] and p[o1]); IN: both elements are known to exist.
template <bool VEC, bool IN, typename T>
__device__ __forceinline__ void take_pair(const T* p, int o1, bool ok0, bool ok1, float& a, float& b) {
    if (VEC) {
        gate_pair(p, a, b);
    } else {
        a = to_float(p[0]);
        b = to_float(p[IN ? 1 : o1]);
    }
    if (!IN) {
        a = ok0 ? a : 0.f;
        b = ok1 ? b : 0.f;
    }
}

// partial[s][i][e] = sum over the s-th slice of tokens of x[t,i] * dlogits[t,e]
// The summation index is the token, and both operands are stored token-major, so a half-wave reads consecutive
// elements of one token's row: no transposition.  A block owns 64 rows i x 64 columns e of one slice.  The rows and
// columns of an instruction's 32 x 32 block are interleaved with those of its neighbour (row r of block a is
// i0 + 2r + a, column c of block b is e0 + 2c + b), so that one 4-byte load of x and one 8-byte load of dlogits
// per lane feed four instructions.  The block's four waves take interleaved runs of 16 tokens each (enough waves in
// flight to hide the loads' latency), and their partial tiles are added through LDS in wave order.
// Bound by the latency of its loads where the blocks are few: all of a round's are issued before the first is waited for
// (with a branch around each for the edges they were waited for one by one: float32 T 256 d 128 E 8 15 -> 11 us, T 2048
// d 1024 E 16 16 -> 12).  Rounds whose tokens all exist fetch without a choice of address; columns past the end of d or E
// read an element that exists and are cleared.
// grid = (ceil(d/64), ceil(E/64), splits).  VECX, VECE: the pairs of x, of dlogits may be fetched with one load.
// MODE:
//   DW_FREE   whole rounds in the compiler's own order: other waves hide the latency, and loads sunk between the matrix
//             instructions take fewer registers.  float32 from 512 blocks on, us without | with it: T 16384 d 1000 E 256
//             173 | 111, T 3001 36 | 27, T 16384 d 2048 E 64 85 | 62 (1024 blocks); below: T 3001 d 1000 E 64 (192
//             blocks) 12 | 17, T 65536 d 128 E 64 (64) 44 | 107.  bf16: 115 | 117 at d 1000 E 256, 32 | 52 at E 64.
//   DW_TAIL   no slice has a whole round (T < 16): the code for them is left out (0.7 us of 7.5)
enum DwMode { DW_BATCH = 0, DW_FREE = 1, DW_TAIL = 2 };
template <typename T, bool VECX, bool VECE, int MODE>
__global__ __launch_bounds__(256, MODE == DW_FREE ? 4 : 1) void gate_bwd_dw_kernel(const T* __restrict__ x, const float* __restrict__ dl,
                                                          float* __restrict__ partial, int Tn, int d, int E,
                                                          int t_per_split) {
    __shared__ float red[4][32][64];   // [wave][accumulator register][lane], used once per row block a
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = blockIdx.x * 64, e0 = blockIdx.y * 64;
    const int tb = blockIdx.z * t_per_split;
    int te = tb + t_per_split;
    te = te < Tn ? te : Tn;
    const int h = lane >> 5, c = lane & 31;
    const int ia = i0 + 2 * c, ea = e0 + 2 * c;
    const bool ok_i0 = ia < d, ok_i1 = ia + 1 < d, ok_e0 = ea < E, ok_e1 = ea + 1 < E;
    const T* xa = x + (ok_i0 ? ia : 0);
    const float* ba = dl + (ok_e0 ? ea : 0);
    gate_f32x16_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    constexpr int U = 8;   // instructions' worth of operands fetched before the first is used
    const int o_i = ok_i1 ? 1 : 0, o_e = ok_e1 ? 1 : 0;
    // t_in: all of the round's tokens exist; x_in, e_in: so do all of the block's rows i (columns e)
    auto round = [&](auto t_in, auto x_in, auto e_in, int t0) {
        float av[U][2], bv[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + 2 * u + h;
            const bool ok_t = decltype(t_in)::value || t < te;
            const T* px = xa + (size_t)(ok_t ? t : tb) * d;
            const float* pb = ba + (size_t)(ok_t ? t : tb) * E;
            if (decltype(t_in)::value) {
                take_pair<VECX, decltype(x_in)::value>(px, o_i, ok_i0, ok_i1, av[u][0], av[u][1]);
                take_pair<VECE, decltype(e_in)::value>(pb, o_e, ok_e0, ok_e1, bv[u][0], bv[u][1]);
            } else {
                load_pair<VECX>(px, ok_t && ok_i0, ok_t && ok_i1, av[u][0], av[u][1]);
                load_pair<VECE>(pb, ok_t && ok_e0, ok_t && ok_e1, bv[u][0], bv[u][1]);
            }
        }
        // all of them in flight before the first is waited for
        if (MODE != DW_FREE || !decltype(x_in)::value || !decltype(e_in)::value) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u][a], bv[u][b], acc[a][b], 0, 0, 0);
    };
    int t0 = tb + wave * 2 * U;
    auto full_rounds = [&](auto x_in, auto e_in) {
        for (; t0 + 2 * U <= te; t0 += 4 * 2 * U) round(std::true_type{}, x_in, e_in, t0);
    };
    if (MODE != DW_TAIL) {
        if (i0 + 64 <= d && e0 + 64 <= E)
            full_rounds(std::true_type{}, std::true_type{});
        else if (i0 + 64 <= d)
            full_rounds(std::true_type{}, std::false_type{});
        else
            full_rounds(std::false_type{}, std::false_type{});
    }
    for (; t0 < te; t0 += 4 * 2 * U) round(std::false_type{}, std::false_type{}, std::false_type{}, t0);
    float* out = partial + (size_t)blockIdx.z * d * E;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            red[wave][v][lane] = acc[a][0][v];
            red[wave][16 + v][lane] = acc[a][1][v];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int n = threadIdx.x + 256 * r;   // (accumulator register, lane) pair
            const int reg = n >> 6, l = n & 63;
            const float sum = ((red[0][reg][l] + red[1][reg][l]) + red[2][reg][l]) + red[3][reg][l];
            const int v = reg & 15;
            const int i = i0 + 2 * (8 * (v >> 2) + 4 * (l >> 5) + (v & 3)) + a;
            const int e = e0 + 2 * (l & 31) + (reg >> 4);
            if (i < d && e < E) out[(size_t)i * E + e] = sum;
        }
        __syncthreads();
    }
}

template <typename T>
__global__ __launch_bounds__(256) void gate_bwd_dw_reduce_kernel(const float* __restrict__ partial, int splits,
                                                                 size_t n, T* __restrict__ dwr) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    // eight loads at a time in flight, added in ascending order (d 2048, E 64, 32 partials: 10.5 -> 5.2 us)
    float s = 0.f;
    int sp = 0;
    for (; sp + 8 <= splits; sp += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = partial[(size_t)(sp + q) * n + i];
#pragma unroll
        for (int q = 0; q < 8; ++q) s += v[q];
    }
    for (; sp < splits; ++sp) s += partial[(size_t)sp * n + i];
    dwr[i] = from_float<T>(s);
}

// dx_gate[t,i] = sum_e dlogits[t,e] * w[i,e]
// The summation index e is contiguous in both operands.  The instruction sums over its two k-slots and the loop
// over its steps, so any assignment of experts to (step, slot) gives the same sum: slot h of step q takes expert
// 32*h + q of a chunk of 64, and a lane then reads 32 consecutive experts of its row with 16-byte loads.
// One wave: 32 tokens x up to kDxCols columns i; the token rows of dlogits stay in registers across the columns.
constexpr int kDxCols = 256;

// full: all 32 exist, whatever the alignment of the row (wave-uniform)
template <typename T>
__device__ __forceinline__ void load_row32(const T* __restrict__ p, int n_valid, bool full, float (&v)[32]);
template <>
__device__ __forceinline__ void load_row32<float>(const float* __restrict__ p, int n_valid, bool full,
                                                  float (&v)[32]) {
    if (full) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const GateVec<float> f = reinterpret_cast<const GateVec<float>*>(p)[q];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * q + j] = __uint_as_float(f.v[j]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 32; ++q) v[q] = load_or_zero(p + q, q < n_valid);
    }
}
template <>
__device__ __forceinline__ void load_row32<bf16_t>(const bf16_t* __restrict__ p, int n_valid, bool full,
                                                   float (&v)[32]) {
    if (full) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const GateVec<bf16_t> f = reinterpret_cast<const GateVec<bf16_t>*>(p)[q];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[8 * q + 2 * j] = __uint_as_float(f.v[j] << 16);
                v[8 * q + 2 * j + 1] = __uint_as_float(f.v[j] & 0xffff0000u);
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < 32; ++q) v[q] = load_or_zero(p + q, q < n_valid);
    }
}

// FEW: E < 64, no run of 32 is known to be complete (the code for complete ones left out: bf16 T 65536 d 2048 E 8
// 335 -> 247 us)
template <typename T, bool FEW>
__global__ __launch_bounds__(256) void gate_bwd_dx_kernel(const float* __restrict__ dl, const T* __restrict__ w,
                                                          T* __restrict__ dxg, int Tn, int d, int E, int cols) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = (blockIdx.x * 4 + wave) * 32;
    if (t0 >= Tn) return;
    const int h = lane >> 5, c = lane & 31;
    const int ibeg = blockIdx.y * cols;
    const int iend = ibeg + cols < d ? ibeg + cols : d;
    const bool ok_t = t0 + c < Tn;
    const float* arow = dl + (size_t)(ok_t ? t0 + c : 0) * E + 32 * h;
    const bool one_chunk = FEW || E <= 64;
    float av[32];
    // (full: rows past the last one read row 0 and are cleared)
    if (one_chunk) load_row32<float>(arow, ok_t ? E - 32 * h : 0, !FEW && E == 64, av);
    if (one_chunk && !ok_t) {
#pragma unroll
        for (int q = 0; q < 32; ++q) av[q] = 0.f;
    }
    for (int i0 = ibeg; i0 < iend; i0 += 32) {
        const bool ok_i = i0 + c < d;
        const T* brow = w + (size_t)(ok_i ? i0 + c : 0) * E + 32 * h;
        gate_f32x16_t acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        for (int e0 = 0; e0 < E; e0 += 64) {
            float bv[32];
            const int n_valid = E - e0 - 32 * h;   // experts left in this lane's run of 32
            if (!one_chunk) {
                load_row32<float>(arow + e0, ok_t ? n_valid : 0, !FEW && E - e0 >= 64, av);
                if (!ok_t) {
#pragma unroll
                    for (int q = 0; q < 32; ++q) av[q] = 0.f;
                }
            }
            load_row32<T>(brow + e0, ok_i ? n_valid : 0, !FEW && E - e0 >= 64, bv);
            if (!ok_i) {
#pragma unroll
                for (int q = 0; q < 32; ++q) bv[q] = 0.f;
            }
#pragma unroll
            for (int q = 0; q < 32; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[q], bv[q], acc, 0, 0, 0);
        }
        if (ok_i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = t0 + 8 * (v >> 2) + 4 * h + (v & 3);
                if (t < Tn) dxg[(size_t)t * d + i0 + c] = from_float<T>(acc[v]);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// The same two products for bf16 operands on the bf16 matrix instruction (16 summands per instruction and operand
// row instead of 2).  x and w are bf16 as stored; dlogits is float32 and goes in as the sum of two bf16 terms,
// hi = bf16(v) and lo = bf16(v - hi), i.e. with 16 significant bits: every product is exact in float32, the sums are
// float32, and what is dropped (2^-17 of a term) is far below the bf16 rounding of the results.
// Used when d % 64 == 0, E % 64 == 0 and the operands are 16-byte aligned; otherwise the kernels above.
// ---------------------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 gate_bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short gate_s16x4_t;
typedef __attribute__((ext_vector_type(8))) short gate_s16x8_t;

// v[0..7] -> hi and lo as packed bf16 pairs
__device__ __forceinline__ void split_bf16x8(const float (&v)[8], uint4& hi, uint4& lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        h[q] = pack_bf16x2(v[2 * q], v[2 * q + 1]);
        const float r0 = v[2 * q] - __uint_as_float(h[q] << 16);
        const float r1 = v[2 * q + 1] - __uint_as_float(h[q] & 0xffff0000u);
        l[q] = pack_bf16x2(r0, r1);
    }
    hi = make_uint4(h[0], h[1], h[2], h[3]);
    lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// partial[s][i][e] = sum over the s-th slice of tokens of x[t,i] * dlogits[t,e].  Both operands are stored
// token-major while the instruction wants 8 consecutive tokens per lane, so a block stages 64 tokens x (64 columns i
// of x, 64 experts of dlogits as hi and lo) in LDS as they lie in memory and takes its operands with the
// transposing LDS read.  Four waves: one 32 x 32 block of the 64 x 64 output each.  grid = (d/64, E/64, splits).
constexpr int kDwTok = 64;
constexpr int kDwStride = 144;   // bytes per staged token row: 64 bf16 + 16 bytes of padding

// operand for v_mfma_f32_32x32x16_bf16 from a token-major tile: column col_base + lane%32, tokens
// 16*ks + 8*(lane/32) .. +7.  In a group of 16 lanes, lane s addresses 4 consecutive columns (s%4) of token row
// (s/4); the transposing read hands every lane one column with 4 consecutive tokens.
__device__ __forceinline__ gate_bf16x8_t dw_frag(const char* tile, int col_base, int ks) {
    const int lane = threadIdx.x & 63;
    const int G = lane >> 4, s = lane & 15;
    const int col = col_base + 16 * (G & 1) + 4 * (s & 3);
    const int k0 = 16 * ks + 8 * (G >> 1) + (s >> 2);
    gate_s16x4_t h[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const char* a = tile + (k0 + 4 * q) * kDwStride + col * 2;
        h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) gate_s16x4_t*)(
            (__attribute__((address_space(3))) void*)a));
    }
    const gate_s16x8_t v = {h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]};
    return __builtin_bit_cast(gate_bf16x8_t, v);
}

__global__ __launch_bounds__(256) void gate_bwd_dw_mfma_kernel(const bf16_t* __restrict__ x,
                                                               const float* __restrict__ dl,
                                                               float* __restrict__ partial, int Tn, int d, int E,
                                                               int t_per_split) {
    __shared__ __align__(16) char xs[kDwTok * kDwStride];
    __shared__ __align__(16) char dhi[kDwTok * kDwStride];
    __shared__ __align__(16) char dlo[kDwTok * kDwStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.x * 64, e0 = blockIdx.y * 64;
    const int tb = blockIdx.z * t_per_split;
    int te = tb + t_per_split;
    te = te < Tn ? te : Tn;
    const int mi = wave >> 1, ni = wave & 1;
    // staging: token rows tid/8 and tid/8 + 32 of a chunk; 8 columns of x (16 bytes) and 8 experts of dlogits each
    const int sr = tid >> 3, sp = tid & 7;
    uint4 xr[2];
    float4 dr[2][2];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = t0 + sr + 32 * j;
            xr[j] = make_uint4(0, 0, 0, 0);
            dr[j][0] = dr[j][1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (t < te) {
                xr[j] = *reinterpret_cast<const uint4*>(x + (size_t)t * d + i0 + sp * 8);
                const float4* p = reinterpret_cast<const float4*>(dl + (size_t)t * E + e0 + sp * 8);
                dr[j][0] = p[0];
                dr[j][1] = p[1];
            }
        }
    };
    auto stage = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int o = (sr + 32 * j) * kDwStride + sp * 16;
            const float v[8] = {dr[j][0].x, dr[j][0].y, dr[j][0].z, dr[j][0].w,
                                dr[j][1].x, dr[j][1].y, dr[j][1].z, dr[j][1].w};
            uint4 hi, lo;
            split_bf16x8(v, hi, lo);
            *reinterpret_cast<uint4*>(xs + o) = xr[j];
            *reinterpret_cast<uint4*>(dhi + o) = hi;
            *reinterpret_cast<uint4*>(dlo + o) = lo;
        }
    };
    gate_f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    if (tb < te) fetch(tb);
    for (int t0 = tb; t0 < te; t0 += kDwTok) {
        stage();
        __syncthreads();
        if (t0 + kDwTok < te) fetch(t0 + kDwTok);   // in flight while this chunk is multiplied
#pragma unroll
        for (int ks = 0; ks < kDwTok / 16; ++ks) {
            const gate_bf16x8_t a = dw_frag(xs, 32 * mi, ks);
            const gate_bf16x8_t bh = dw_frag(dhi, 32 * ni, ks);
            const gate_bf16x8_t bl = dw_frag(dlo, 32 * ni, ks);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bl, acc, 0, 0, 0);
        }
        __syncthreads();   // everybody is done reading before the next chunk is staged
    }
    float* out = partial + (size_t)blockIdx.z * d * E;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int i = i0 + 32 * mi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        const int e = e0 + 32 * ni + (lane & 31);
        out[(size_t)i * E + e] = acc[v];
    }
}

// dx_gate[t,i] = sum_e dlogits[t,e] * w[i,e]: e is contiguous in both operands, so a lane takes its 8 consecutive
// experts straight from memory (dlogits: 8 floats -> hi, lo; w: 16 bytes).  One wave: 32 tokens x kDxCols columns.
// The wave's rows of dlogits are fetched and split once per 64 experts: for E == 64 they stay in registers across the
// column blocks; for larger E the chunks of 64 experts are the outer loop and the kDxCols / 32 column blocks keep
// an accumulator each.  (Fewer columns per wave, i.e. more and shorter waves, is slower: 64 columns 32 us against 26
// at config 2 - fetching and splitting the rows of dlogits costs more than short waves hide.)
// w is the instruction's first operand: the result block is [column i][token], so that a lane ends up with runs of 4
// consecutive columns of one token row and stores 8 bytes at a time.
constexpr int kDxColsManyExperts = 128;   // E > 64: four accumulators per wave (eight leave one wave per SIMD)
template <bool ONE_CHUNK>
__global__ __launch_bounds__(256) void gate_bwd_dx_mfma_kernel(const float* __restrict__ dl,
                                                               const bf16_t* __restrict__ w,
                                                               bf16_t* __restrict__ dxg, int Tn, int d, int E) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = (blockIdx.x * 4 + wave) * 32;
    if (!ONE_CHUNK && t0 >= Tn) return;   // (E == 64: every wave takes part in the staging and its barrier)
    const int h = lane >> 5, c = lane & 31;
    // columns per wave; d % 64 == 0, so every 32-column block below is complete
    constexpr int COLS = ONE_CHUNK ? kDxCols : kDxColsManyExperts;
    const int ibeg = blockIdx.y * COLS;
    const int iend = ibeg + COLS < d ? ibeg + COLS : d;
    const bool ok_t = t0 + c < Tn;
    const float* arow = dl + (size_t)(ok_t ? t0 + c : 0) * E + 8 * h;
    uint4 ah[4], al[4];
    auto load_a = [&](int e0) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (ok_t) {
                const float4* p = reinterpret_cast<const float4*>(arow + e0 + 16 * ks);
                const float4 f0 = p[0], f1 = p[1];
                v[0] = f0.x; v[1] = f0.y; v[2] = f0.z; v[3] = f0.w;
                v[4] = f1.x; v[5] = f1.y; v[6] = f1.z; v[7] = f1.w;
            }
            split_bf16x8(v, ah[ks], al[ks]);
        }
    };
    auto multiply = [&](int i0, int e0, gate_f32x16_t& acc) {
        const bf16_t* brow = w + (size_t)(i0 + c) * E + 8 * h + e0;
        uint4 b[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) b[ks] = *reinterpret_cast<const uint4*>(brow + 16 * ks);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const gate_bf16x8_t bb = __builtin_bit_cast(gate_bf16x8_t, b[ks]);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bb, __builtin_bit_cast(gate_bf16x8_t, ah[ks]), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bb, __builtin_bit_cast(gate_bf16x8_t, al[ks]), acc, 0, 0, 0);
        }
    };
    // lane (h, c): token t0 + c, columns i0 + 8j + 4h .. +3 in acc[4j .. 4j+3]
    auto store = [&](int i0, const gate_f32x16_t& acc) {
        if (!ok_t) return;
        bf16_t* orow = dxg + (size_t)(t0 + c) * d + i0 + 4 * h;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *reinterpret_cast<uint2*>(orow + 8 * j) =
                make_uint2(pack_bf16x2(acc[4 * j], acc[4 * j + 1]), pack_bf16x2(acc[4 * j + 2], acc[4 * j + 3]));
    };
    if (ONE_CHUNK) {
        // E == 64.  The four waves of a block work on the same columns, so the block stages its kDxCols rows of w in
        // LDS once (rows of 128 bytes padded to kDwStride) and the column blocks take their operands from there:
        // with loads from memory between the stores, every wait for an operand would also wait for the stores
        // issued before it (the counter is in issue order).
        __shared__ __align__(16) char wsm[kDxCols * kDwStride];
        {
            const int r = threadIdx.x >> 3, piece = threadIdx.x & 7;   // 32 rows x 8 pieces of 16 bytes per pass
#pragma unroll
            for (int pass = 0; pass < kDxCols / 32; ++pass) {
                const int row = pass * 32 + r;
                uint4 q = make_uint4(0, 0, 0, 0);
                if (ibeg + row < iend) q = *reinterpret_cast<const uint4*>(w + (size_t)(ibeg + row) * E + piece * 8);
                *reinterpret_cast<uint4*>(wsm + row * kDwStride + piece * 16) = q;
            }
        }
        load_a(0);
        __syncthreads();
        for (int i0 = ibeg; i0 < iend; i0 += 32) {
            gate_f32x16_t acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
            const char* brow = wsm + (i0 - ibeg + c) * kDwStride + 16 * h;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const gate_bf16x8_t bb = *reinterpret_cast<const gate_bf16x8_t*>(brow + 32 * ks);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bb, __builtin_bit_cast(gate_bf16x8_t, ah[ks]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bb, __builtin_bit_cast(gate_bf16x8_t, al[ks]), acc, 0, 0, 0);
            }
            store(i0, acc);
        }
    } else {
        constexpr int NB = COLS / 32;
        gate_f32x16_t acc[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
        for (int e0 = 0; e0 < E; e0 += 64) {
            load_a(e0);
#pragma unroll
            for (int n = 0; n < NB; ++n)
                if (ibeg + 32 * n < iend) multiply(ibeg + 32 * n, e0, acc[n]);
        }
#pragma unroll
        for (int n = 0; n < NB; ++n)
            if (ibeg + 32 * n < iend) store(ibeg + 32 * n, acc[n]);
    }
}

template <typename T>
static int launch_gate_logits(const void* x, const void* w, const float* bias, float* logits, int Tn, int d,
                              int E, hipStream_t s) {
    const long blocks32 = (long)((Tn + 31) / 32) * ((E + 31) / 32);
    // whole 16-byte vectors in an operand: none of its loads needs a branch, and a stage's are in flight together
    const bool vx = d % (16 / (int)sizeof(T)) == 0, vw = E % (16 / (int)sizeof(T)) == 0;
#define XMOE_GATE_V(TL, VX, VW)                                                                                         \
    XMOE_LAUNCH(K_GATE_LOGITS, s,                                                                                       \
                hipLaunchKernelGGL((gate_logits_kernel<T, TL, VX, VW>), dim3((Tn + TL - 1) / TL, (E + TL - 1) / TL),    \
                                   dim3(512), 0, s, (const T*)x, (const T*)w, bias, logits, Tn, d, E))
#define XMOE_GATE(TL)                                  \
    do {                                               \
        if (vx && vw) XMOE_GATE_V(TL, true, true);     \
        else if (vx) XMOE_GATE_V(TL, true, false);     \
        else if (vw) XMOE_GATE_V(TL, false, true);     \
        else XMOE_GATE_V(TL, false, false);            \
    } while (0)
    if (E > 16 && blocks32 >= kGateBigBlocks)
        XMOE_GATE(32);
    else
        XMOE_GATE(16);
#undef XMOE_GATE
#undef XMOE_GATE_V
    return XMOE_OK;
}

template <typename T>
static int launch_gate_bwd(const void* x, const void* w, const float* dl, int Tn, int d, int E, void* dwr,
                           void* dxg, float* partial, hipStream_t s) {
    const int splits = gate_bwd_splits(Tn);
    const int tps = (Tn + splits - 1) / splits;
    dim3 g1((d + 63) / 64, (E + 63) / 64, splits);
    if (sizeof(T) == 2 && d % 64 == 0 && E % 64 == 0 && aligned16(x) && aligned16(w) && aligned16(dl) &&
        aligned16(dxg)) {
        XMOE_LAUNCH(K_GATE_BWD_DW, s,
                    hipLaunchKernelGGL(gate_bwd_dw_mfma_kernel, g1, dim3(256), 0, s, (const bf16_t*)x, dl, partial, Tn,
                                       d, E, tps));
        const size_t n_ = (size_t)d * E;
        XMOE_LAUNCH(K_GATE_BWD_DW_REDUCE, s,
                    hipLaunchKernelGGL(gate_bwd_dw_reduce_kernel<T>, dim3((unsigned)((n_ + 255) / 256)), dim3(256), 0,
                                       s, partial, splits, n_, (T*)dwr));
        if (E == 64) {
            dim3 g2m((Tn + 127) / 128, (d + kDxCols - 1) / kDxCols);
            XMOE_LAUNCH(K_GATE_BWD_DX, s,
                        hipLaunchKernelGGL(gate_bwd_dx_mfma_kernel<true>, g2m, dim3(256), 0, s, dl, (const bf16_t*)w,
                                           (bf16_t*)dxg, Tn, d, E));
        } else {
            dim3 g2m((Tn + 127) / 128, (d + kDxColsManyExperts - 1) / kDxColsManyExperts);
            XMOE_LAUNCH(K_GATE_BWD_DX, s,
                        hipLaunchKernelGGL(gate_bwd_dx_mfma_kernel<false>, g2m, dim3(256), 0, s, dl, (const bf16_t*)w,
                                           (bf16_t*)dxg, Tn, d, E));
        }
        return XMOE_OK;
    }
    // d (E) even: a pair lies in a row of x (dlogits) whole or not at all
    const bool px = d % 2 == 0 && (reinterpret_cast<uintptr_t>(x) & (2 * sizeof(T) - 1)) == 0;
    const bool pe = E % 2 == 0 && (reinterpret_cast<uintptr_t>(dl) & 7u) == 0;
#define XMOE_GATE_DW_M(VX, VE, MODE)                                                                                    \
    XMOE_LAUNCH(K_GATE_BWD_DW, s,                                                                                       \
                hipLaunchKernelGGL((gate_bwd_dw_kernel<T, VX, VE, MODE>), g1, dim3(256), 0, s, (const T*)x, dl,         \
                                   partial, Tn, d, E, tps))
#define XMOE_GATE_DW(VX, VE)                                                           \
    do {                                                                               \
        if (tps < 16) XMOE_GATE_DW_M(VX, VE, DW_TAIL);                                 \
        else if (batch) XMOE_GATE_DW_M(VX, VE, DW_BATCH);                              \
        else XMOE_GATE_DW_M(VX, VE, (sizeof(T) == 2 ? (int)DW_BATCH : (int)DW_FREE));  \
    } while (0)
    const bool batch = sizeof(T) == 2 || (long)g1.x * g1.y * g1.z < 512;
    if (px && pe) XMOE_GATE_DW(true, true);
    else if (px) XMOE_GATE_DW(true, false);
    else if (pe) XMOE_GATE_DW(false, true);
    else XMOE_GATE_DW(false, false);
#undef XMOE_GATE_DW
#undef XMOE_GATE_DW_M
    size_t n = (size_t)d * E;
    XMOE_LAUNCH(K_GATE_BWD_DW_REDUCE, s,
                hipLaunchKernelGGL(gate_bwd_dw_reduce_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                                   s, partial, splits, n, (T*)dwr));
    // columns per wave: fewer where that many would leave CUs without a block.  Fetching the rows of dlogits again costs
    // less than the idle CUs (float32 T 256 d 128 E 8: 14 -> 7 us, T 2048 d 1024 E 16: 26 -> 11, bf16 T 3001 d 1000 E 24:
    // 34 -> 19; part of it from fetching the elements of rows that are no whole vectors without branches)
    int cols = kDxCols;
    while (cols > 32 && (long)((Tn + 127) / 128) * ((d + cols - 1) / cols) < 512) cols /= 2;
    dim3 g2((Tn + 127) / 128, (d + cols - 1) / cols);
    if (E < 64)
        XMOE_LAUNCH(K_GATE_BWD_DX, s,
                    hipLaunchKernelGGL((gate_bwd_dx_kernel<T, true>), g2, dim3(256), 0, s, dl, (const T*)w, (T*)dxg, Tn, d,
                                       E, cols));
    else
        XMOE_LAUNCH(K_GATE_BWD_DX, s,
                    hipLaunchKernelGGL((gate_bwd_dx_kernel<T, false>), g2, dim3(256), 0, s, dl, (const T*)w, (T*)dxg, Tn,
                                       d, E, cols));
    return XMOE_OK;
}

template <int PL>
static int launch_route(const float* logits, int Tn, int E, int k, int32_t* idx, float* w, hipStream_t s) {
    XMOE_LAUNCH(K_ROUTE, s,
                hipLaunchKernelGGL(route_kernel<PL>, dim3((Tn + 3) / 4), dim3(256), 0, s, logits, Tn, E, k, idx, w));
    return XMOE_OK;
}
template <int PL>
static int launch_route_bwd(const float* logits, const int32_t* idx, const float* grad, const int32_t* row_of_slot, int Tn,
                            int E, int k, float* dw, float* dl, hipStream_t s) {
    const dim3 grid((Tn + 3) / 4);
    if (row_of_slot)
        XMOE_LAUNCH(K_ROUTE_BWD, s, hipLaunchKernelGGL((route_bwd_kernel<PL, true>), grid, dim3(256), 0, s, logits, idx,
                                                       grad, row_of_slot, Tn, E, k, dw, dl));
    else
        XMOE_LAUNCH(K_ROUTE_BWD, s, hipLaunchKernelGGL((route_bwd_kernel<PL, false>), grid, dim3(256), 0, s, logits, idx,
                                                       grad, row_of_slot, Tn, E, k, dw, dl));
    return XMOE_OK;
}
static int route_bwd(const float* logits, const int32_t* idx, const float* grad, const int32_t* row_of_slot, int T, int E,
                     int k, float* dw, float* dlogits, hipStream_t s) {
    if (T < 0 || E < 1 || k < 1 || k > E) return XMOE_ERR_INVALID_ARG;
    if (E > XMOE_MAX_EXPERTS || k > 64) return XMOE_ERR_UNSUPPORTED;
    if ((long long)T * k >= (1ll << 31) || (long long)T * E >= (1ll << 31)) return XMOE_ERR_INVALID_ARG;
    if (T == 0) return XMOE_OK;
    if (!logits || !idx || !grad || !dw || !dlogits) return XMOE_ERR_INVALID_ARG;
    if (E <= 64) return launch_route_bwd<1>(logits, idx, grad, row_of_slot, T, E, k, dw, dlogits, s);
    if (E <= 128) return launch_route_bwd<2>(logits, idx, grad, row_of_slot, T, E, k, dw, dlogits, s);
    if (E <= 256) return launch_route_bwd<4>(logits, idx, grad, row_of_slot, T, E, k, dw, dlogits, s);
    return launch_route_bwd<8>(logits, idx, grad, row_of_slot, T, E, k, dw, dlogits, s);
}

}  // namespace xmoe

using namespace xmoe;

extern "C" {

int xmoe_gate_logits(const void* x, const void* w_router, const float* bias, float* logits, int T, int d, int E,
                     int dt, void* stream) {
    if (!dtype_ok(dt)) return XMOE_ERR_UNSUPPORTED;
    if (T < 0 || d < 1 || E < 1) return XMOE_ERR_INVALID_ARG;
    if ((long long)T * E >= (1ll << 31) || (long long)T * d >= (1ll << 40)) return XMOE_ERR_INVALID_ARG;
    if (T == 0) return XMOE_OK;
    if (!x || !w_router || !logits) return XMOE_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    return dt == XMOE_F32 ? launch_gate_logits<float>(x, w_router, bias, logits, T, d, E, s)
                          : launch_gate_logits<bf16_t>(x, w_router, bias, logits, T, d, E, s);
}

int xmoe_route(const float* logits, int T, int E, int k, int32_t* topk_idx, float* topk_w, void* stream) {
    if (T < 0 || E < 1 || k < 1 || k > E) return XMOE_ERR_INVALID_ARG;
    if (E > XMOE_MAX_EXPERTS || k > 64) return XMOE_ERR_UNSUPPORTED;
    if ((long long)T * k >= (1ll << 31) || (long long)T * E >= (1ll << 31)) return XMOE_ERR_INVALID_ARG;
    if (T == 0) return XMOE_OK;
    if (!logits || !topk_idx || !topk_w) return XMOE_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (E <= 64) return launch_route<1>(logits, T, E, k, topk_idx, topk_w, s);
    if (E <= 128) return launch_route<2>(logits, T, E, k, topk_idx, topk_w, s);
    if (E <= 256) return launch_route<4>(logits, T, E, k, topk_idx, topk_w, s);
    return launch_route<8>(logits, T, E, k, topk_idx, topk_w, s);
}

int xmoe_route_bwd(const float* logits, const int32_t* topk_idx, const float* dw, int T, int E, int k,
                   float* dlogits, void* stream) {
    return route_bwd(logits, topk_idx, dw, nullptr, T, E, k, const_cast<float*>(dw), dlogits, (hipStream_t)stream);
}

int xmoe_route_bwd_rows(const float* logits, const int32_t* topk_idx, const float* row_grad, const int32_t* row_of_slot,
                        int T, int E, int k, float* dw, float* dlogits, void* stream) {
    if (T > 0 && !row_of_slot) return XMOE_ERR_INVALID_ARG;
    return route_bwd(logits, topk_idx, row_grad, row_of_slot, T, E, k, dw, dlogits, (hipStream_t)stream);
}

int xmoe_gate_logits_bwd(const void* x, const void* w_router, const float* dlogits, int T, int d, int E, int dt,
                         void* dw_router, void* dx_gate, void* ws, size_t ws_bytes, void* stream) {
    if (!dtype_ok(dt)) return XMOE_ERR_UNSUPPORTED;
    if (T < 0 || d < 1 || E < 1) return XMOE_ERR_INVALID_ARG;
    if ((long long)T * E >= (1ll << 31)) return XMOE_ERR_INVALID_ARG;
    if (!dw_router) return XMOE_ERR_INVALID_ARG;
    if (T == 0) {   // a sum over no tokens: dw_router = 0, dx_gate has no rows
        const size_t n = (size_t)d * E;
        const dim3 grid((unsigned)((n + 255) / 256));
        if (dt == XMOE_F32)
            XMOE_LAUNCH(K_GATE_BWD_DW_REDUCE, (hipStream_t)stream,
                        hipLaunchKernelGGL(gate_bwd_dw_reduce_kernel<float>, grid, dim3(256), 0, (hipStream_t)stream,
                                           (const float*)nullptr, 0, n, (float*)dw_router));
        else
            XMOE_LAUNCH(K_GATE_BWD_DW_REDUCE, (hipStream_t)stream,
                        hipLaunchKernelGGL(gate_bwd_dw_reduce_kernel<bf16_t>, grid, dim3(256), 0, (hipStream_t)stream,
                                           (const float*)nullptr, 0, n, (bf16_t*)dw_router));
        return XMOE_OK;
    }
    if (!x || !w_router || !dlogits || !dx_gate) return XMOE_ERR_INVALID_ARG;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) || ws_bytes < gate_bwd_ws_bytes(T, d, E))
        return XMOE_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    return dt == XMOE_F32
               ? launch_gate_bwd<float>(x, w_router, dlogits, T, d, E, dw_router, dx_gate, (float*)ws, s)
               : launch_gate_bwd<bf16_t>(x, w_router, dlogits, T, d, E, dw_router, dx_gate, (float*)ws, s);
}

}  // extern "C"
