// kan_bwd_dx.hip -- input gradient of the KAN layer on the matrix cores
// (eq. kan_forward differentiated):
//
//   dx[b, i] = sum_o dy[b, o] ( sum_j C[o, i, j] N_j'(x[b, i]) + Wb[o, i] silu'(x[b, i]) )
//
// Gm = dy W^T over the outputs (Gm[b, (i, c)] for every column c of every
// feature), then per (row, feature) the dot product of its columns with
// (silu'(x), N_0'(x), ...).  The MFMA puts the K rows (feature, column) in the
// A operand (packed weights, staged in LDS and shared by the workgroup's eight
// waves) and the batch rows in the B operand (dy of RF 32-row tiles per wave, held
// in registers for the whole kernel); the A rows are permuted so that each
// lane's 16 accumulators are 16 consecutive columns of one feature for one batch
// row, and the derivative contraction runs in the lane.
//
// bf16: one bf16 operand each, two row tiles per wave, so that every A fragment
// read from LDS feeds two MFMAs (with one, the reads alone fill the LDS's
// bandwidth at the matrix cores' rate).  784 -> 256 at 65536 rows: 496 -> 377 us
// (two row tiles and columns selected in registers 420, A fragments read four
// groups ahead 377).
// fp32: both operands as two fp16 terms (kan_bwd_dw.hip) and three products:
// 96 cycles per 16 outputs of a 32 x 32 tile where the fp32 instruction takes
// 512.  dy is scaled per batch row and the weights per K tile and chunk of outputs
// (coefficients and SiLU weights each by their own) by the power of two that brings the
// largest to 2^14.  784 -> 256 at 16384 rows: 805 -> 277-300 us, relative error (2-norm)
// against float64 5e-7 -> 1.6e-7 (the window at its own coordinate; fewer roundings).
// The terms hold 22 bits of the largest weight of every window; a K tile with weights
// that they cannot hold so (kan_bwd_pack.h) is held in fp32 and taken after the others
// on the fp32 instruction, and rows with a non-finite dy are then computed apart.
#include "kan_bwd_pack.h"

#include <algorithm>

namespace kan {

namespace {

constexpr int kNW = 8;
constexpr int kThreads = 64 * kNW;

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));  // 16 bytes at an element's alignment
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));

__device__ __forceinline__ float silu_slope(float x) {
    const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-x));
    return s * __builtin_fmaf(x, 1.0f - s, 1.0f);
}

// ------------------------------------------------------------------- packing

template <typename T>
__global__ __launch_bounds__(256) void pack_dx2_kernel(Dx2Args a) {
    pack_dx2<T>(a, blockIdx.x, blockIdx.y);
}

// -------------------------------------------------------------------- kernel

// The derivative's segment form on the four window columns (kan_backward.hip): tau
// in [0, 1), clo = floor(s) - 1 the first of them.
__device__ __forceinline__ void window_slopes(float tau, float (&d)[4]) {
    const float t2 = tau * tau;
    d[0] = -0.5f * (1.0f - tau) * (1.0f - tau);
    d[1] = __builtin_fmaf(1.5f, t2, -2.0f * tau);
    d[2] = __builtin_fmaf(-1.5f, t2, __builtin_fmaf(tau, 1.0f, 0.5f));
    d[3] = 0.5f * t2;
}

// N'(u) at v = u - 2: sign(v) (2 b^2 - w^2 / 2) with a = min(|v|, 2), w = 2 - a and
// b = max(1 - a, 0) (exactly 0 off the support; a NaN gives 0, the SiLU slope
// carries it).
__device__ __forceinline__ float slope_at(float v) {
    const float a = __builtin_fminf(__builtin_fabsf(v), 2.0f);
    const float w = 2.0f - a;
    const float b = __builtin_amdgcn_fmed3f(1.0f - a, 0.0f, 1.0f);
    return __builtin_copysignf(__builtin_fmaf(2.0f * b, b, -0.5f * w * w), -v);
}

// fp32: dx of the features with a tile held in fp32, on the fp32 instruction (their
// other tiles' weights from the two terms), for the wave's row tile rf.  dy comes from
// memory again, in fp32, and the weights straight from the workspace, both a group of
// outputs ahead.  A function of its own, so that the main loop keeps its registers;
// args: the kernel's, in place.  16384 x 784 -> 256 with every tile so: 1.29 ms a call,
// 0.29 ms with none (0.8 ms where the fp32 instruction was the kernel's own), 0.30 ms
// with one.
template <int RF, bool C16>
__device__ __attribute__((noinline)) void wide_tiles(const uint32_t* args, int rf) {
    constexpr int NT = 2;
    struct Words { uint32_t w[sizeof(Dx2Args) / 4]; } words;
    static_assert(sizeof(Words) == sizeof(Dx2Args), "whole words");
#pragma unroll
    for (size_t i = 0; i < sizeof(Dx2Args) / 4; ++i)
        words.w[i] = __builtin_amdgcn_readfirstlane(args[i]);
    const Dx2Args a = __builtin_bit_cast(Dx2Args, words);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int64_t wrow = (int64_t)blockIdx.x * (kNW * 32 * RF) + wave * (32 * RF) +
                         32 * __builtin_amdgcn_readfirstlane(rf);
    if (wrow >= a.batch) return;
    const int64_t row = wrow + r, rowc = min(row, a.batch - 1);
    const int ch = blockIdx.y, g0 = ch * a.gmax, S = min(a.gmax, a.groups - g0);
    const int t_begin = blockIdx.z * a.tiles_per_split;
    const int t_end = min(t_begin + a.tiles_per_split, a.ntiles);
    const int tpf = C16 ? 1 : a.cp / 32;
    const uint64_t bytes = (uint64_t)(a.batch - wrow) * a.out * 4;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(static_cast<const float*>(a.dy) + wrow * a.out), (short)0,
        (int)(bytes < 0xffffffffull ? bytes : 0xffffffffull), kBufferWord3);
    // dy of the lane half's eight outputs of group s (loads past the tensor give 0)
    auto load_dy = [&](int s, u32x4 (&d)[2]) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
            d[m] = __builtin_bit_cast(
                u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                           rs, ((uint32_t)r * (uint32_t)a.out +
                                (uint32_t)((g0 + s) * 16 + 8 * h + 4 * m)) * 4u, 0, 0));
    };
#pragma unroll 1
    for (int next = t_begin; next < t_end;) {
        // the first feature with such a tile, 64 tiles at a look
        const int tl = next + lane;
        const uint64_t wide = __ballot(tl < t_end && (a.wexp[min(tl, t_end - 1) * a.nchunk + ch] & kPackWide) != 0);
        if (wide == 0) {
            next += 64;
            continue;
        }
        const int t0 = (next + __ffsll((unsigned long long)wide) - 1) / tpf * tpf;
        next = t0 + tpf;
        const int f = C16 ? 2 * t0 + h : t0 / tpf;
        const float x = f < a.in ? static_cast<const float*>(a.xt)[(int64_t)f * a.bpad + rowc] : 0.0f;
        const float lo = coord_lo(x, a.xlim, a.inv_lo, a.a_frac);
        float sum = 0.0f;
#pragma unroll 1
        for (int t = t0; t < t0 + tpf; ++t) {
            const int we = __builtin_amdgcn_readfirstlane(a.wexp[t * a.nchunk + ch]);
            // (a feature of several tiles: its SiLU column is the first A row of its first)
            const int wx = (r == 0 && t == t0 ? pack_es(we) : pack_ex(we)) - kPackExp;
            const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc(
                a.wtp + ((int64_t)t * a.groups + g0) * (NT * 64), (short)0, S * NT * 1024,
                kBufferWord3);
            auto load_wt = [&](int s, int term) {
                return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                     ws, lane * 16, (s * NT + term) * 1024, 0));
            };
            u32x4 n0 = load_wt(0, 0), n1 = load_wt(0, 1), dn[2];
            load_dy(0, dn);
            floatx16 acc;
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
#pragma unroll 1
            for (int s = 0; s < S; ++s) {
                const u32x4 q0 = n0, q1 = n1;
                u32x4 d[2] = {dn[0], dn[1]};
                const int sn = min(s + 1, S - 1);
                n0 = load_wt(sn, 0);
                n1 = load_wt(sn, 1);
                load_dy(sn, dn);
                float w[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = __uint_as_float(e < 4 ? q0[e % 4] : q1[e % 4]);
                if ((we & kPackWide) == 0) {
                    const f16x8_t h0 = __builtin_bit_cast(f16x8_t, q0);
                    const f16x8_t h1 = __builtin_bit_cast(f16x8_t, q1);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        w[e] = __builtin_ldexpf((float)h0[e] + (float)h1[e], wx);
                }
                if ((g0 + s) * 16 + 16 > a.out) {  // (past the row: the next row's)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if ((g0 + s) * 16 + 8 * h + e >= a.out) d[e / 4][e % 4] = 0u;
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(
                        w[e], __uint_as_float(d[e / 4][e % 4]), acc, 0, 0, 0);
            }
            const int c0 = C16 ? 0 : 32 * (t - t0) + 16 * h;
            float sb = 0.0f;
#pragma unroll
            for (int q = 0; q < 16; ++q) {  // (a sum counts in its window alone)
                const float v = __builtin_fmaf(x, a.inv_h, a.a_int + 1.0f - (float)(c0 + q)) + lo;
                if (c0 + q > 0 && v >= -2.0f && v < 2.0f)
                    sb = __builtin_fmaf(acc[q], slope_at(v), sb);
            }
            sum += __builtin_fmaf(c0 == 0 ? acc[0] : 0.0f, silu_slope(x), a.inv_h * sb);
        }
        if (!C16) sum += __shfl_xor(sum, 32);  // (both lane halves' columns)
        if (row < a.batch && f < a.in && (C16 || h == 0)) {
            if (a.dxp != nullptr) a.dxp[((int64_t)ch * a.batch + row) * a.in + f] = sum;
            else static_cast<float*>(a.dx)[row * a.in + f] = sum;
        }
    }
}

// SM bounds the 16-output groups of a chunk; RF row tiles per wave; TPB K tiles per
// stage (a barrier each; the epilogue of one tile overlaps the other wave's
// MFMAs of the next); C16: features of 16 K rows, whose window columns are
// selected in registers (through the LDS, as for wider features, they cost as
// much LDS time as the A fragments, and that bounds the kernel: bf16 784 -> 256
// at 65536 rows 432 us).
template <typename T, int SM, int RF, int TPB, bool C16>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void dx2_kernel(Dx2Args a) {
    constexpr bool BF = sizeof(T) == 2;
    constexpr int NT = BF ? 1 : 2;
    constexpr int TU = SM * NT * 64;  // 16-byte units of a K tile in LDS
    __shared__ u32x4 lds[2][TPB * TU];
    // per wave: a lane's 16 accumulators after 4 zero floats (stride 80 bytes: the
    // 16-byte writes of 16 lanes fall in distinct banks; the next lane's zeros, and
    // 4 after the last lane, follow them), read back at the window's columns
    __shared__ u32x4 gat[C16 ? 1 : kNW][64 * 5 + 1];
    __shared__ int rowbad[BF ? 1 : kNW * 32 * RF];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, r = lane & 31, h = lane >> 5;
    constexpr int BM = kNW * 32 * RF;
    const int64_t wg_row0 = (int64_t)blockIdx.x * BM;
    const int64_t row0 = wg_row0 + wave * (32 * RF) + r;
    const int ch = blockIdx.y;
    const int g0 = ch * a.gmax;
    const int S = min(a.gmax, a.groups - g0);
    const int t_begin = blockIdx.z * a.tiles_per_split;
    const int t_end = min(t_begin + a.tiles_per_split, a.ntiles);
    const int nst = (t_end - t_begin + TPB - 1) / TPB;
    int64_t rowc[RF];
#pragma unroll
    for (int rf = 0; rf < RF; ++rf) rowc[rf] = min(row0 + 32 * rf, a.batch - 1);

    // weights: this chunk's groups of the stage's K tiles (tiles past the split's
    // last re-read it; their results are not stored)
    const uint32_t lds0 =
        (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)&lds[0][0]);
    auto load_w = [&](int st, int buf) {
#pragma unroll
        for (int k = 0; k < TPB; ++k) {
            const int t = min(t_begin + st * TPB + k, t_end - 1);
            const uint64_t base = reinterpret_cast<uint64_t>(
                reinterpret_cast<const char*>(a.wtp) + ((int64_t)t * a.groups + g0) * (NT * 1024));
            u32x4 wrs;
            wrs[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
            wrs[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
            wrs[2] = (uint32_t)(S * NT * 1024);
            wrs[3] = (uint32_t)kBufferWord3;
            const uint32_t dst = lds0 + (uint32_t)((buf * TPB + k) * TU) * 16u;
#pragma unroll
            for (int i = 0; i < (SM * NT + kNW - 1) / kNW; ++i) {
                const int wl = wave + kNW * i;
                if (wl < S * NT)
                    dma16(wrs, (uint32_t)lane * 16u, (uint32_t)wl * 1024u,
                          dst + (uint32_t)wl * 1024u);
            }
        }
    };

    constexpr bool cp16 = C16;
    const int tpf = cp16 ? 1 : a.cp / 32;  // tiles per feature (cp >= 32)
    auto feat0 = [&](int t) -> int { return cp16 ? 2 * t : t / tpf; };
    const T* xt = static_cast<const T*>(a.xt);
    auto load_x = [&](int st, T (&xs)[TPB][RF]) {
#pragma unroll
        for (int k = 0; k < TPB; ++k) {
            const int t = min(t_begin + st * TPB + k, t_end - 1);
            const T* xb = xt + (int64_t)feat0(t) * a.bpad + (cp16 && h ? a.bpad : 0);
#pragma unroll
            for (int rf = 0; rf < RF; ++rf) xs[k][rf] = xb[rowc[rf]];
        }
    };

    // ---- prologue: the first stage's loads, then dy
    T xq[TPB][RF];
    load_x(0, xq);
    load_w(0, 0);
    // LDS rows of groups past the chunk's are zero (never written again)
    for (int u = S * NT * 64 + tid; u < TU; u += kThreads)
#pragma unroll
        for (int k = 0; k < TPB; ++k) {
            lds[0][k * TU + u] = u32x4{0u, 0u, 0u, 0u};
            lds[1][k * TU + u] = u32x4{0u, 0u, 0u, 0u};
        }
    if constexpr (!C16) {
        char* gw0 = reinterpret_cast<char*>(gat[wave]);
        *reinterpret_cast<u32x4*>(gw0 + lane * 80) = u32x4{0u, 0u, 0u, 0u};
        if (lane == 63) *reinterpret_cast<u32x4*>(gw0 + 64 * 80) = u32x4{0u, 0u, 0u, 0u};
    }
    // B operands: the lane's batch rows of dy for every group of the chunk.  All loads
    // are 8 elements wide, at any alignment of the row, and go out before the first
    // use; what they read past the row's outputs is masked, and only a load that
    // would pass the tensor's end is taken element by element.
    u32x4 dyr[RF][NT][SM];
    int esc[RF];
    const int64_t total = a.batch * (int64_t)a.out;
    constexpr int NV = 8 * (int)sizeof(T) / 16;  // 16-byte units of eight elements
    typedef typename std::conditional<BF, u32x4_a2, u32x4_a4>::type u32x4_el;
    u32x4 raw[RF][SM][NV];
#pragma unroll
    for (int rf = 0; rf < RF; ++rf) {
        const int64_t at = rowc[rf] * a.out + g0 * 16 + 8 * h;
#pragma unroll
        for (int s = 0; s < SM; ++s) {
            if (total < 8) continue;
            const T* p = static_cast<const T*>(a.dy) + min(at + 16 * min(s, S - 1), total - 8);
#pragma unroll
            for (int k = 0; k < NV; ++k)
                raw[rf][s][k] = reinterpret_cast<const u32x4_el*>(p)[k];
        }
    }
#pragma unroll
    for (int rf = 0; rf < RF; ++rf) {
        const int64_t at = rowc[rf] * a.out + g0 * 16 + 8 * h;
        T v[SM][8];
#pragma unroll
        for (int s = 0; s < SM; ++s) {
            const int o0 = (g0 + s) * 16 + 8 * h;
            if ((g0 + s) * 16 + 16 > a.out) {  // (uniform) the last group, or one past it
                const bool past = at + 16 * s + 8 > total;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    T t = T(0);
                    if (s < S && o0 + e < a.out) {
                        if (past) t = static_cast<const T*>(a.dy)[at + 16 * s + e];
                        else if constexpr (BF) t = (uint16_t)(raw[rf][s][0][e / 2] >> (16 * (e & 1)));
                        else t = __uint_as_float(raw[rf][s][e / 4 < NV ? e / 4 : 0][e % 4]);
                    }
                    v[s][e] = t;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if constexpr (BF) v[s][e] = (uint16_t)(raw[rf][s][0][e / 2] >> (16 * (e & 1)));
                    else v[s][e] = __uint_as_float(raw[rf][s][e / 4 < NV ? e / 4 : 0][e % 4]);
                }
            }
        }
        esc[rf] = 0;
        if constexpr (BF) {
#pragma unroll
            for (int s = 0; s < SM; ++s)
                dyr[rf][0][s] = u32x4{(uint32_t)v[s][0] | (uint32_t)v[s][1] << 16,
                                      (uint32_t)v[s][2] | (uint32_t)v[s][3] << 16,
                                      (uint32_t)v[s][4] | (uint32_t)v[s][5] << 16,
                                      (uint32_t)v[s][6] | (uint32_t)v[s][7] << 16};
        } else {
            float m = 0.0f;
            bool bad = false;
#pragma unroll
            for (int s = 0; s < SM; ++s)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float av = __builtin_fabsf(v[s][e]);
                    const bool fin = av < __builtin_inff();
                    bad |= !fin;
                    m = __builtin_fmaxf(m, fin ? av : 0.0f);
                }
            m = __builtin_fmaxf(m, __shfl_xor(m, 32));
            bad |= __shfl_xor((int)bad, 32) != 0;
            if (h == 0) rowbad[wave * 32 * RF + 32 * rf + r] = bad;
            const int ex = (int)(__float_as_uint(m) >> 23) - 127;
            esc[rf] = ex - kPackExp;
#pragma unroll
            for (int s = 0; s < SM; ++s) {
                f16x8_t t0, t1;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = __builtin_amdgcn_fmed3f(__builtin_ldexpf(v[s][e], kPackExp - ex),
                                                            -60000.0f, 60000.0f);
                    t0[e] = (_Float16)x;
                    t1[e] = (_Float16)(x - (float)t0[e]);
                }
                dyr[rf][0][s] = __builtin_bit_cast(u32x4, t0);
                dyr[rf][NT - 1][s] = __builtin_bit_cast(u32x4, t1);
            }
        }
    }

    // Results of a stage, stored at the start of the next one: the wait for the
    // weights at a stage's end then finds the stores long done.
    float dxacc[RF], val[TPB][RF];
#pragma unroll
    for (int rf = 0; rf < RF; ++rf) dxacc[rf] = 0.0f;
    const int64_t chrow = a.dxp != nullptr ? (int64_t)ch * a.batch : 0;
    auto put = [&](int rf, int f, float v) {
        const int64_t row = row0 + 32 * rf;
        if (row >= a.batch || f >= a.in) return;
        if (a.dxp != nullptr) {
            a.dxp[(chrow + row) * a.in + f] = v;
        } else if constexpr (BF) {
            static_cast<uint16_t*>(a.dx)[row * a.in + f] = f32_to_bf16(v);
        } else {
            static_cast<float*>(a.dx)[row * a.in + f] = v;
        }
    };
    // bf16, two tiles of two features each: the lane halves exchange so that each
    // lane stores two consecutive features (4 bytes) instead of two single ones
    const bool pairs = BF && TPB == 2 && cp16 && a.dxp == nullptr && a.in % 2 == 0 &&
                       reinterpret_cast<uintptr_t>(a.dx) % 4 == 0;
    auto store_stage = [&](int st) {
        if (pairs) {
            if constexpr (TPB == 2) {
#pragma unroll
                for (int rf = 0; rf < RF; ++rf) {
                    // half 0: features 2 t, 2 t + 1; half 1: 2 t + 2, 2 t + 3
                    const float other = __shfl_xor(h == 0 ? val[1][rf] : val[0][rf], 32);
                    const float v0 = h == 0 ? val[0][rf] : other, v1 = h == 0 ? other : val[1][rf];
                    const int t = t_begin + 2 * st + h;
                    const int64_t row = row0 + 32 * rf;
                    if (row < a.batch && t < t_end && 2 * t < a.in)
                        *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.dx) + row * a.in +
                                                     2 * t) =
                            __builtin_bit_cast(uint32_t, bf16x2_t{(__bf16)v0, (__bf16)v1});
                }
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < TPB; ++k) {
            const int t = t_begin + st * TPB + k;
            if (t >= t_end) break;
            if (cp16) {
#pragma unroll
                for (int rf = 0; rf < RF; ++rf) put(rf, 2 * t + h, val[k][rf]);
            } else if ((t + 1) % tpf == 0 && h == 0) {
#pragma unroll
                for (int rf = 0; rf < RF; ++rf) put(rf, t / tpf, val[k][rf]);
            }
        }
    };

    char* gl = reinterpret_cast<char*>(gat[C16 ? 0 : wave]) + lane * 80;
    auto fence = [&]() {
        __builtin_amdgcn_s_waitcnt((0x7 << 4));  // vmcnt(0) lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    fence();
#pragma unroll 1
    for (int st = 0; st < nst; ++st) {
        const int buf = st & 1;
        if (st > 0) store_stage(st - 1);
        T xn[TPB][RF];
        load_x(st + 1, xn);
        load_w(st + 1, buf ^ 1);
#pragma unroll
        for (int k = 0; k < TPB; ++k) {
            const int t = t_begin + st * TPB + k;
            // (fp32, one row tile: the products with a second term in a chain of their own)
            constexpr bool ACC2 = !BF && RF == 1;
            floatx16 acc[RF], acc2;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
#pragma unroll
                for (int rf = 0; rf < RF; ++rf) acc[rf][q] = 0.0f;
                acc2[q] = 0.0f;
            }
            const u32x4* tl = lds[buf] + k * TU;
#pragma unroll
            for (int s = 0; s < SM; ++s) {
                u32x4 w[NT];
#pragma unroll
                for (int n = 0; n < NT; ++n) w[n] = tl[(s * NT + n) * 64 + lane];
#pragma unroll
                for (int rf = 0; rf < RF; ++rf) {
                    if constexpr (BF) {
                        acc[rf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, w[0]), __builtin_bit_cast(bf16x8, dyr[rf][0][s]),
                            acc[rf], 0, 0, 0);
                    } else {
                        auto mul = [&](int n, int m, floatx16& c) __attribute__((always_inline)) {
                            c = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                __builtin_bit_cast(f16x8_t, w[n]),
                                __builtin_bit_cast(f16x8_t, dyr[rf][m][s]), c, 0, 0, 0);
                        };
                        floatx16& small = ACC2 ? acc2 : acc[rf];
                        // (the least product too where it is nearly free)
                        if constexpr (SM <= 4) mul(NT - 1, NT - 1, small);
                        mul(NT - 1, 0, small);
                        mul(0, 0, acc[rf]);
                        mul(0, NT - 1, small);
                    }
                }
            }
            {
                // A fragments read PRE groups ahead of their MFMAs (left to itself the
                // compiler reads each just before its use, and every pair of MFMAs
                // waits on the LDS)
                constexpr int PRE = SM < 4 ? SM : 4;
                constexpr int NP = RF * (BF ? 1 : SM <= 4 ? 4 : 3);
                __builtin_amdgcn_sched_group_barrier(0x100, PRE * NT, 0);
#pragma unroll
                for (int s = 0; s < SM - PRE; ++s) {
                    __builtin_amdgcn_sched_group_barrier(0x008, NP, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, PRE * NP, 0);
            }
            if constexpr (ACC2) {
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[0][q] += acc2[q];
            }
            // epilogue: dx of the lane's feature from its 16 columns
            const int fu = feat0(t);
            const int f = cp16 ? fu + h : fu;
            const int c0 = cp16 ? 0 : 32 * t - fu * a.cp + 16 * h;
            int we = 0;
            if constexpr (!BF) we = a.wexp[min(t, a.ntiles - 1) * a.nchunk + ch];
#pragma unroll
            for (int rf = 0; rf < RF; ++rf) {
                float xv;
                if constexpr (BF) xv = bf16_to_f32(xq[k][rf]);
                else xv = xq[k][rf];
                xv = f < a.in ? xv : 0.0f;
                const float lo = coord_lo(xv, a.xlim, a.inv_lo, a.a_frac);
                float sb = 0.0f;
                if constexpr (C16) {
                    // window columns w0 .. w0 + 3, clamped into 1 .. 15 (a column taken
                    // in by the clamp is at |v| >= 2, where N' is exactly 0); one of
                    // them per residue g (mod 4), column 4 ((w0 + 3 - g) / 4) + g
                    const float sv = __builtin_fmaf(xv, a.inv_h, a.a_int + 1.0f) + lo;
                    const float wf = __builtin_amdgcn_fmed3f(__builtin_floorf(sv), 2.0f, 13.0f) - 1.0f;
                    const int w0 = (int)wf;
                    const float d = __builtin_fmaf(xv, a.inv_h, a.a_int + 1.0f - wf) + lo;
                    // byte g: (g - w0) mod 4
                    const uint32_t kg = __builtin_amdgcn_alignbit(0x03020100u, 0x03020100u,
                                                                  (uint32_t)(32 - 8 * (w0 & 3)));
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const bool hi = w0 >= 5 + g;
                        const float u0 = hi ? acc[rf][8 + g] : acc[rf][g];
                        const float u1 = hi ? acc[rf][12 + g] : acc[rf][4 + g];
                        const float col = ((w0 + 3 - g) & 4) != 0 ? u1 : u0;
                        sb = __builtin_fmaf(col, slope_at(d - (float)((kg >> (8 * g)) & 0xffu)), sb);
                    }
                } else {
                    // the lane's 16 columns through its LDS slot, read back at the four
                    // window columns (columns outside the lane's 16 read the zeros
                    // around them, columns past nb have zero weights, and the SiLU
                    // column reads as 0 too)
                    const float sc = __builtin_amdgcn_fmed3f(
                        __builtin_fmaf(xv, a.inv_h, a.a_int + 1.0f - (float)c0) + lo, -8.0f, 24.0f);
                    const float fl = __builtin_floorf(sc);
                    float d[4];
                    window_slopes(sc - fl, d);
#pragma unroll
                    for (int m = 0; m < 4; ++m)
                        *reinterpret_cast<floatx4*>(gl + 16 + 16 * m) =
                            floatx4{m == 0 && c0 == 0 ? 0.0f : acc[rf][4 * m],
                                    acc[rf][4 * m + 1], acc[rf][4 * m + 2], acc[rf][4 * m + 3]};
                    const int qlo = min(max((int)fl - 1, -4), 16);
                    const float* gw = reinterpret_cast<const float*>(gl + 16 + 4 * qlo);
#pragma unroll
                    for (int q = 0; q < 4; ++q) sb = __builtin_fmaf(gw[q], d[q], sb);
                }
                const float s0 = c0 == 0 ? acc[rf][0] : 0.0f;
                float v;
                if constexpr (BF)
                    v = __builtin_fmaf(s0, silu_slope(xv), a.inv_h * sb);
                else
                    v = __builtin_ldexpf(s0 * silu_slope(xv), pack_es(we) - kPackExp + esc[rf]) +
                        __builtin_ldexpf(a.inv_h * sb, pack_ex(we) - kPackExp + esc[rf]);
                if (!cp16) {
                    // features of several tiles: the running sum, complete (both
                    // lane halves added) at the feature's last tile
                    v += dxacc[rf];
                    const bool last = (t + 1) % tpf == 0;
                    dxacc[rf] = last ? 0.0f : v;
                    if (last) v += __shfl_xor(v, 32);
                }
                val[k][rf] = v;
            }
        }
#pragma unroll
        for (int k = 0; k < TPB; ++k)
#pragma unroll
            for (int rf = 0; rf < RF; ++rf) xq[k][rf] = xn[k][rf];
        fence();
    }
    if (nst > 0) store_stage(nst - 1);

    if constexpr (!BF) {
        int any = 0;
        for (int i = tid; i < BM; i += kThreads) any |= rowbad[i];
        for (int t = t_begin + tid; t < t_end; t += kThreads) any |= a.wexp[t * a.nchunk + ch] & kPackWide;
        if (__syncthreads_or(any)) {
#pragma unroll 1
            for (int rf = 0; rf < RF; ++rf)
                wide_tiles<RF, C16>((const uint32_t*)__builtin_amdgcn_kernarg_segment_ptr(), rf);
            // Rows with a non-finite dy: the same sums in plain fp32, with the zeros and
            // infinities the matrix instruction would meet.
            int rows = 0;
            for (int i = tid; i < BM; i += kThreads) rows |= rowbad[i];
            if (!__syncthreads_or(rows)) return;
            const int f_beg = cp16 ? 2 * t_begin : t_begin / tpf;
            const int f_end = min(a.in, cp16 ? 2 * t_end : t_end / tpf);
            const int nf = f_end - f_beg;
            const int o_beg = 16 * g0, o_end = min(a.out, 16 * (g0 + S));
            const float* dy = static_cast<const float*>(a.dy);
            for (int64_t u = tid; u < (int64_t)BM * nf; u += kThreads) {
                const int rl = (int)(u / nf), f = f_beg + (int)(u % nf);
                const int64_t row = wg_row0 + rl;
                if (row >= a.batch || rowbad[rl] == 0) continue;
                const float x = xt[(int64_t)f * a.bpad + row];
                const float sc = __builtin_amdgcn_fmed3f(
                    __builtin_fmaf(x, a.inv_h, a.a_int + 1.0f) +
                        coord_lo(x, a.xlim, a.inv_lo, a.a_frac),
                    -8.0f, (float)(a.cp + 8));
                const float fl = __builtin_floorf(sc);
                float d[4];
                window_slopes(sc - fl, d);
                float sb = 0.0f, s0 = 0.0f;
                for (int q = -1; q < 4; ++q) {
                    const int c = q < 0 ? 0 : (int)fl - 1 + q;
                    if (q >= 0 && (c < 1 || c >= a.cp)) continue;
                    float g = 0.0f;
                    for (int o = o_beg; o < o_end && g == g; ++o)
                        g = __builtin_fmaf(dy[row * a.out + o], weight<float>(a, o, f, c), g);
                    if (q < 0) s0 = g;
                    else sb = __builtin_fmaf(g, d[q], sb);
                }
                const float v = __builtin_fmaf(s0, silu_slope(x), a.inv_h * sb);
                if (a.dxp != nullptr) a.dxp[(chrow + row) * a.in + f] = v;
                else static_cast<float*>(a.dx)[row * a.in + f] = v;
            }
        }
    }
}

template <typename T, int SM, int RF>
hipError_t launch_sm(const BwdGeom& g, const Dx2Args& a, hipStream_t s) {
    constexpr int BM = kNW * 32 * RF;
    // (two K tiles per stage where the LDS holds them)
    constexpr int TPB = sizeof(T) == 2 || SM <= 8 ? 2 : 1;
    const dim3 grid((unsigned)((a.batch + BM - 1) / BM), (unsigned)g.nchunk,
                    (unsigned)g.dx_ksplit);
    if (a.cp == 16)
        hipLaunchKernelGGL((dx2_kernel<T, SM, RF, 2, true>), grid, dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((dx2_kernel<T, SM, RF, TPB, false>), grid, dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_t(const BwdGeom& g, const Dx2Args& a, bool packed, hipStream_t s) {
    if (!packed) {
        hipLaunchKernelGGL(pack_dx2_kernel<T>, dim3((unsigned)a.ntiles, (unsigned)a.nchunk),
                           dim3(256), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int sm = std::min(g.groups, g.gmax);  // groups of the largest chunk
    if (sm <= 1) return launch_sm<T, 1, 2>(g, a, s);
    if (sm <= 2) return launch_sm<T, 2, 2>(g, a, s);
    if (sm <= 4) return launch_sm<T, 4, 2>(g, a, s);
    constexpr int RF = sizeof(T) == 2 ? 2 : 1;
    if (sm <= 8) return launch_sm<T, 8, RF>(g, a, s);
    if (sm <= 16) return launch_sm<T, 16, RF>(g, a, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_dx_split(bool bf16, const BwdGeom& g, const Dx2Args& a, bool packed,
                           hipStream_t s) {
    return bf16 ? launch_t<uint16_t>(g, a, packed, s) : launch_t<float>(g, a, packed, s);
}

}  // namespace kan
