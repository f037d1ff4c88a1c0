// kan_bwd_pack.h -- the weights of the backward's dx contraction in the order its
// matrix-core kernel reads them (kan_bwd_dx.hip), by 256-thread workgroups: in a
// kernel of its own or, for small layers, in one launch with the transpositions
// (kan_backward.hip).
#pragma once

#include "kan_internal.h"

namespace kan {

// Weight of column c (0: SiLU) of feature f for output o; 0 outside the layer.
template <typename T>
__device__ __forceinline__ T weight(const Dx2Args& a, int o, int f, int c) {
    if (o >= a.out || f >= a.in || c > a.nb) return T(0);
    const int64_t row = (int64_t)o * a.in + f;
    return c == 0 ? static_cast<const T*>(a.bw)[row]
                  : static_cast<const T*>(a.coef)[row * a.nb + c - 1];
}

// fp32: a window (four consecutive coefficients of a feature for an output: what one
// input's derivative meets) whose largest is 2^kPackWindowBits below the tile's
// scale loses more than the last two bits of its fp32 values.
constexpr int kPackWindowBits = 17;
// SiLU weights have a scale of their own.  One that is that far below it: what the terms
// lose of the other outputs' gradients, where it alone meets the largest, is then past
// 2^-17 of the sum (past the grid there is nothing else).  (A window's bits would be met
// by chance in many tiles: its largest of four is not.)
constexpr int kPackSiluBits = 22;
constexpr int kPackExp = 14;  // the largest of a scale's weights, and dy of a row: [2^14, 2^15)
// The word of a tile: the exponents of the coefficients' and the SiLU weights' scales,
// or that the tile's weights are held in fp32.
constexpr int kPackWide = 1 << 24;
__device__ __forceinline__ int pack_word(int ex, int es) { return (ex + 512) | (es + 512) << 12; }
__device__ __forceinline__ int pack_ex(int w) { return (w & 0xfff) - 512; }
__device__ __forceinline__ int pack_es(int w) { return (w >> 12 & 0xfff) - 512; }

// The next lane's value (the wave's last lane: its own).
__device__ __forceinline__ float next_lane(float v) {
    const int u = (int)__float_as_uint(v);
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(u, u, 0x130, 0xf, 0xf, false));
}

// One workgroup packs K tile t for output chunk ch (groups g0 .. g0 + S - 1 of 16
// outputs): [t][g][term][lane (r, h)][e], outputs 16 g + 8 h + e of the K row of A
// row r.  fp32: two fp16 terms of the weights, scaled per (tile, chunk), coefficients and
// SiLU weights each by their own, and wexp[t nchunk + ch] = pack_word, or kPackWide: the
// tile holds its weights in fp32 instead (outputs 16 g + 8 h + 4 term + 0 .. 3 in a
// unit), as the terms cannot hold them: a weight is not finite, or some window, SiLU
// column or SiLU weight is too far below its scale, or a window or SiLU weight is zero for
// some outputs only (the others' gradients are then all that a dx has, however small
// beside those outputs').
template <typename T>
__device__ __forceinline__ void pack_dx2(const Dx2Args& a, int t, int ch) {
    constexpr bool BF = sizeof(T) == 2;
    constexpr int NT = BF ? 1 : 2;
    __shared__ __align__(16) uint16_t buf[NT][32][32][8];
    const int tid = threadIdx.x;
    const int g0 = ch * a.gmax, S = min(a.gmax, a.groups - g0);
    const int kl = tid & 31, e = tid >> 5;  // local K row, output within eight
    const int R = 32 * t + kl, f = R / a.cp, c = R % a.cp;
    // A row of the local K row (inverse of tile_row)
    const int r = 8 * ((kl % 16) / 4) + 4 * (kl / 16) + kl % 4;
    // the thread's column of the weights, one load per output (unconditional within
    // groups of eight, so that they are in flight together)
    const bool ok = f < a.in && c <= a.nb;
    const T* col = static_cast<const T*>(a.bw);
    int64_t stride = 0;
    if (ok) {
        col = c == 0 ? col + f : static_cast<const T*>(a.coef) + (int64_t)f * a.nb + c - 1;
        stride = (int64_t)a.in * (c == 0 ? 1 : a.nb);
    }
    T v[32];
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) {
#pragma unroll
        for (int i = 8 * ib; i < 8 * ib + 8; ++i) v[i] = T(0);
        if (4 * ib < S) {
#pragma unroll
            for (int i = 8 * ib; i < 8 * ib + 8; ++i)
                v[i] = col[(int64_t)min(16 * g0 + 8 * i + e, a.out - 1) * stride];
        }
#pragma unroll
        for (int i = 8 * ib; i < 8 * ib + 8; ++i)
            if (!ok || 16 * g0 + 8 * i + e >= a.out || i >= 2 * S) v[i] = T(0);
    }
    int ex = 0, es = 0;
    bool wide = false;
    if constexpr (!BF) {
        __shared__ floatx2 redm[4];
        __shared__ floatx2 reds[4];
        __shared__ int zeros[38], others[38], silu[32];  // (windows: per first K row; see edges)
        if (tid < 38) zeros[tid] = others[tid] = 0;
        if (tid < 32) silu[tid] = 0;
        __syncthreads();
        float m = 0.0f, mw = __builtin_inff();
        bool bad = false;
        // the windows that begin at the thread's column: the largest and the least of
        // their maxima's bits less 1 (an empty window is the largest then)
        uint32_t hi = 0u, lo = 0xffffffffu;
        const int outs = min((a.out - 16 * g0 - e + 7) / 8, 2 * S);  // the thread's
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const float av = __builtin_fabsf(v[i]);
            bad |= !(av < __builtin_inff());
            m = __builtin_fmaxf(m, av);
            // (past the thread's last output: its first again)
            const float w1 = i < outs ? av : __builtin_fabsf(v[0]);
            const float w2 = __builtin_fmaxf(w1, next_lane(w1));
            const float w3 = __builtin_fmaxf(w1, next_lane(w2));
            // (a SiLU weight is a window of its own)
            const uint32_t w4 = __float_as_uint(c == 0 ? w1 : __builtin_fmaxf(w1, next_lane(w3))) - 1u;
            hi = max(hi, w4);
            lo = min(lo, w4);
        }
        float ms = __builtin_inff();  // the least SiLU weight
        if (f < a.in && (c == 0 || (c + 3 <= a.nb && kl + 3 < 32)) && outs > 0) {
            if (hi == 0xffffffffu) zeros[kl] = 1;
            if (lo != 0xffffffffu) {
                others[kl] = 1;
                (c == 0 ? ms : mw) = __uint_as_float(lo + 1u);
            }
        }
        if (c == 0 && f < a.in) atomicMax(&silu[kl], (int)__float_as_uint(m));
        // features of several tiles: the windows over the tile's first and last edge,
        // an output per thread
        const int f0 = 32 * t / a.cp, cs = 32 * t % a.cp, o = 16 * g0 + tid;
        if (a.cp > 16 && tid < 16 * S && o < a.out) {
            const T* w = static_cast<const T*>(a.coef) + ((int64_t)o * a.in + f0) * a.nb - 1;
#pragma unroll
            for (int edge = 0; edge < 2; ++edge) {
                const int at = cs + 32 * edge;  // windows that begin 3 .. 1 columns before it
                float n[6];
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const int cc = at - 3 + k;
                    n[k] = cc >= 1 && cc <= a.nb ? __builtin_fabsf(w[cc]) : 0.0f;
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (at - 3 + k < 1 || at + k > a.nb) continue;
                    const float m4 = __builtin_fmaxf(__builtin_fmaxf(n[k], n[k + 1]),
                                                     __builtin_fmaxf(n[k + 2], n[k + 3]));
                    (m4 > 0.0f ? others : zeros)[32 + 3 * edge + k] = 1;
                    mw = m4 > 0.0f ? __builtin_fminf(mw, m4) : mw;
                }
            }
        }
        if (bad) m = __builtin_inff();
        float msl = c == 0 ? m : 0.0f;  // the largest SiLU weight
        m = c == 0 ? 0.0f : m;
#pragma unroll
        for (int k = 1; k < 64; k *= 2) {
            m = __builtin_fmaxf(m, __shfl_xor(m, k));
            msl = __builtin_fmaxf(msl, __shfl_xor(msl, k));
            mw = __builtin_fminf(mw, __shfl_xor(mw, k));
            ms = __builtin_fminf(ms, __shfl_xor(ms, k));
        }
        if (tid % 64 == 0) redm[tid / 64] = floatx2{m, mw}, reds[tid / 64] = floatx2{msl, ms};
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            m = __builtin_fmaxf(m, redm[k][0]);
            mw = __builtin_fminf(mw, redm[k][1]);
            msl = __builtin_fmaxf(msl, reds[k][0]);
            ms = __builtin_fminf(ms, reds[k][1]);
        }
        auto exponent = [](float q) -> int { return (int)(__float_as_uint(q) >> 23) - 127; };
        ex = exponent(m);
        es = exponent(msl);
        bool w = !(m < __builtin_inff()) || !(msl < __builtin_inff()) ||
                 exponent(mw) < ex - kPackWindowBits ||  // (infinity: no window)
                 exponent(ms) < es - kPackSiluBits;
        if (tid < 38) w |= (zeros[tid] & others[tid]) != 0;
        if (tid < 32)
            w |= silu[tid] != 0 && exponent(__uint_as_float((uint32_t)silu[tid])) < es - kPackWindowBits;
        wide = __syncthreads_or(w);
        if (tid == 0) a.wexp[t * a.nchunk + ch] = wide ? kPackWide : pack_word(ex, es);
    }
    if (!BF && wide) {
        float* raw = reinterpret_cast<float*>(&buf[0][0][0][0]);  // [output octet][A row][e]
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            if constexpr (!BF) raw[(i * 32 + r) * 8 + e] = v[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            if constexpr (BF) {
                buf[0][i][r][e] = v[i];
            } else {
                const float x = __builtin_ldexpf(v[i], kPackExp - (c == 0 ? es : ex));
                const _Float16 h0 = (_Float16)x;
                buf[0][i][r][e] = __builtin_bit_cast(uint16_t, h0);
                buf[NT - 1][i][r][e] = __builtin_bit_cast(uint16_t, (_Float16)(x - (float)h0));
            }
        }
    }
    __syncthreads();
    u32x4* dst = a.wtp + ((int64_t)t * a.groups + g0) * (NT * 64);
    for (int u = tid; u < S * NT * 64; u += 256) {
        const int lane = u % 64, term = u / 64 % NT, g = u / (64 * NT);
        const int at = 2 * g + lane / 32;
        if (!BF && wide)
            dst[u] = reinterpret_cast<const u32x4*>(&buf[0][0][0][0])[(at * 32 + lane % 32) * 2 + term];
        else
            dst[u] = *reinterpret_cast<const u32x4*>(&buf[term][at][lane % 32][0]);
    }
}

}  // namespace kan
