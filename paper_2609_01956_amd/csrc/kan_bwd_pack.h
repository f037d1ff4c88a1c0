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

// One workgroup packs K tile t for output chunk ch (groups g0 .. g0 + S - 1 of 16
// outputs): [t][g][term][lane (r, h)][e], outputs 16 g + 8 h + e of the K row of A
// row r.  fp32: scaled per (tile, chunk), wexp[t nchunk + ch] = the exponent
// (biased by 512; bit 16: a weight was not finite, and taken as 0).
template <typename T>
__device__ __forceinline__ void pack_dx2(const Dx2Args& a, int t, int ch) {
    constexpr bool BF = sizeof(T) == 2;
    constexpr int NT = BF ? 1 : 2;
    __shared__ __align__(16) uint16_t buf[NT][32][32][8];
    __shared__ float redm[256];
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
    int ex = 0;
    if constexpr (!BF) {
        float m = 0.0f;
        bool bad = false;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const float av = __builtin_fabsf(v[i]);
            const bool fin = av < __builtin_inff();
            bad |= !fin;
            v[i] = fin ? v[i] : 0.0f;
            m = __builtin_fmaxf(m, fin ? av : 0.0f);
        }
        redm[tid] = m;
        const int anybad = __syncthreads_or(bad);
        for (int k = 128; k >= 1; k >>= 1) {
            if (tid < k) redm[tid] = __builtin_fmaxf(redm[tid], redm[tid + k]);
            __syncthreads();
        }
        ex = (int)(__float_as_uint(redm[0]) >> 23) - 127;
        if (tid == 0) a.wexp[t * a.nchunk + ch] = (ex + 512) | (anybad ? 1 << 16 : 0);
    }
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        if constexpr (BF) {
            buf[0][i][r][e] = v[i];
        } else {
            const float x = __builtin_ldexpf(v[i], 12 - ex);
            const _Float16 h0 = (_Float16)x;
            buf[0][i][r][e] = __builtin_bit_cast(uint16_t, h0);
            buf[NT - 1][i][r][e] = __builtin_bit_cast(uint16_t, (_Float16)(x - (float)h0));
        }
    }
    __syncthreads();
    u32x4* dst = a.wtp + ((int64_t)t * a.groups + g0) * (NT * 64);
    for (int u = tid; u < S * NT * 64; u += 256) {
        const int lane = u % 64, term = u / 64 % NT, g = u / (64 * NT);
        dst[u] = *reinterpret_cast<const u32x4*>(&buf[term][2 * g + lane / 32][lane % 32][0]);
    }
}

}  // namespace kan
