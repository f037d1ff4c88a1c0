// kan_window_kernel.h -- fused KAN-layer forward (eq. kan_forward) on the
// structured-sparse matrix instruction for any grid and degrees 1 .. 3: fp32
// layers as two fp16 terms per operand, and bf16 layers (cubic ones only where a
// feature takes other than two blocks of eight columns; those have a kernel of their
// own).
//
// Of a feature's basis columns only the k + 1 <= 4 whose support holds x can be
// nonzero (eq. bounded), and they are consecutive.  A feature's columns
// [SiLU, N_0 .. N_{nb-1}] are cut into blocks of 16; a step of the contraction
// is one block of a feature pair, 32 K slots of v_smfmac_f32_32x32x32_bf16
// (half of a wave per feature, four groups of four slots each).  Group g of a
// block holds its columns congruent to g (mod 4), so the window's four columns
// fall one per group and any two values per group can be nonzero: the dense
// contraction's exact zeros cost half the matrix-core time of the dense
// instruction, whatever G is.
//
// fp32 (NS = 2 terms): a basis value or a coefficient, scaled by a power of two,
// is the sum of two fp16 terms (each the round-to-nearest fp16 of what the
// former leaves: 11 + 11 bits and a sign, so all but the last of an fp32
// value's 24 bits, and that one where the first term rounds well: 4e-8 of it
// rms).  Both terms of a basis value sit in the
// two slots of its group at the same position, so one structured-sparse
// instruction multiplies both with a weight term, and two of them give all four
// products, exact in fp32 and accumulated in fp32.  The SiLU column, whose
// values have no bound, stays in fp32: one v_mfma_f32_32x32x2_f32 per feature
// pair.  Together 128 cycles per 32 x 32 tile and feature pair at G <= 12, where
// the fp32 instruction over all columns takes 1024, and fewer roundings of the
// accumulator, which set the layer's error: relative error (2-norm) against
// float64 at 65536 x 784 -> 256, G = 10: 8.7e-7, with the fp32 instruction 1.1e-6;
// 8192 x 128 -> 128, G = 100: 1.8e-7 both.  Times of a call at these sizes: 3198 ->
// 674 us and 312 -> 76 us.  Coefficients are scaled per output column by the power of two
// that brings the column's largest to [2^12, 2^13), and basis values by 2^12; a
// column's coefficients then have an absolute error of 2^-37 of its largest.  That
// is 2^-22 or less of the largest of any k + 1 consecutive coefficients of a
// feature (what one input meets) where none of these windows but empty ones is
// 2^15 below the column's scale.  A workgroup with a column that does not meet
// this (colmax_kernel), or with a sum that is not finite (a coefficient or an input
// that is not, or a SiLU value that only the scaled weight takes past fp32), takes
// its sums over all columns on the fp32 instruction (dense_tile) instead.
// bf16: a weight that is not finite would not meet exactly the values that it
// meets in the dense contraction (0 times infinity is NaN): it is taken as 0, an
// infinite SiLU weight as finite, and the terms are added at the end
// (fix_nonfinite).
//
// window_kernel: 8 waves, 256 rows x 64 NFW columns; the two waves of a 64-row
// group take the two column halves, each generates the A of one of the group's
// two 32-row tiles and passes it to the other through LDS.  Weights come
// expanded in the caller's workspace (expand_kernel) in the order the
// matrix cores read them, straight into LDS (D stages of SPB steps ahead).
#pragma once

#include "kan_internal.h"

namespace kan {
namespace win {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x16_t __attribute__((ext_vector_type(16)));

constexpr int kBasisExp = 12;  // fp32: basis values are scaled by 2^12 before the split
constexpr float kBasisScale = 4096.0f;

__device__ __forceinline__ uint32_t pk_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, bf16x2_t{(__bf16)lo, (__bf16)hi});
}
// bf16(v) in the low half, 0 in the high half.
__device__ __forceinline__ uint32_t lo_bf16(float v) {
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, 0" : "=v"(r) : "v"(v));
    return r;
}
// silu(x) / 2.
__device__ __forceinline__ float half_silu(float x) {
    return x * __builtin_amdgcn_rcpf(__builtin_fmaf(__expf(-x), 2.0f, 2.0f));
}
// N_K / 2 at v = u - (K + 1) / 2.
template <int K>
__device__ __forceinline__ float half_basis_k(float v) {
    if constexpr (K == 3) return half_basis(v);
    else return 0.5f * basis_deg<K>(v);
}

template <int NS> struct Elem;
template <> struct Elem<2> {
    typedef float T;
    static __device__ __forceinline__ float val(uint32_t u) { return __uint_as_float(u); }
    static __device__ __forceinline__ float val(float v) { return v; }
    static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<1> {
    typedef uint16_t T;
    static __device__ __forceinline__ float val(uint32_t u) { return __uint_as_float(u << 16); }
    static __device__ __forceinline__ float val(uint16_t v) { return bf16_to_f32(v); }
    static __device__ __forceinline__ void st(uint16_t* p, float v) { *p = f32_to_bf16(v); }
};

// ------------------------------------------------------------------- weights

// Column c of feature f for output o, read from the packed buffer
// (kan_internal.h; the dense layouts: fp32, and bf16 other than two blocks).
template <typename T>
__device__ __forceinline__ T packed_at(const WinArgs& a, int o, int pair, int f, int c) {
    constexpr int KJ = sizeof(T) == 2 ? 8 : 2;
    const int tile = o / a.pk_ntile, n = o % a.pk_ntile;
    const int64_t blk = (int64_t)tile * a.pk_nblk_pad + (int64_t)pair * a.pk_nsb + c / KJ;
    return static_cast<const T*>(a.wp)[((blk * 2 + f) * a.pk_ntile + n) * KJ + c % KJ];
}

// Columns of a window whose largest is 2^kWindowBits below the column's scale lose
// more than the last two bits of an fp32 value.
constexpr int kWindowBits = 15;

// Per output column over the pairs of group blockIdx.y (16 columns per workgroup),
// colmax[group][output] = largest finite |coefficient|, largest finite |SiLU
// weight|, and the least nonzero maximum of any k + 1 consecutive coefficients of
// a feature (infinity: there is none; 0: a coefficient is not finite).  A thread
// takes 8 units of two columns of a feature at a time, and the two before them for
// the windows that begin there, all ten in flight: its reads bound this kernel.
static __global__ __launch_bounds__(kThreads) void colmax_kernel(WinArgs a) {
    __shared__ floatx4 red[kWaves][16];
    constexpr int SEG = 8, NV = SEG + 2;
    const int cl = threadIdx.x & 15, sub = threadIdx.x >> 4;
    const int o = blockIdx.x * 16 + cl;
    const int per = (a.npairs + kColGroups - 1) / kColGroups;
    const int p_beg = min((int)blockIdx.y * per, a.npairs);
    const int p_end = min(p_beg + per, a.npairs);
    const int nseg = (a.pk_nsb + SEG - 1) / SEG;
    float mc = 0.0f, mb = 0.0f, mw = __builtin_inff();
    if (o < a.out) {
        const int tile = o / a.pk_ntile, n = o % a.pk_ntile;
        const floatx2* w = static_cast<const floatx2*>(a.wp) +
                           (int64_t)tile * a.pk_nblk_pad * 2 * a.pk_ntile + n;
        for (int it = sub; it < (p_end - p_beg) * 2 * nseg; it += kThreads / 16) {
            const int sg = it % nseg, pf = it / nseg;  // feature pf & 1 of pair p_beg + pf / 2
            const int64_t blk0 = (int64_t)(p_beg + pf / 2) * a.pk_nsb;
            const int b0 = sg * SEG - 2;
            floatx2 v[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int b = min(max(b0 + i, 0), a.pk_nsb - 1);
                v[i] = w[((blk0 + b) * 2 + (pf & 1)) * a.pk_ntile];
            }
            float m[2 * NV];  // |column 2 b0 + i|
#pragma unroll
            for (int i = 0; i < 2 * NV; ++i) {
                const int c = 2 * b0 + i;
                const float av = __builtin_fabsf(v[i / 2][i % 2]);
                const bool fin = av < __builtin_inff();
                m[i] = c >= 1 && c <= a.nb && fin ? av : 0.0f;
                mc = __builtin_fmaxf(mc, m[i]);
                if (c == 0) mb = __builtin_fmaxf(mb, fin ? av : 0.0f);
                if (c >= 1 && c <= a.nb && !fin) mw = 0.0f;
            }
#pragma unroll
            for (int i = 4; i < 2 * NV; ++i) {  // the window that ends with column c
                const int c = 2 * b0 + i;
                float x = __builtin_fmaxf(m[i], m[i - 1]);
                if (a.kdeg >= 2) x = __builtin_fmaxf(x, m[i - 2]);
                if (a.kdeg >= 3) x = __builtin_fmaxf(x, m[i - 3]);
                if (c > a.kdeg && c <= a.nb && x > 0.0f) mw = __builtin_fminf(mw, x);
            }
        }
    }
#pragma unroll
    for (int d = 16; d < 64; d *= 2) {
        mc = __builtin_fmaxf(mc, __shfl_xor(mc, d));
        mb = __builtin_fmaxf(mb, __shfl_xor(mb, d));
        mw = __builtin_fminf(mw, __shfl_xor(mw, d));
    }
    if ((sub & 3) == 0) red[sub >> 2][cl] = floatx4{mc, mb, mw, 0.0f};
    __syncthreads();
    if (threadIdx.x < 16 && o < a.out) {
#pragma unroll
        for (int i = 1; i < kWaves; ++i) {
            const floatx4 v = red[i][cl];
            mc = __builtin_fmaxf(mc, v[0]);
            mb = __builtin_fmaxf(mb, v[1]);
            mw = __builtin_fminf(mw, v[2]);
        }
        reinterpret_cast<floatx4*>(static_cast<char*>(a.ws) + a.off_cm)[(int64_t)blockIdx.y * a.out +
                                                                       o] =
            floatx4{mc, mb, mw, 0.0f};
    }
}

// Scale exponent of an output column from its largest values: coefficients are
// multiplied by 2^(12 - e).  e follows the coefficients, held within 2^24 of the
// SiLU weights (scaled along with them).  wide: the scale does not serve every
// window, or it would make the SiLU weights smaller than they are (which
// could lose one).
static __device__ __forceinline__ int scale_exp(const WinArgs& a, int o, bool& wide) {
    const floatx4* cm = reinterpret_cast<const floatx4*>(static_cast<const char*>(a.ws) + a.off_cm);
    float mc = 0.0f, mb = 0.0f, mw = __builtin_inff();
#pragma unroll
    for (int g = 0; g < kColGroups; ++g) {
        const floatx4 v = cm[(int64_t)g * a.out + o];
        mc = __builtin_fmaxf(mc, v[0]);
        mb = __builtin_fmaxf(mb, v[1]);
        mw = __builtin_fminf(mw, v[2]);
    }
    const int ec = (int)(__float_as_uint(mc) >> 23) - 127, eb = (int)(__float_as_uint(mb) >> 23) - 127;
    const int e = max(ec, eb - 24);
    const int ew = (int)(__float_as_uint(mw) >> 23) - 127;  // (128: no window)
    wide = mw == 0.0f || ew < e - kWindowBits || e > 12 + kBasisExp;
    return e;
}

// One workgroup expands one step (block j of a feature pair) of one column tile
// into step_u 16-byte units: unit (s, f, w, n) holds term s of columns
// 16 j + 4 (e % 4) + 2 w + e / 4, e = 0 .. 7, of feature f and output n; in fp32
// then the scaled SiLU weights [f][n].  Coefficients that are not finite become
// 0 and set the step's flag; in fp32 a column whose scale does not serve it sets the
// flag of all its steps.
template <int NS>
__global__ __launch_bounds__(256) void expand_kernel(WinArgs a) {
    typedef typename Elem<NS>::T T;
    const int step = blockIdx.x, tile = blockIdx.y;
    const int pair = step / a.nbk, j = step % a.nbk;
    const int bn = a.bn;
    u32x4* dst0 = reinterpret_cast<u32x4*>(static_cast<char*>(a.ws) + a.off_w) +
                  ((int64_t)tile * a.steps_pad + step) * a.step_u;
    // (256 is a multiple of bn: a thread's output is the same in every turn)
    const int n = threadIdx.x % bn, o = tile * bn + n;
    int ex = 0;
    bool wide = false;
    if constexpr (NS == 2)
        if (o < a.out) ex = scale_exp(a, o, wide);
    int bad = wide;
    for (int u = threadIdx.x; u < 4 * bn; u += 256) {
        const int w = u / bn % 2, f = u / (2 * bn);
        u32x4* dst = dst0 + u;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = 16 * j + 4 * (e % 4) + 2 * w + e / 4;
            v[e] = 0.0f;
            if (o < a.out && c <= a.nb && (NS == 1 || c > 0)) {
                const T t = packed_at<T>(a, o, pair, f, c);
                if constexpr (NS == 2) v[e] = t;
                else v[e] = bf16_to_f32(t);
                if (!(__builtin_fabsf(v[e]) < __builtin_inff())) {
                    // (an infinite SiLU weight, which can meet an infinite value: the
                    // largest finite one of its sign)
                    const bool silu_inf = NS == 1 && c == 0 && v[e] == v[e];
                    v[e] = silu_inf ? __builtin_copysignf(__uint_as_float(0x7f7f0000u), v[e]) : 0.0f;
                    bad = 1;
                }
            }
        }
        if constexpr (NS == 1) {
            dst[0] = u32x4{pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3]), pk_bf16(v[4], v[5]),
                           pk_bf16(v[6], v[7])};
        } else {
            f16x8_t t0, t1;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float r = __builtin_ldexpf(v[e], 12 - ex);
                t0[e] = (_Float16)r;
                t1[e] = (_Float16)(r - (float)t0[e]);
            }
            dst[0] = __builtin_bit_cast(u32x4, t0);
            dst[4 * bn] = __builtin_bit_cast(u32x4, t1);
            if (w == 0) {
                float b = 0.0f;
                if (o < a.out && j == 0) b = __builtin_ldexpf(packed_at<float>(a, o, pair, f, 0),
                                                              12 + kBasisExp - ex);
                reinterpret_cast<float*>(dst0 + 8 * bn)[f * bn + n] = b;
                if (step == 0 && f == 0)
                    reinterpret_cast<int*>(static_cast<char*>(a.ws) + a.off_us)[o] =
                        ex - 12 - kBasisExp;
            }
        }
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0)
        reinterpret_cast<int*>(static_cast<char*>(a.ws) + a.off_flag)[tile * a.steps + step] = bad;
    if (NS == 1 && step == a.steps - 1) {
        // (a last step that fills a stage of two: zero weights)
        const int64_t left = (int64_t)(a.steps_pad - a.steps) * a.step_u;
        u32x4* end = dst0 + a.step_u;
        for (int64_t u = threadIdx.x; u < left; u += 256) end[u] = u32x4{0, 0, 0, 0};
    }
}

// ----------------------------------------------------------- non-finite terms

// bf16: adds to the workgroup's tile of outputs (already stored) the terms of the
// non-finite weights (flagged steps), with the values and products the dense
// contraction has (also 0 times an infinite weight, NaN).  P: the split's partial
// sums, or null.
template <int K>
__device__ __forceinline__ void fix_nonfinite(const WinArgs& a, float* P, int64_t row_beg,
                                              int col_beg, int bm, int t_beg, int t_end,
                                              const int* flag) {
    typedef Elem<1> E;
    const uint16_t* x = static_cast<const uint16_t*>(a.x);
    uint16_t* y = static_cast<uint16_t*>(a.y);
    for (int u = threadIdx.x; u < bm * a.bn; u += kThreads) {
        const int64_t row = row_beg + u / a.bn;
        const int o = col_beg + u % a.bn;
        if (row >= a.batch || o >= a.out) continue;
        float add = 0.0f;
        for (int t = t_beg; t < t_end && add == add; ++t) {
            if (flag[t] == 0) continue;
            const int p = t / a.nbk, c_beg = 16 * (t % a.nbk);
            const int c_end = min(c_beg + 15, a.nb);
            for (int f = 0; f < 2 && 2 * p + f < a.in; ++f) {
                const float xv = E::val(x[row * a.in + 2 * p + f]);
                const float lo = coord_lo(xv, a.xlim, a.inv_lo, a.a_frac);
                for (int c = c_beg; c <= c_end; ++c) {
                    const float w = E::val(packed_at<uint16_t>(a, o, p, f, c));
                    if (__builtin_fabsf(w) < __builtin_inff()) continue;
                    const float v =
                        __builtin_fmaf(xv, a.inv_h, a.a_int + 1.0f - (float)c) + lo;
                    add += (c == 0 ? half_silu(xv) : half_basis_k<K>(v)) * w;
                }
            }
        }
        if (add == 0.0f) continue;
        const int64_t at = row * a.out + o;
        if (P != nullptr) P[at] += 2.0f * add;
        else E::st(y + at, E::val(y[at]) + 2.0f * add);
    }
}

// -------------------------------------------- fp32 instruction, every column

// The sums of a wave's two row tiles (rows row[0], row[1] of lane r) and NF column
// fragments (outputs col[nf] of lane r) over the pairs [p_beg, p_end), every column
// of their features on the fp32 instruction: acc = y / 2.  The weights come from the
// packed buffer a block ahead, a fragment's 32 outputs in one contiguous run per
// lane half.  Whole calls where every workgroup takes this path, against the kernel that
// reads the packed weights through LDS: 8192 x 128 -> 128, G = 100: 349 us (316), 16384 x
// 256 -> 64: 140 (124), 4096 x 256 -> 256, G = 20, degree 1: 184 (214), 65536 x 784 -> 256:
// 4.9 ms (3.2: one fragment at a time generates the basis values four times).
template <int K, int NF>
__device__ __forceinline__ void dense_tile(const WinArgs& a, const int64_t (&row)[2],
                                           const int (&col)[NF], int h, int p_beg, int p_end,
                                           floatx16 (&acc)[2][NF]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int nf = 0; nf < NF; ++nf)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][nf][q] = 0.0f;
    const float* x = static_cast<const float*>(a.x);
    const floatx2* w[NF];
    floatx2 wn[NF];
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) {
        w[nf] = static_cast<const floatx2*>(a.wp) +
                (((int64_t)(col[nf] / a.pk_ntile) * a.pk_nblk_pad + (int64_t)p_beg * a.pk_nsb) * 2 +
                 h) * a.pk_ntile + col[nf] % a.pk_ntile;
        wn[nf] = *w[nf];
    }
    const int step = 2 * a.pk_ntile;
    int left = (p_end - p_beg) * a.pk_nsb - 1;  // blocks after the one in wn
    float xn[2];
    auto load_x = [&](int p) {
        const int f = 2 * p + h;  // (an odd feature count's phantom: x = 0, zero weights)
#pragma unroll
        for (int i = 0; i < 2; ++i) xn[i] = f < a.in ? x[row[i] * a.in + f] : 0.0f;
    };
    load_x(p_beg);
#pragma unroll 1
    for (int p = p_beg; p < p_end; ++p) {
        const float xv[2] = {xn[0], xn[1]};
        load_x(min(p + 1, p_end - 1));
        float lo[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) lo[i] = coord_lo(xv[i], a.xlim, a.inv_lo, a.a_frac);
#pragma unroll 1
        for (int b = 0; b < a.pk_nsb; ++b) {
            floatx2 wv[NF];
            const int adv = left > 0 ? step : 0;
            --left;
#pragma unroll
            for (int nf = 0; nf < NF; ++nf) {
                wv[nf] = wn[nf];
                w[nf] += adv;
                wn[nf] = *w[nf];
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float c = (float)(2 * b + j);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    float v = half_basis_k<K>(__builtin_fmaf(xv[i], a.inv_h, a.a_int + 1.0f - c) +
                                              lo[i]);
                    if (j == 0 && b == 0) v = half_silu(xv[i]);
#pragma unroll
                    for (int nf = 0; nf < NF; ++nf)
                        acc[i][nf] = __builtin_amdgcn_mfma_f32_32x32x2f32(v, wv[nf][j], acc[i][nf],
                                                                          0, 0, 0);
                }
            }
        }
    }
}

// -------------------------------------------------------------------- kernel

template <int NS, int NFW, bool MB, int K>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void window_kernel(WinArgs a) {
    typedef typename Elem<NS>::T T;
    constexpr int SPB = NS == 2 ? 1 : 2;  // steps per stage (a barrier each)
    constexpr int D = NS == 2 ? 1 : 2;    // stages between a load and its use
    constexpr int NBS = D + 1;            // weight stages in LDS
    constexpr int BN = 64 * NFW;
    constexpr int BM = 256;
    constexpr int STEP_U = win_step_units(NS == 1, BN);  // 16-byte units of a step's weights
    constexpr int STG_U = SPB * STEP_U;
    constexpr int WL = STG_U / 64;        // wave loads of a stage
    constexpr int NLD = (WL + kWaves - 1) / kWaves;
    // The loads of a stage that every wave issues, when they are the same for
    // all of them (D > 1 counts them): the x of its steps, then its weights.
    static_assert(D == 1 || WL % kWaves == 0, "loads per wave");
    constexpr int LDS_STAGE = SPB + NLD;
    static_assert(LDS_STAGE < 16, "vmcnt field");
    __shared__ u32x4 bs[NBS * STG_U];
    __shared__ u32x4 as[2][kWaves][SPB][64];   // A, its positions, fp32: SiLU
    __shared__ uint32_t ai[2][kWaves][SPB][64];
    __shared__ float asl[NS == 2 ? 2 : 1][kWaves][SPB][64];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int r = lane & 31, h = lane >> 5;
    const int wr = wave & 3, wc = wave >> 2;  // row group, column half (= tile generated)
    const int64_t row_beg = (int64_t)blockIdx.x * BM;
    const int tile = blockIdx.y;
    const int st_beg = blockIdx.z * a.sps;  // the split's first stage
    const int nst = min(a.sps, a.stages - st_beg);

    // weights of this tile from the split's first stage on
    const char* wsrc = static_cast<const char*>(a.ws) + a.off_w +
                       ((size_t)tile * a.steps_pad + (size_t)st_beg * SPB) * (STEP_U * 16);
    const uint64_t wbase = reinterpret_cast<uint64_t>(wsrc);
    u32x4 wrs;
    wrs[0] = __builtin_amdgcn_readfirstlane((uint32_t)wbase);
    wrs[1] = __builtin_amdgcn_readfirstlane((uint32_t)(wbase >> 32) & 0xffffu);
    wrs[2] = __builtin_amdgcn_readfirstlane((uint32_t)nst * (uint32_t)(STG_U * 16));
    wrs[3] = (uint32_t)kBufferWord3;
    const uint32_t bs_lds =
        (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)bs);

    // x: the rows of the tile this wave generates
    const T* xw = static_cast<const T*>(a.x) + row_beg * (int64_t)a.in;
    const uint64_t x_left = (uint64_t)(a.batch - row_beg) * (uint64_t)a.in * sizeof(T);
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(xw), (short)0, (int)(x_left < 0xffffffffull ? x_left : 0xffffffffull),
        kBufferWord3);
    int64_t xrow = row_beg + wr * 64 + wc * 32 + r;
    xrow = xrow < a.batch ? xrow : a.batch - 1;
    const uint32_t xbyte = (uint32_t)(((xrow - row_beg) * a.in + h) * (int)sizeof(T));
    // (an odd feature count: the last pair's phantom lanes read the real
    // feature and use x = 0)
    const int odd_pair = (a.in & 1) ? a.npairs - 1 : -1;

    // The split's steps start at a whole pair.  xp, xj: pair and block of the
    // next step to load x for; gp, gj: of the next to generate.
    const int t_beg = st_beg * SPB;
    const int p_beg = MB ? t_beg / a.nbk : t_beg;
    int xp = p_beg, xj = 0, gp = p_beg, gj = 0;
    auto next = [&](int& p, int& j) {
        if constexpr (MB) {
            j = j + 1 == a.nbk ? 0 : j + 1;
            p += j == 0 ? 1 : 0;
        } else {
            ++p;
        }
    };
    auto load_x = [&](uint32_t (&xs)[SPB]) {
#pragma unroll
        for (int q = 0; q < SPB; ++q) {
            const int p = min(xp, a.npairs - 1);
            next(xp, xj);
            const uint32_t vo = xbyte - (p == odd_pair && h ? (uint32_t)sizeof(T) : 0u);
            if constexpr (NS == 2)
                xs[q] = __builtin_amdgcn_raw_buffer_load_b32(xrs, vo, 8 * p, 0);
            else
                xs[q] = __builtin_amdgcn_raw_buffer_load_b16(xrs, vo, 4 * p, 0);
        }
    };
    // weights of stage st to LDS buffer st % NBS (stages past the last re-read it)
    auto load_w = [&](int stage, int buf) {
        const int st = min(stage, nst - 1);
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int wl = wave + kWaves * i;
            if (i + 1 < NLD || WL % kWaves == 0 || wl < WL)
                dma16(wrs, (uint32_t)lane * 16u,
                      (uint32_t)st * (uint32_t)(STG_U * 16) + (uint32_t)wl * 1024u,
                      bs_lds + (uint32_t)buf * (uint32_t)(STG_U * 16) + (uint32_t)wl * 1024u);
        }
    };

    // ---- A of a step.  The feature's window: val[g] holds the value of group g
    // (its column c0 + ((g - c0) mod 4)): both fp16 terms, or in bf16 the value in
    // the low half; silu the SiLU value (bf16: in the high half, the second slot
    // of group 0, at position 0).  Position of group g's column in its block:
    // (column / 4) mod 4, two bits per slot in pos.  Only MB: the block of c0
    // and how many groups wrapped into the next one.
    uint32_t val[4], silu = 0, pos;
    int blk0 = 0, wrap = 0;
    const float cmax = (float)(16 * a.nbk - 4);
    // The generation in four parts of some 20 VALU instructions each, so that the
    // main loop can put them between its MFMAs.
    struct Gen {
        float x, lo, d, sl, bv[4];
        int c0;
        uint32_t kg;
    };
    auto gen_part = [&](auto part, Gen& G, uint32_t raw, bool phantom) __attribute__((always_inline)) {
        constexpr int PART = decltype(part)::value;
        if constexpr (PART == 0) {
            float x = Elem<NS>::val(raw);
            x = phantom && h != 0 ? 0.0f : x;
            G.x = x;
            G.lo = coord_lo(x, a.xlim, a.inv_lo, a.a_frac);
            const float sv = __builtin_fmaf(x, a.inv_h, a.a_int + 1.0f) + G.lo;
            // first window column, within the blocks and past the SiLU column: a
            // column the clamp takes in is at |v| >= (K + 1) / 2, where the form
            // is exactly 0 (a NaN coordinate gives column 1 and NaN values).  Degrees
            // 1 and 2 need 2 and 3 of the four columns: the window starts 1 and 1/2
            // lower, so that the rounding of its position loses no value.
            constexpr float low = 0.5f * (float)(K - 1) + (K == 1 ? 1.0f : K == 2 ? 0.5f : 0.0f);
            const float cf = __builtin_amdgcn_fmed3f(__builtin_floorf(sv - low), 1.0f, cmax);
            G.c0 = (int)cf;
            // v of column c0 in one rounding at its own magnitude
            G.d = __builtin_fmaf(x, a.inv_h, a.a_int + 1.0f - cf) + G.lo;
            // byte g: (g - c0) mod 4
            G.kg = __builtin_amdgcn_alignbit(0x03020100u, 0x03020100u,
                                             (uint32_t)(32 - 8 * (G.c0 & 3)));
        } else if constexpr (PART == 1 || PART == 2) {
#pragma unroll
            for (int g = 2 * PART - 2; g < 2 * PART; ++g)
                G.bv[g] = half_basis_k<K>(G.d - (float)((G.kg >> (8 * g)) & 0xffu));
            if constexpr (PART == 1) G.sl = half_silu(G.x);
        } else {
            const int q = G.c0 >> 2, rr = G.c0 & 3;
            const uint32_t low = (1u << (4 * rr)) - 1u;  // groups g < rr
            if constexpr (NS == 2) {
                silu = __float_as_uint(G.sl);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float v = G.bv[g] * kBasisScale;
                    const _Float16 t = (_Float16)v;
                    val[g] = __builtin_bit_cast(uint32_t, f16x2_t{t, (_Float16)(v - (float)t)});
                }
                if constexpr (MB)
                    pos = (q & 3) == 3 ? 0xffffu & ~low
                                       : (uint32_t)(q & 3) * 0x5555u + (0x5555u & low);
                else
                    pos = __umul24((uint32_t)q, 0x5555u) + (0x5555u & low);
            } else {
                const uint32_t w0 = pk_bf16(G.bv[0], G.sl);
                val[0] = MB ? (w0 & 0xffffu) : w0;
                silu = w0 & 0xffff0000u;
#pragma unroll
                for (int g = 1; g < 4; ++g) val[g] = lo_bf16(G.bv[g]);
                if constexpr (MB)
                    pos = ((uint32_t)(q & 3) * 0x1111u + (0x1111u & low)) & 0x3333u;
                else
                    pos = __umul24((uint32_t)q, 0x1111u) + (0x1111u & low);
            }
            if constexpr (MB) {
                blk0 = G.c0 >> 4;
                wrap = (q & 3) == 3 ? rr : 0;
            }
        }
    };
    // the A operand of block j of the feature generated last
    auto block_a = [&](int j, bool real) -> u32x4 {
        if constexpr (MB) {
            // groups of the window in block j: those not wrapped (j = blk0) or
            // those wrapped (j = blk0 + 1)
            const int rel = j - blk0;
            const uint32_t low = (1u << wrap) - 1u;
            const uint32_t keep = !real ? 0u : rel == 0 ? ~low : rel == 1 ? low : 0u;
            uint32_t m[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) m[g] = (uint32_t)((int)(keep << (31 - g)) >> 31);
            const uint32_t sm = NS == 1 && real && j == 0 ? 0xffffffffu : 0u;
            return u32x4{(val[0] & m[0]) | (silu & sm), val[1] & m[1], val[2] & m[2],
                         val[3] & m[3]};
        } else {
            if (SPB > 1 && !real) return u32x4{0u, 0u, 0u, 0u};
            return u32x4{val[0], val[1], val[2], val[3]};
        }
    };
    // the A of the next stage (x already loaded): generated at a pair's first
    // block, exchanged through exchange stage e
    struct AOp {
        u32x4 a[SPB];
        uint32_t pos[SPB];
        float silu[SPB];
    };
    // part 0 .. 3 of the next step's A; the last passes it on (exchange stage e)
    auto make_part = [&](auto part, Gen& G, uint32_t raw, int q, int e,
                         AOp& A) __attribute__((always_inline)) {
        constexpr int PART = decltype(part)::value;
        if (!MB || gj == 0) gen_part(part, G, raw, gp == odd_pair);
        if constexpr (PART == 3) {
            const bool real = SPB == 1 || gp < a.npairs;
            A.a[q] = block_a(gj, real);
            A.pos[q] = pos;
            next(gp, gj);
            as[e][wave][q][lane] = A.a[q];
            ai[e][wave][q][lane] = A.pos[q];
            if constexpr (NS == 2) {
                A.silu[q] = __uint_as_float(silu);
                asl[e][wave][q][lane] = A.silu[q];
            }
        }
    };
    AOp own;
    Gen gn;

    // fp32, where the registers allow (64 and 128 columns): the products with the
    // second weight terms and the SiLU column in accumulators of their own, so that
    // the main ones round twice per step and not six times
    constexpr bool ACC2 = NS == 2 && NFW <= 2;
    floatx16 acc[2][NFW], acc2[2][ACC2 ? NFW : 1];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int nf = 0; nf < NFW; ++nf)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                acc[i][nf][q] = 0.0f;
                if constexpr (ACC2) acc2[i][nf][q] = 0.0f;
            }
    auto silu_mul = [&](const u32x4* bb, int nf, int col, float own_s, float par_s) {
        const float b = reinterpret_cast<const float*>(bb + 8 * BN)[h * BN + col];
        floatx16& c0 = ACC2 ? acc2[0][ACC2 ? nf : 0] : acc[0][nf];
        floatx16& c1 = ACC2 ? acc2[1][ACC2 ? nf : 0] : acc[1][nf];
        c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(own_s, b, c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(par_s, b, c1, 0, 0, 0);
    };

    // vmcnt(n), lgkmcnt(0)
    auto wait_stage = [&](auto nn) {
        constexpr int n = decltype(nn)::value;
        __builtin_amdgcn_s_waitcnt((n & 15) | (0x7 << 4) | (0x0 << 8) | ((n >> 4) << 14));
    };
    auto fence = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    const int t_end = min((st_beg + nst) * SPB, a.steps);
    const int* flag = reinterpret_cast<const int*>(static_cast<const char*>(a.ws) + a.off_flag) +
                      tile * a.steps;
    int bad = 0;

    // ---- prologue: x and weights of stages 0 .. D - 1, the A of stage 0
    uint32_t xq[D][SPB];
    {
        uint32_t x0[SPB];
        load_x(x0);
#pragma unroll
        for (int d = 0; d < D; ++d) load_x(xq[d]);
#pragma unroll
        for (int d = 0; d < D; ++d) load_w(d, d);
        StaticFor<0, 4 * SPB>::run([&](auto k) {
            constexpr int kk = decltype(k)::value;
            make_part(std::integral_constant<int, kk % 4>{}, gn, x0[kk / 4], kk / 4, 0, own);
        });
        for (int t = t_beg + tid; t < t_end; t += kThreads) bad |= flag[t];
        wait_stage(std::integral_constant<int, 0>{});
        fence();
    }
    // (fp32: the flagged steps' workgroup takes its sums by dense_tile alone)
    bad = __syncthreads_or(bad);
    const int nst_run = NS == 2 && bad ? 0 : nst;
    u32x4 par;
    int par_pos = 0;
    float par_silu = 0.0f;
    int cj = 0;                   // MB, fp32: block of the step
    int buf = 0, fill = D % NBS;  // LDS buffer of the stage, and of the one D ahead
#pragma unroll 1
    for (int st = 0; st < nst_run; ++st) {
        const int e = st & 1;
        uint32_t xn[SPB], xl[SPB];
#pragma unroll
        for (int q = 0; q < SPB; ++q) xn[q] = xq[0][q];
        load_x(xl);
        load_w(st + D, fill);
        AOp nxt;
        const u32x4* bb = bs + buf * STG_U;
        // The stage's SPB NFW segments: a fragment's MFMAs, and a share of the next
        // stage's generation (4 parts per step) in front of them, so that a SIMD's
        // two waves fall into alternating VALU and matrix phases.
        StaticFor<0, SPB * NFW>::run([&](auto seg) __attribute__((always_inline)) {
            constexpr int S = decltype(seg)::value, q = S / NFW, nf = S % NFW;
            const int pw = wr + 4 * (1 - wc);  // the partner
            if constexpr (nf == 0) {
                par = as[e][pw][q][lane];
                par_pos = (int)ai[e][pw][q][lane];
                if constexpr (NS == 2) par_silu = asl[e][pw][q][lane];
            }
            const int own_pos = (int)own.pos[q];
            const int col = (wc * NFW + nf) * 32 + r;
            const u32x4* bq = bb + q * STEP_U;
            u32x4 b[NS][2];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                b[s][0] = bq[(s * 4 + h) * BN + col];
                b[s][1] = bq[(s * 4 + 2 + h) * BN + col];
            }
            constexpr int P0 = 4 * SPB * S / (SPB * NFW), P1 = 4 * SPB * (S + 1) / (SPB * NFW);
            StaticFor<P0, P1>::run([&](auto k) __attribute__((always_inline)) {
                constexpr int kk = decltype(k)::value;
                make_part(std::integral_constant<int, kk % 4>{}, gn, xn[kk / 4], kk / 4, e ^ 1,
                          nxt);
            });
#pragma unroll
            for (int s = NS - 1; s >= 0; --s) {
                if constexpr (NS == 2) {
                    const f16x16_t bv = __builtin_shufflevector(
                        __builtin_bit_cast(f16x8_t, b[s][0]), __builtin_bit_cast(f16x8_t, b[s][1]), 0,
                        1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                    floatx16& c0 = ACC2 && s == 1 ? acc2[0][ACC2 ? nf : 0] : acc[0][nf];
                    floatx16& c1 = ACC2 && s == 1 ? acc2[1][ACC2 ? nf : 0] : acc[1][nf];
                    c0 = __builtin_amdgcn_smfmac_f32_32x32x32_f16(
                        __builtin_bit_cast(f16x8_t, own.a[q]), bv, c0, own_pos, 0, 0);
                    c1 = __builtin_amdgcn_smfmac_f32_32x32x32_f16(
                        __builtin_bit_cast(f16x8_t, par), bv, c1, par_pos, 0, 0);
                } else {
                    const bf16x16 bv = __builtin_shufflevector(
                        __builtin_bit_cast(bf16x8, b[s][0]), __builtin_bit_cast(bf16x8, b[s][1]), 0, 1,
                        2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                    acc[0][nf] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(
                        __builtin_bit_cast(bf16x8, own.a[q]), bv, acc[0][nf], own_pos, 0, 0);
                    acc[1][nf] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(
                        __builtin_bit_cast(bf16x8, par), bv, acc[1][nf], par_pos, 0, 0);
                }
            }
            if constexpr (NS == 2) {
                // the SiLU column, with the feature's first block
                if (!MB || cj == 0) silu_mul(bq, nf, col, own.silu[q], par_silu);
                if constexpr (MB && nf == NFW - 1) cj = cj + 1 == a.nbk ? 0 : cj + 1;
            }
            if constexpr (!MB) __builtin_amdgcn_sched_barrier(0);
        });
        own = nxt;
        wait_stage(std::integral_constant<int, (D - 1) * LDS_STAGE>{});
#pragma unroll
        for (int d = 0; d + 1 < D; ++d)
#pragma unroll
            for (int q = 0; q < SPB; ++q) xq[d][q] = xq[d + 1][q];
#pragma unroll
        for (int q = 0; q < SPB; ++q) xq[D - 1][q] = xl[q];
        buf = buf + 1 == NBS ? 0 : buf + 1;
        fill = fill + 1 == NBS ? 0 : fill + 1;
        fence();
    }
    wait_stage(std::integral_constant<int, 0>{});  // (no load to LDS may outlive the workgroup)

    // ---- epilogue: y = 2 acc (fp32: unscaled); acc[i] is the row group's tile i ^ wc
    const int col_beg = tile * BN;
    float* P = a.ks > 1 ? reinterpret_cast<float*>(static_cast<char*>(a.ws) + a.off_p) +
                              (int64_t)blockIdx.z * a.batch * a.out
                        : nullptr;
    T* y = static_cast<T*>(a.y);
    // one 32 x 32 tile's sums times 2^us
    auto store = [&](int i, int col, const floatx16& c, int us, int half)
                     __attribute__((always_inline)) {
        const int64_t row0 = row_beg + wr * 64 + (i ^ wc) * 32 + 4 * half;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int64_t row = row0 + 8 * (q / 4) + q % 4;
            if (row < a.batch && col < a.out) {
                const float v = NS == 2 ? __builtin_ldexpf(c[q], us) : 2.0f * c[q];
                if (P != nullptr) P[row * a.out + col] = v;
                else Elem<NS>::st(y + row * a.out + col, v);
            }
        }
    };
    if constexpr (NS == 2) {
        float fin = 0.0f;  // (NaN once a sum is not finite)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int nf = 0; nf < NFW; ++nf)
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    if constexpr (ACC2) acc[i][nf][q] += acc2[i][nf][q];
                    fin = __builtin_fmaf(acc[i][nf][q], 0.0f, fin);
                }
        if (__builtin_amdgcn_readfirstlane(__syncthreads_or(bad | !(fin == 0.0f)))) {
            // fragments at a time (two at 256 columns would make the main loop spill)
            constexpr int NF = NFW == 2 ? 2 : 1;
#pragma unroll 1
            for (int n0 = 0; n0 < NFW; n0 += NF) {
                // (opaque, so that the stores' addresses are not computed ahead for all
                // turns or for both paths, which would spill)
                int rr = r, hh = h;
                asm volatile("" : "+v"(rr), "+v"(hh));
                int64_t row[2];
                int col[NF], colc[NF];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    row[i] = min(row_beg + wr * 64 + (i ^ wc) * 32 + rr, a.batch - 1);
#pragma unroll
                for (int n = 0; n < NF; ++n) {
                    col[n] = col_beg + (wc * NFW + n0 + n) * 32 + rr;
                    colc[n] = min(col[n], a.out - 1);
                }
                floatx16 d[2][NF];
                dense_tile<K, NF>(a, row, colc, hh, p_beg, t_end / a.nbk, d);
#pragma unroll
                for (int n = 0; n < NF; ++n) {
                    store(0, col[n], d[0][n], 1, hh);
                    store(1, col[n], d[1][n], 1, hh);
                }
            }
            return;
        }
    }
#pragma unroll
    for (int nf = 0; nf < NFW; ++nf) {
        const int col = col_beg + (wc * NFW + nf) * 32 + r;
        int us = 1;
        if constexpr (NS == 2)
            us = 1 + reinterpret_cast<const int*>(static_cast<const char*>(a.ws) + a.off_us)[col];
        store(0, col, acc[0][nf], us, h);
        store(1, col, acc[1][nf], us, h);
    }
    if constexpr (NS == 1) {
        if (bad) {
            __syncthreads();  // (the outputs are stored)
            fix_nonfinite<K>(a, P, row_beg, col_beg, BM, t_beg, t_end, flag);
        }
    }
}

template <int NS, int NFW, bool MB>
hipError_t launch_k(const WinArgs& a, dim3 grid, hipStream_t s) {
    switch (a.kdeg) {
        case 1: hipLaunchKernelGGL((window_kernel<NS, NFW, MB, 1>), grid, dim3(kThreads), 0, s, a); break;
        case 2: hipLaunchKernelGGL((window_kernel<NS, NFW, MB, 2>), grid, dim3(kThreads), 0, s, a); break;
        case 3: hipLaunchKernelGGL((window_kernel<NS, NFW, MB, 3>), grid, dim3(kThreads), 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int NS>
hipError_t launch_ns(const WinGeom& g, const WinArgs& a, hipStream_t s) {
    if constexpr (NS == 2)
        hipLaunchKernelGGL(colmax_kernel, dim3((unsigned)((a.out + 15) / 16), kColGroups), dim3(kThreads),
                           0, s, a);
    hipLaunchKernelGGL(expand_kernel<NS>, dim3((unsigned)a.steps, (unsigned)g.ntiles), dim3(256), 0,
                       s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)g.rblocks, (unsigned)g.ntiles, (unsigned)g.ks);
    const bool mb = g.nbk > 1;
    switch (g.nfw) {
        case 1: return mb ? launch_k<NS, 1, true>(a, grid, s) : launch_k<NS, 1, false>(a, grid, s);
        case 2: return mb ? launch_k<NS, 2, true>(a, grid, s) : launch_k<NS, 2, false>(a, grid, s);
        case 4: return mb ? launch_k<NS, 4, true>(a, grid, s) : launch_k<NS, 4, false>(a, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace win
}  // namespace kan
