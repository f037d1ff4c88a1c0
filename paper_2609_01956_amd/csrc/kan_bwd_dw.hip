// kan_bwd_dw.hip -- weight gradients of the KAN layer on the matrix cores
// (eq. kan_forward differentiated):
//
//   dC[o, i, j] = sum_b dy[b, o] N_j(x[b, i]),   dWb[o, i] = sum_b dy[b, o] silu(x[b, i])
//
// as dW^T = A^T dy over the batch, for layers whose cp K rows per feature divide
// 256 (cp a power of two: every workgroup's 256 K rows are whole features).
// bf16: one bf16 operand each.  fp32: both operands as two fp16 terms (what the
// first leaves, rounded again: 22 bits and a sign), three products (the fourth
// is below 2^-22 of the first), exact in fp32, fp32 accumulation: 96 cycles per
// 16 rows of a 32 x 32 tile where the fp32 matrix instruction takes 512 (784 ->
// 256 at 16384 rows, the weight gradients alone: 844 -> 339 us a call; relative error
// against float64 6.2e-7 -> 4.0e-7).  dy is
// scaled per output and SiLU values per feature by the power of two that brings
// the largest of the workgroup's rows to 2^14 (from the maxima that the
// transposition leaves per 64 rows), basis values by 2^12, and second terms by
// 2^11 more: their products have accumulators of their own, and so an operand is
// within 2^-36 or 2^-23 of its value.  Where an output's dy or a feature's SiLU values
// range over more than 2^29 (the transposition leaves the least, too), a sum can be
// made of values alone that the terms hold badly; the sums that are then below
// what these errors can add up to, times 2^17, are taken again at the end
// (exact_tile), and so are those of an output with a non-finite dy and of a SiLU row
// with an infinite value.
//
// Per chunk of 32 batch rows the workgroup stages dy (transposed) and the A
// operand in LDS, double-buffered.  A is built once per workgroup: a thread owns
// one (row, feature), writes the four window columns and the SiLU column and
// clears the four it wrote two chunks before in the same stage; everything else
// stays 0.  The window is clamped to the feature's columns 1 .. cp - 4: what it
// then takes in is exactly 0, or a padding row past nb, which nobody reads; so
// the four K rows are consecutive and one address serves all of them.
#include "kan_internal.h"

namespace kan {

namespace {

constexpr int kThreads = 512;
constexpr int kBasisExp = 12, kDyExp = 14;
constexpr int kTermExp = 11;     // second terms: their own scale
constexpr float kTermScale = 1 << kTermExp;
constexpr int kSpreadBits = 29;  // exponents within which two terms hold 21 bits and more

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float half_silu_w(float x) {
    return x * __builtin_amdgcn_rcpf(__builtin_fmaf(__expf(-x), 2.0f, 2.0f));
}

// Exponent of a maximum (of finite values): scaling by 2^(14 - e) brings it to [2^14, 2^15).
__device__ __forceinline__ int max_exp(float m) {
    return (int)((__float_as_uint(m) >> 23) & 0xffu) - 127;
}

// ------------------------------------------------------- transposition, fp32

// dst[c][b] = src[b][c], zero-padded to ceil(cols / 32) * 32 rows and rpad (a
// multiple of 64) columns, in tiles of 64 rows by 32 columns; and per tile the
// largest finite |value| of each column, with the sign bit set if a value is not
// finite, and the least nonzero |value|, or at most that of |silu(value)| / 2 (infinity if none):
// range[b / 64][c], c < ceil(cols / 32) * 32.
template <bool SILU>
__global__ __launch_bounds__(256) void transpose_range_kernel(const float* __restrict__ src,
                                                              float* __restrict__ dst,
                                                              floatx2* __restrict__ range,
                                                              int64_t rows, int cols, int64_t rpad) {
    __shared__ float tile[64][33];
    __shared__ float red[8][33], redl[8][33];
    const int64_t b0 = (int64_t)blockIdx.x * 64;
    const int c0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    float m = 0.0f, lo = __builtin_inff(), neg = 0.0f;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t b = b0 + ty + 8 * k;
        const float v = (b < rows && c0 + tx < cols) ? src[b * cols + c0 + tx] : 0.0f;
        tile[ty + 8 * k][tx] = v;
        const float av = __builtin_fabsf(v);
        const bool fin = av < __builtin_inff();
        m = __builtin_fmaxf(m, fin ? av : 0.0f);
        bad |= !fin;
        lo = av > 0.0f ? __builtin_fminf(lo, av) : lo;  // (a NaN isn't)
        if (SILU) neg = __builtin_fminf(neg, v);
    }
    if (SILU && lo < __builtin_inff()) {
        // least |silu|: of the value nearest 0, at its negative, or of the lowest (to
        // -85, below which it is soon 0)
        const float l0 = half_silu_w(-__builtin_fminf(lo, 85.0f));
        const float l1 = half_silu_w(__builtin_fmaxf(neg, -85.0f));
        lo = __builtin_fminf(-l0, neg < 0.0f ? -l1 : -l0);
    }
    redl[ty][tx] = lo;
    red[ty][tx] = bad ? -m : m;
    if (bad && m == 0.0f) red[ty][tx] = -0.0f;
    __syncthreads();
    const int bl = threadIdx.x & 63, cq = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int cl = cq + 4 * k;
        dst[(int64_t)(c0 + cl) * rpad + b0 + bl] = tile[bl][cl];
    }
    if (threadIdx.x < 32) {
        uint32_t s = 0;
        float mx = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float v = red[k][threadIdx.x];
            mx = __builtin_fmaxf(mx, __builtin_fabsf(v));
            s |= __float_as_uint(v) & 0x80000000u;
            lo = __builtin_fminf(lo, redl[k][threadIdx.x]);
        }
        range[(int64_t)blockIdx.x * (gridDim.y * 32) + c0 + threadIdx.x] =
            floatx2{__uint_as_float(__float_as_uint(mx) | s), lo};
    }
}

// -------------------------------------------------------------------- kernel

// fp32: elements of a wave's tile (32 K rows from kt, 32 outputs from o0; bit q of
// mask: the lane's accumulator q) summed again on the fp32 instruction, straight from
// the transposed operands, 64 batch rows at a time: the blocks where a dy or an x of
// the tile is not finite, and those with a row in the support of one of the K rows of
// small (bit r: K row kt + r).  A function of its own, so that the main loop keeps its
// registers; args: the kernel's, in place.  dW of 16384 x 784 -> 256: 0.38 ms per call
// without such elements, 1.4 ms where they are all (one row of gradients of 1e10
// beside others of 1; 0.8 ms where the fp32 instruction was the kernel's own).
__device__ __attribute__((noinline)) void exact_tile(const uint32_t* args, int kt, int o0,
                                                     uint32_t mask, uint32_t small) {
    struct Words { uint32_t w[sizeof(Dw2Args) / 4]; } words;
    static_assert(sizeof(Words) == sizeof(Dw2Args), "whole words");
#pragma unroll
    for (size_t i = 0; i < sizeof(Dw2Args) / 4; ++i)
        words.w[i] = __builtin_amdgcn_readfirstlane(args[i]);
    const Dw2Args a = __builtin_bit_cast(Dw2Args, words);
    kt = __builtin_amdgcn_readfirstlane(kt);
    o0 = __builtin_amdgcn_readfirstlane(o0);
    small = __builtin_amdgcn_readfirstlane(small);
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int f = min((kt + r) / a.cp, a.in - 1), c = (kt + r) % a.cp;  // the lane's K row
    const float* xr = static_cast<const float*>(a.xt) + (int64_t)f * a.bpad + 32 * h;
    const float* dr = static_cast<const float*>(a.dyt) + (int64_t)(o0 + r) * a.bpad + 32 * h;
    // the lane's range per block: an output's, or a K row's feature's
    const bool has = h != 0 || o0 + r < a.out32;
    const floatx2* rng = h != 0 ? a.xrange + f : a.dyrange + min(o0 + r, a.out32 - 1);
    const int rw = h != 0 ? a.in32 : a.out32;
    // the tile's features (two of 16 columns, or 32 columns from c0 of one) and K rows
    // of small
    const int f0 = kt / a.cp, c0 = kt % a.cp, f1 = a.cp == 16 ? min(f0 + 1, a.in - 1) : f0;
    const float* x0 = static_cast<const float*>(a.xt) + (int64_t)f0 * a.bpad + lane;
    const float* x1 = static_cast<const float*>(a.xt) + (int64_t)f1 * a.bpad + lane;
    const uint32_t small0 = a.cp == 16 ? small & 0xffffu : small;
    const uint32_t small1 = a.cp == 16 ? small >> 16 : 0u;
    const bool every = c0 == 0 && ((small0 | small1) & 1u) != 0;  // a SiLU row: every block
    auto meets = [&](float x, uint32_t cols) -> bool {
        const float sv = __builtin_fmaf(x, a.inv_h, a.a_int + 1.0f) +
                         coord_lo(x, a.xlim, a.inv_lo, a.a_frac);
        // window columns first .. first + 3, and one more on each side for sv's rounding
        const int first = (int)__builtin_amdgcn_fmed3f(__builtin_floorf(sv) - 1.0f, -8.0f,
                                                       (float)(a.cp + 8)) - c0;
        const uint64_t win = first < -8 || first > 32 ? 0 : 0x3full << (first + 8) >> 1;
        return ((uint32_t)(win >> 8) & cols) != 0;
    };
    const int64_t b_begin = (int64_t)blockIdx.y * a.rows_per_split;
    const int64_t b_end = min(b_begin + a.rows_per_split, a.bpad);
    auto value = [&](float x, int col) -> float {  // of K row col of x's feature
        const float v = half_basis(__builtin_fmaf(x, a.inv_h, a.a_int + 1.0f - (float)col) +
                                   coord_lo(x, a.xlim, a.inv_lo, a.a_frac));
        return col == 0 ? half_silu_w(x) : v;
    };
    float* P = a.P + ((int64_t)blockIdx.y * a.out32 + o0) * a.kr + kt;
    // A few elements (sums that cancel): one after the other, a row per lane.  (Softmax
    // gradients, 16384 x 784 -> 256, some elements in all: dW 588 -> 412 us)
    int count = __builtin_popcount(mask);
#pragma unroll
    for (int k = 1; k < 64; k *= 2) count += __shfl_xor(count, k);
    if (__builtin_amdgcn_readfirstlane(count) <= 8) {
#pragma unroll 1
        for (uint64_t who = __ballot(mask != 0); who != 0; who = __ballot(mask != 0)) {
            const int src = __ffsll((unsigned long long)who) - 1;
            const int q = __builtin_amdgcn_readlane(__ffs((int)mask) - 1, src);
            const int kr = 8 * (q / 4) + 4 * (src / 32) + q % 4, o = src % 32;
            const int col = (kt + kr) % a.cp;
            const float* xs = static_cast<const float*>(a.xt) + (int64_t)((kt + kr) / a.cp) * a.bpad;
            const float* ds = static_cast<const float*>(a.dyt) + (int64_t)(o0 + o) * a.bpad;
            float sum = 0.0f;
#pragma unroll 8
            for (int64_t b = b_begin + lane; b < b_end; b += 64)
                sum = __builtin_fmaf(value(xs[b], col), ds[b], sum);
#pragma unroll
            for (int k = 1; k < 64; k *= 2) sum += __shfl_xor(sum, k);
            if (lane == src) P[(int64_t)o * a.kr + kr] = sum;
            if (lane == src) mask &= mask - 1;
        }
        return;
    }
    floatx16 acc;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
    bool done = false;
#pragma unroll 1
    for (int64_t bb = b_begin; bb < b_end && !done; bb += 16 * 64) {
        const int n = (int)min((int64_t)16, (b_end - bb) / 64);
        uint32_t blocks = 0;
        if (small == 0) {
#pragma unroll 8
            for (int j = 0; j < n; ++j) {
                const bool in = has && __float_as_uint(rng[(bb / 64 + j) * rw][0]) >> 31 != 0;
                blocks |= (uint32_t)(__ballot(in) != 0) << j;
            }
        } else {
#pragma unroll 8
            for (int j = 0; j < n; ++j) {
                bool in = every || (has && __float_as_uint(rng[(bb / 64 + j) * rw][0]) >> 31 != 0);
                in |= meets(x0[bb + 64 * j], small0) || meets(x1[bb + 64 * j], small1);
                blocks |= (uint32_t)(__ballot(in) != 0) << j;
            }
        }
#pragma unroll 1
        for (; blocks != 0; blocks &= blocks - 1) {
            const int64_t b0 = bb + 64 * (__ffs((int)blocks) - 1);
#pragma unroll 2
            for (int i = 0; i < 32; i += 4) {
                const floatx4 x4 = *reinterpret_cast<const floatx4*>(xr + b0 + i);
                const floatx4 d4 = *reinterpret_cast<const floatx4*>(dr + b0 + i);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(value(x4[e], c), d4[e], acc, 0, 0, 0);
            }
            uint32_t open = mask;  // (a NaN stays one)
#pragma unroll
            for (int q = 0; q < 16; ++q) open &= ~(acc[q] != acc[q] ? 1u << q : 0u);
            done = __ballot(open != 0) == 0;
            if (done) break;
        }
    }
#pragma unroll
    for (int q = 0; q < 16; ++q)
        if ((mask >> q & 1) != 0) P[(int64_t)r * a.kr + 4 * h + 8 * (q / 4) + q % 4] = acc[q];
}

// FULL: cp = 16, so every thread owns a (row, feature) of each chunk.
template <typename T, int OH, int NFW, bool FULL>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void dw_split_kernel(Dw2Args a) {
    constexpr bool BF = sizeof(T) == 2;
    constexpr int NT = BF ? 1 : 2;              // terms per operand
    constexpr int RF = OH, KG = 8 / OH;
    constexpr int KT = 256;
    constexpr int OT = OH * NFW * 32;
    constexpr int AROW = 80;                    // bytes of an A row: 32 values and 16 of padding
    constexpr int UR = BF ? 4 : 8;              // 16-byte loads of a chunk's 32 dy values
    constexpr int DU = (OT * UR + kThreads - 1) / kThreads;
    static_assert(KG * RF * 32 == KT, "K rows");
    // dy rows of 64 bytes, their 16-byte units permuted by the row so that a
    // fragment read of 16 rows falls in distinct banks (A rows: by the padding)
    __shared__ u32x4 dys[2][NT][OT * 4];
    __shared__ u32x4 as[2][NT][KT * AROW / 16];
    __shared__ int nanf[16];
    // scale exponents; bit 16: non-finite, bit 17: a spread past kSpreadBits
    __shared__ int exd[BF ? 1 : OT], exs[BF ? 1 : 16];

    const T* __restrict__ xt = static_cast<const T*>(a.xt);
    const T* __restrict__ dyt = static_cast<const T*>(a.dyt);
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, r = lane & 31, h = lane >> 5;
    const int kg = wave / OH, oh = wave % OH;
    const int kt0 = blockIdx.x * KT, ot0 = blockIdx.z * OT;
    const int F0 = kt0 / a.cp, nfeat = FULL ? 16 : KT / a.cp;
    const int64_t b_begin = (int64_t)blockIdx.y * a.rows_per_split;
    const int64_t b_end = min(b_begin + a.rows_per_split, a.bpad);
    const int nchunks = (int)((b_end - b_begin) / 32);

    if (tid < 16) nanf[tid] = 0;
    for (int i = tid; i < 2 * NT * KT * AROW / 16; i += kThreads)
        (&as[0][0][0])[i] = u32x4{0u, 0u, 0u, 0u};
    if constexpr (!BF) {
        // ranges over the split's rows
        const int64_t m0 = b_begin / 64, m1 = (b_end + 63) / 64;
        for (int i = tid; i < OT + 16; i += kThreads) {
            const bool isx = i >= OT;
            const int c = isx ? F0 + i - OT : ot0 + i;
            const int w = isx ? a.in32 : a.out32;
            const floatx2* src = isx ? a.xrange : a.dyrange;
            float m = 0.0f, lo = __builtin_inff();
            uint32_t s = 0;
            if (c < w)
#pragma unroll 8
                for (int64_t k = m0; k < m1; ++k) {
                    const floatx2 v = src[k * w + c];
                    m = __builtin_fmaxf(m, __builtin_fabsf(v[0]));
                    s |= __float_as_uint(v[0]) >> 31;
                    lo = __builtin_fminf(lo, v[1]);
                }
            if (max_exp(lo) < max_exp(m) - kSpreadBits) s |= 2u;
            // (low half: the exponent, biased by 512)
            const int e = (max_exp(m) + 512) | (int)(s << 16);
            if (isx) exs[i - OT] = e;
            else exd[i] = e;
        }
    }
    __syncthreads();

    // the thread's (row, feature) of each chunk, and its LDS place in an A row
    const int bl = tid & 31, fl = tid >> 5;
    const bool own = FULL || fl < nfeat;
    const int fx = min(F0 + min(fl, nfeat - 1), a.in - 1);
    const bool pad_f = F0 + fl >= a.in;
    const T* xsrc = xt + (int64_t)fx * a.bpad + b_begin + bl;
    const uint32_t abase = (uint32_t)(min(fl, nfeat - 1) * a.cp * AROW + bl * 2);
    const float cmax = (float)(a.cp - 4);
    int sscale = 0;
    if constexpr (!BF) sscale = kDyExp - ((exs[min(fl, nfeat - 1)] & 0xffff) - 512);
    // dy units of the thread: outputs ol + k kThreads / UR, 16-byte load w of each
    // output's 32 values (the transposed dy has rows up to the last tile's end:
    // what those past out32 hold is not used)
    constexpr int KO = kThreads / UR;
    static_assert(KO % 16 == 0, "the units' permutation is the same for every k");
    const int ol0 = tid / UR, w0 = tid % UR;
    const bool dlast = (OT * UR) % kThreads == 0 || ol0 < OT;  // (OT < KO: some threads idle)
    const T* dsrc = dyt + (int64_t)(ot0 + (dlast ? ol0 : 0)) * a.bpad + b_begin +
                    w0 * (16 / (int)sizeof(T));
    const uint32_t dput = (uint32_t)(ol0 * 64 + (((BF ? w0 : w0 / 2) ^ ((ol0 >> 2) & 3)) * 16) +
                                     (BF ? 0 : (w0 & 1) * 8));
    const int64_t dstep = (int64_t)KO * a.bpad;

    // dy of the next chunk: bf16 in two register sets, loaded two chunks ahead;
    // fp32 in one (its registers are short), loaded when the former was staged
    constexpr int ND = BF ? 2 : 1;
    typedef u32x4 DSet[DU];
    DSet dq[ND];
    T xq[2];
    uint32_t prev[2];  // window address written two chunks ago in each stage
    prev[0] = prev[1] = abase + AROW;
    bool nanx = false;
    auto issue_dy = [&](int ck, DSet& d) {
        const int64_t b0 = 32 * (int64_t)min(ck, nchunks - 1);
#pragma unroll
        for (int k = 0; k < DU; ++k)
            d[k] = *reinterpret_cast<const u32x4*>(dsrc + b0 + k * dstep);
    };
    auto issue_x = [&](int ck, T& xs) { xs = xsrc[32 * (int64_t)min(ck, nchunks - 1)]; };

    // Staging of a chunk in parts, placed between the MFMAs of the other stage:
    // parts 0 .. 3 the A values, parts 4 .. 3 + DU a dy unit each.
    struct Gen {
        float x, lo, d, sl, bv[4];
        uint32_t adr;
    };
    Gen gn;
    auto st16 = [&](int buf, int t, uint32_t adr, uint16_t v) {
        *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(&as[buf][t][0]) + adr) = v;
    };
    auto stage_part = [&](auto part, int buf, const DSet& d, T xs,
                          uint32_t& pv) __attribute__((always_inline)) {
        constexpr int P = decltype(part)::value;
        if constexpr (P >= 4) {
            constexpr int k = P - 4;
            if (dlast) {
                if constexpr (BF) {
                    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(&dys[buf][0][0]) + dput + k * (KO * 64)) =
                        d[k];
                } else {
                    const int ds = kDyExp + kTermExp + 512 - (exd[ol0 + k * KO] & 0xffff);
                    f16x4_t t0, t1;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        // (a non-finite dy becomes a finite one: its output is computed apart)
                        const float v = __builtin_amdgcn_fmed3f(
                            __builtin_ldexpf(__uint_as_float(d[k][e]), ds), -0x1p26f, 0x1p26f);
                        t0[e] = (_Float16)(v * (1.0f / kTermScale));
                        t1[e] = (_Float16)__builtin_fmaf((float)t0[e], -kTermScale, v);
                    }
                    *reinterpret_cast<u32x2_t*>(reinterpret_cast<char*>(&dys[buf][0][0]) + dput + k * (KO * 64)) =
                        __builtin_bit_cast(u32x2_t, t0);
                    *reinterpret_cast<u32x2_t*>(reinterpret_cast<char*>(&dys[buf][1][0]) + dput + k * (KO * 64)) =
                        __builtin_bit_cast(u32x2_t, t1);
                }
            }
        } else if (own) {
            if constexpr (P == 0) {
                float x;
                if constexpr (BF) x = bf16_to_f32(xs);
                else x = xs;
                x = pad_f ? 0.0f : x;
                gn.x = x;
                nanx |= x != x;
                gn.lo = coord_lo(x, a.xlim, a.inv_lo, a.a_frac);
                const float sv = __builtin_fmaf(x, a.inv_h, a.a_int + 1.0f) + gn.lo;
                const float cf = __builtin_amdgcn_fmed3f(__builtin_floorf(sv) - 1.0f, 1.0f, cmax);
                gn.d = __builtin_fmaf(x, a.inv_h, a.a_int + 1.0f - cf) + gn.lo;
                gn.adr = abase + __umul24((uint32_t)(int)cf, (uint32_t)AROW);
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int m = 0; m < 4; ++m) st16(buf, t, pv + m * AROW, 0);
                pv = gn.adr;
            } else if constexpr (P == 1) {
                gn.sl = half_silu_w(gn.x);
                gn.bv[0] = half_basis(gn.d);
                gn.bv[1] = half_basis(gn.d - 1.0f);
            } else if constexpr (P == 2) {
                gn.bv[2] = half_basis(gn.d - 2.0f);
                gn.bv[3] = half_basis(gn.d - 3.0f);
            } else {
                if constexpr (BF) {
                    const uint32_t w01 = __builtin_bit_cast(
                        uint32_t, bf16x2_t{(__bf16)gn.bv[0], (__bf16)gn.bv[1]});
                    const uint32_t w23 = __builtin_bit_cast(
                        uint32_t, bf16x2_t{(__bf16)gn.bv[2], (__bf16)gn.bv[3]});
                    st16(buf, 0, abase, f32_to_bf16(gn.sl));
                    st16(buf, 0, gn.adr, (uint16_t)w01);
                    st16(buf, 0, gn.adr + AROW, (uint16_t)(w01 >> 16));
                    st16(buf, 0, gn.adr + 2 * AROW, (uint16_t)w23);
                    st16(buf, 0, gn.adr + 3 * AROW, (uint16_t)(w23 >> 16));
                } else {
                    auto two = [&](uint32_t adr, float v, float scale) {
                        const _Float16 t = (_Float16)(v * scale);
                        st16(buf, 0, adr, __builtin_bit_cast(uint16_t, t));
                        st16(buf, 1, adr,
                             __builtin_bit_cast(uint16_t, (_Float16)__builtin_fmaf(
                                                              (float)t, -kTermScale,
                                                              v * (scale * kTermScale))));
                    };
                    two(abase, __builtin_ldexpf(gn.sl, sscale), 1.0f);
#pragma unroll
                    for (int m = 0; m < 4; ++m)
                        two(gn.adr + m * AROW, gn.bv[m], (float)(1 << kBasisExp));
                }
            }
        }
    };

    // fp32: the products with a second term have accumulators of their own, so that
    // the main ones round twice per 16 rows (six times, their sums have a larger
    // error than the fp32 instruction's: 7.9e-7 against 6.7e-7 relative to float64
    // over 65536 rows); at most 64 registers each, so tiles of up to 128 outputs.
    static_assert(BF || RF * NFW <= 4, "fp32: two sets of accumulators");
    floatx16 acc[RF][NFW], acc2[BF ? 1 : RF][BF ? 1 : NFW];
#pragma unroll
    for (int rt = 0; rt < RF; ++rt)
#pragma unroll
        for (int nf = 0; nf < NFW; ++nf)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                acc[rt][nf][q] = 0.0f;
                if constexpr (!BF) acc2[rt][nf][q] = 0.0f;
            }

    // The MFMAs of stage buf, in segments; between them the next chunk is staged
    // into stage buf ^ 1.
    constexpr int NPART = 4 + DU, NSEG = 2 * NFW;
    u32x4 A[RF][NT];
    auto chunk = [&](int buf, const DSet& d, T xs, uint32_t& pv, auto with) {
        StaticFor<0, NSEG>::run([&](auto seg) __attribute__((always_inline)) {
            constexpr int S = decltype(seg)::value, s = S / NFW, nf = S % NFW;
            if constexpr (nf == 0) {
#pragma unroll
                for (int rt = 0; rt < RF; ++rt)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        A[rt][t] = as[buf][t][(32 * (kg * RF + rt) + r) * (AROW / 16) + 2 * s + h];
            }
            u32x4 b[NT];
            const int ol = (oh * NFW + nf) * 32 + r;
#pragma unroll
            for (int t = 0; t < NT; ++t) b[t] = dys[buf][t][ol * 4 + ((2 * s + h) ^ ((ol >> 2) & 3))];
            if constexpr (decltype(with)::value) {
                StaticFor<NPART * S / NSEG, NPART*(S + 1) / NSEG>::run(
                    [&](auto p) __attribute__((always_inline)) { stage_part(p, buf ^ 1, d, xs, pv); });
            }
#pragma unroll
            for (int rt = 0; rt < RF; ++rt) {
                if constexpr (BF) {
                    acc[rt][nf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8, A[rt][0]), __builtin_bit_cast(bf16x8, b[0]),
                        acc[rt][nf], 0, 0, 0);
                } else {
                    auto mul = [&](int ta, int tb, floatx16& c) __attribute__((always_inline)) {
                        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                            __builtin_bit_cast(f16x8_t, A[rt][ta]), __builtin_bit_cast(f16x8_t, b[tb]),
                            c, 0, 0, 0);
                    };
                    mul(NT - 1, 0, acc2[BF ? 0 : rt][BF ? 0 : nf]);
                    mul(0, 0, acc[rt][nf]);
                    mul(0, NT - 1, acc2[BF ? 0 : rt][BF ? 0 : nf]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // Stage ck % 2 holds chunk ck, staged during chunk ck - 1.  The loop stages one
    // chunk past the last (loads clamped to the last; never multiplied).
    issue_x(0, xq[0]);
    issue_x(1, xq[1]);
    issue_dy(0, dq[0]);
    if constexpr (BF) issue_dy(1, dq[1 % ND]);
    StaticFor<0, NPART>::run([&](auto p) { stage_part(p, 0, dq[0], xq[0], prev[0]); });
    if constexpr (!BF) issue_dy(1, dq[0]);
    __syncthreads();
    int ck = 0;
    for (; ck + 1 < nchunks; ck += 2) {
        issue_x(ck + 2, xq[0]);
        if constexpr (BF) issue_dy(ck + 2, dq[0]);
        chunk(0, dq[1 % ND], xq[1], prev[1], std::true_type{});
        if constexpr (!BF) issue_dy(ck + 2, dq[0]);
        __syncthreads();
        issue_x(ck + 3, xq[1]);
        if constexpr (BF) issue_dy(ck + 3, dq[1 % ND]);
        chunk(1, dq[0], xq[0], prev[0], std::true_type{});
        if constexpr (!BF) issue_dy(ck + 3, dq[0]);
        __syncthreads();
    }
    if (ck < nchunks) chunk(0, dq[0], xq[1], prev[1], std::false_type{});
    if (own && nanx) nanf[fl] = 1;
    bool fix = false;  // (fp32) some element is to be summed again
    if constexpr (BF) {
        __syncthreads();
    } else {
        int any = 0;
        for (int i = tid; i < OT + 16; i += kThreads) any |= (i < OT ? exd[i] : exs[i - OT]) >> 16;
        fix = __syncthreads_or(any) != 0;
    }
    // Bounds of the error of a sum by the terms' 2^-36 (scaled as the sum: basis
    // values are at most 2^12 / 3, the others less than 2^15), times 2^17.
    const float rows = (float)(b_end - b_begin);
    const float tiny = rows * 0x1p-8f, tiny_silu = rows * 0x1p-3f;

    // acc[rt][nf][q] = (scaled dW^T / 2)[K row kt0 + lr][output], lr = 32 (kg RF + rt) +
    // 8 (q / 4) + 4 h + q % 4.  A feature with a NaN input: its basis gradients
    // are NaN (N_j(NaN) is NaN; the clamped form gave 0).
    float* P = a.P + (int64_t)blockIdx.y * a.out32 * a.kr;
#pragma unroll
    for (int rt = 0; rt < RF; ++rt) {
#pragma unroll
        for (int nf = 0; nf < NFW; ++nf) {
            const int ol = (oh * NFW + nf) * 32 + r;
            const int o = ot0 + ol;
            int ed = 0;
            uint32_t again = 0, small = 0;  // elements to be summed again, K rows of small ones
            if constexpr (!BF) ed = (exd[ol] & 0xffff) - 512 - kDyExp;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int lr = 32 * (kg * RF + rt) + 8 * m + 4 * h;
                const int f = lr / (FULL ? 16 : a.cp);
                const int c = lr - f * (FULL ? 16 : a.cp);  // (a multiple of 4)
                const bool isn = nanf[f] != 0;
                floatx4 v;
                uint32_t low = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float t = acc[rt][nf][4 * m + e];
                    if constexpr (!BF) {
                        t = __builtin_fmaf(acc2[BF ? 0 : rt][BF ? 0 : nf][4 * m + e],
                                           1.0f / kTermScale, t);
                        const bool si = e == 0 && c == 0;
                        if (__builtin_fabsf(t) < (si ? tiny_silu : tiny)) low |= 1u << e;
                        const int ea = si ? (exs[f] & 0xffff) - 512 - kDyExp : -kBasisExp;
                        t = __builtin_ldexpf(t, ed + ea);
                    }
                    v[e] = isn && (c != 0 || e != 0) ? __builtin_nanf("") : t;
                }
                if (o < a.out32 && kt0 + lr < a.kr) {
                    *reinterpret_cast<floatx4*>(P + (int64_t)o * a.kr + kt0 + lr) = v;
                    if (!BF && fix && F0 + f < a.in) {
                        // an output's non-finite dy reaches every K row (0 times infinity
                        // is NaN), a feature's non-finite x its SiLU row
                        const int fo = exd[BF ? 0 : ol] >> 16, fx = c == 0 ? exs[BF ? 0 : f] >> 16 : 0;
                        uint32_t bad = ((fo & 1) != 0 ? 15u : 0u) | (fx & 1);
                        uint32_t few = low & (((fo & 2) != 0 ? 15u : 0u) | fx >> 1);
                        // (not the padding past nb, nor what is NaN by its feature)
                        const uint32_t keep = isn ? (c == 0 ? 1u : 0u)
                                                  : (1u << min(4, max(0, a.nb + 1 - c))) - 1u;
                        bad &= keep;
                        few &= keep;
                        again |= (bad | few) << (4 * m);
                        small |= few << (8 * m + 4 * h);
                    }
                }
            }
            if (!BF && __ballot(again != 0) != 0) {
#pragma unroll
                for (int k = 1; k < 64; k *= 2) small |= (uint32_t)__shfl_xor((int)small, k);
                exact_tile((const uint32_t*)__builtin_amdgcn_kernarg_segment_ptr(),
                           kt0 + 32 * (kg * RF + rt), ot0 + (oh * NFW + nf) * 32, again, small);
            }
        }
    }
}

template <typename T, int OH, int NFW>
void launch_shape(const Dw2Args& a, dim3 grid, hipStream_t s) {
    if (a.cp == 16)
        hipLaunchKernelGGL((dw_split_kernel<T, OH, NFW, true>), grid, dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((dw_split_kernel<T, OH, NFW, false>), grid, dim3(kThreads), 0, s, a);
}

template <typename T>
hipError_t launch_t(const BwdGeom& g, const Dw2Args& a, hipStream_t s) {
    const dim3 grid((unsigned)g.ktiles, (unsigned)g.split, (unsigned)g.otiles);
    if (g.oh == 1 && g.nfw == 1) launch_shape<T, 1, 1>(a, grid, s);
    else if (g.oh == 2 && g.nfw == 1) launch_shape<T, 2, 1>(a, grid, s);
    else if (g.oh == 2 && g.nfw == 2) launch_shape<T, 2, 2>(a, grid, s);
    else if (sizeof(T) == 2 && g.oh == 2 && g.nfw == 4) launch_shape<uint16_t, 2, 4>(a, grid, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_transpose_range(const float* src, float* dst, floatx2* range, bool silu,
                                  int64_t rows, int cols, int64_t rpad, hipStream_t s) {
    const dim3 grid((unsigned)(rpad / 64), (unsigned)((cols + 31) / 32));
    if (silu)
        hipLaunchKernelGGL(transpose_range_kernel<true>, grid, dim3(256), 0, s, src, dst, range,
                           rows, cols, rpad);
    else
        hipLaunchKernelGGL(transpose_range_kernel<false>, grid, dim3(256), 0, s, src, dst, range,
                           rows, cols, rpad);
    return hipGetLastError();
}

hipError_t launch_dw_split(bool bf16, const BwdGeom& g, const Dw2Args& a, hipStream_t s) {
    return bf16 ? launch_t<uint16_t>(g, a, s) : launch_t<float>(g, a, s);
}

}  // namespace kan
