// Per-token FP8 quantisation of activations (Sec. 2.1 eq. 2):  A = FP8(x / beta), beta per row.
//   beta = absmax / 448 in FP32 (1 for an all-zero row); quotient as IEEE FP32 division would give
//   it; conversion to OCP E4M3 round-to-nearest-even by the hardware converter.  No quotient of the short form passes 448 by more
//   than its rounding (|x| <= absmax, which is why a row with a NaN may not take it); the full division clamps to +-448: a
//   NaN, and an infinity over its row's infinite scale, become -448.
// The quotient.  A full IEEE division is about eleven instructions per element.  With r = 1 / beta, q = x * r, the residual
// e = fma(q, beta, -x) (exact) and q' = fma(e, -r, q), the stored E4M3 code equals that of the IEEE quotient, the sign of
// zero included, for every finite bf16 x with |x| <= absmax and every beta = absmax / 448 in [2^-60, 2^60]: checked
// exhaustively on the host (5.3e8 pairs).  Rows with beta outside that range, or with a NaN, take the full division.
#include <type_traits>
#include "fq_common.h"
#include "fq_kernels.h"


// Sum of the eight E4M3 values of two words of codes.
__device__ __forceinline__ float fq_sum8(fq_v2i o) {
    const fq_v2f a = __builtin_amdgcn_cvt_pk_f32_fp8(o[0], false), b = __builtin_amdgcn_cvt_pk_f32_fp8(o[0], true);
    const fq_v2f c = __builtin_amdgcn_cvt_pk_f32_fp8(o[1], false), d = __builtin_amdgcn_cvt_pk_f32_fp8(o[1], true);
    return ((a[0] + a[1]) + (b[0] + b[1])) + ((c[0] + c[1]) + (d[0] + d[1]));
}

template <int CTRL>
__device__ __forceinline__ float fq_dpp_add(float v) {
    return v + __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
}

// WPR waves per row, up to CH chunks (of 16 bytes, 8 bf16) of it per thread in registers between the search for the
// largest magnitude and the conversion, so that the row is read once; longer rows are read a second time (REREAD).
// Bound by HBM (3 bytes per element); what keeps it from there is the latency of a row (load, maximum, conversion, store one
// after the other) against the rows a compute unit has under way: fq_launch_quantize_as picks WPR and CH by that.
// Workgroups of max(4, WPR) waves.
// ZP: also write, for every group of 128 codes of the row, the zero-point term the large-M GEMM
// kernels take from their workspace: -2^-6 * (sum of the group's E4M3 values) as two fp16 terms,
// laid out as that kernel reads it ([plane][group / 8][M rows][group % 8]; groups up to the next
// multiple of 16 are zero).  Needs K % 128 == 0 and the row in registers.
// PARTS: that many workgroups per row; each searches the whole row and converts and stores every PARTS-th of the chunks
// its threads hold.  For a few rows, which leave the chip idle: the search is a small part of a row's work.
template <int WPR, int CH, bool ZP, bool REREAD, int PARTS>
__global__ __launch_bounds__(WPR > 4 ? 64 * WPR : 256) void fq_quantize_kernel(const uint16_t* __restrict__ X,
                                                                   uint8_t* __restrict__ A,
                                                                   float* __restrict__ a_scale, int K,
                                                                   uint16_t* __restrict__ planes, int M) {
    static_assert(!(ZP && REREAD), "the zero-point terms are summed from registers");
    static_assert(PARTS == 1 || (WPR >= 4 && !ZP && !REREAD), "one row per workgroup, codes only");
    constexpr int WAVES = WPR > 4 ? WPR : 4, ROWS = WAVES / WPR, T = 64 * WPR;
    constexpr int MAXG = T * CH / 16 + 16;           // groups of a row, padded
    __shared__ unsigned red[WAVES];
    __shared__ __attribute__((aligned(16))) uint16_t zrow[ZP ? ROWS : 1][2][ZP ? MAXG : 8];   // [row][plane][group]
    const int row = (int)threadIdx.x / T, t = (int)threadIdx.x % T;
    const int m = PARTS > 1 ? (int)blockIdx.x / PARTS : (int)blockIdx.x * ROWS + row, mine = (int)blockIdx.x % PARTS;
    if (ZP && M <= FQ_KSPLIT_MAX_M) {                     // the arrival counters behind the planes start at zero
        const int G = K >> 7, C2 = 2 * ((G + 15) >> 4);
        unsigned* counters = reinterpret_cast<unsigned*>(planes + (size_t)2 * C2 * M * 8);
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < FQ_KSPLIT_COUNTERS; i += gridDim.x * blockDim.x)
            counters[i] = 0u;
    }
    const bool on = m < M;                                // (rows past M repeat the last one and store nothing)
    const int nchunk = K >> 3;
    const fq_v4i* x = reinterpret_cast<const fq_v4i*>(X + (size_t)(on ? m : M - 1) * K);
    fq_v2i* a = reinterpret_cast<fq_v2i*>(A + (size_t)(on ? m : M - 1) * K);
    fq_v4i keep[CH];
    fq_v2us most = {0, 0};
    if (!REREAD) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {               // all of the thread's chunks are requested before the first is used
            // (past the row's end its last chunk again, which changes no maximum and is not stored: the branch is the
            // same for the whole wave)
            const int c = t + i * T < nchunk ? t + i * T : nchunk - 1;
            keep[i] = (fq_v4i){0, 0, 0, 0};
            if (CH <= 2 || i * T < nchunk) keep[i] = x[c];
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) most = fq_pattern_max(most, keep[i]);
    } else {
        for (int c = t; c < nchunk; c += T) most = fq_pattern_max(most, x[c]);
    }
    // (WPR > 1: a workgroup is one row)
    auto over_row = [&](unsigned v) __attribute__((always_inline)) {
        if (WPR > 1) {
            if ((t & 63) == 0) red[t >> 6] = v;
            __syncthreads();
            v = red[0];
#pragma unroll
            for (int i = 1; i < WPR; ++i) v = red[i] > v ? red[i] : v;
        }
        return v;
    };
    unsigned top = over_row(fq_wave_max(most[0] > most[1] ? most[0] : most[1]));
    const bool nan = top > FQ_BF16_INF;                   // the same for the whole row
    if (nan) {                                            // the largest of the numbers, then
        float amax = 0.f;
        if (!REREAD) {
#pragma unroll
            for (int i = 0; i < CH; ++i) amax = fq_absmax_numbers(amax, keep[i]);
        } else {
            for (int c = t; c < nchunk; c += T) amax = fq_absmax_numbers(amax, x[c]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        if (WPR > 1) __syncthreads();
        top = over_row(__float_as_uint(amax) >> 16);
    }
    const fq_row_scale sc = fq_scale_of(top);
    const float s = sc.s, rcp = sc.rcp;
    if (t == 0 && on && mine == 0) a_scale[m] = s;
    // One choice of quotient per row (s is the same in every thread of a wave): the range the
    // short quotient was checked on, else the full division; straight-line code either way.
    auto convert = [&](auto fast_tag) __attribute__((always_inline)) {
        constexpr bool FAST = decltype(fast_tag)::value;
        if (REREAD) {
            for (int c = t; c < nchunk; c += T) a[c] = fq_quant8<FAST>(x[c], s, rcp);
            return;
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = t + i * T;
            if (PARTS > 1 && i % PARTS != mine) continue;
            if (CH > 2 && i * T >= nchunk) break;         // (the same for the whole wave)
            if (c < nchunk) {
                const fq_v2i o = fq_quant8<FAST>(keep[i], s, rcp);
                if (on) a[c] = o;
                if (ZP) {
                    // a group is 16 consecutive chunks = 16 consecutive lanes (nchunk is a multiple of 16,
                    // so a group's lanes are all here or all absent)
                    float z = fq_sum8(o);
                    z = fq_dpp_add<0xB1>(z);              // pairs, quads, eights, sixteens
                    z = fq_dpp_add<0x4E>(z);
                    z = fq_dpp_add<0x141>(z);
                    z = fq_dpp_add<0x140>(z);
                    if ((t & 15) == 0) {
                        z *= -0.015625f;
                        const _Float16 hi = (_Float16)z;                  // round to nearest even
                        const _Float16 lo = (_Float16)(z - (float)hi);    // the difference is exact in FP32
                        zrow[row][0][c >> 4] = __builtin_bit_cast(uint16_t, hi);
                        zrow[row][1][c >> 4] = __builtin_bit_cast(uint16_t, lo);
                    }
                }
            }
        }
    };
    if (__builtin_amdgcn_readfirstlane((int)(sc.fast && !nan))) convert(std::true_type());
    else convert(std::false_type());
    if (ZP) {
        // padding groups are zero; then one 16-byte store per (plane, 8 groups) of a row, rows of a workgroup side by side
        const int G = K >> 7, C2 = 2 * ((G + 15) >> 4);
        for (int g = G + t; g < 8 * C2; g += T) zrow[row][0][g] = zrow[row][1][g] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * C2 * ROWS; i += 64 * WAVES) {
            const int r = i % ROWS, pu = i / ROWS, plane = pu / C2, unit = pu - plane * C2, mm = blockIdx.x * ROWS + r;
            if (mm < M)
                *reinterpret_cast<fq_v4i*>(planes + (((size_t)plane * C2 + unit) * M + mm) * 8) =
                    *reinterpret_cast<const fq_v4i*>(&zrow[r][plane][8 * unit]);
        }
    }
}

namespace {

// Waves per row and chunks per thread: few rows take many waves with two chunks each (a row's latency is all there is); many
// rows fewer waves with more (other rows hide the latency, fewer waves meet at a barrier), as long as the last chunk of every
// thread is not mostly empty.  Inputs in turn from 600 MB, replayed from graphs, us without / with zero-point terms, the choice here first:
//     1536 x 1024   <4, 2> 3.4 / 3.9; <1, 4> 3.1 / 3.6      1600 x 1024   <1, 4> 3.1 / 3.6; <4, 2> 3.4 / 4.0
//     1536 x 2048   <4, 2> 4.0 / 4.5; <1, 4> 4.1 / 4.7      2048 x 2048   <1, 4> 4.7 / 5.3; <4, 2> 4.6 / 5.3
//     512 x 4224    <8, 2> 3.5 / 4.1; <4, 3> 3.6 / 4.2      640 x 4224    <4, 3> 3.9 / 4.5; <8, 2> 3.9 / 4.7
//     2048 x 4224   <4, 3> 7.1 / 8.1; <8, 2> 7.6 / 8.8      5120 x 6144   <4, 3> 16.3 / 17.6; <8, 2> 17.0 / 18.8
//     2048 x 8192   <8, 2> 10.6 / 11.6; <4, 8> 10.3 / 11.9  8192 x 8192   <8, 2> 31.8 / 33.6; <4, 8> 31.9 / 33.6
//     256 x 8320    <16, 2> 3.4 / 4.0; <4, 6> 3.7 / 4.4     400 x 8320    <4, 6> 4.5 / 5.3; <16, 2> 4.5 / 5.2
//     1536 x 8320   <4, 6> 9.2 / 10.4; <8, 4> 9.4 / 10.3    1024 x 9600   <4, 6> 7.8 / 8.8; <8, 4> 7.5 / 8.6
//     400 x 11008   <16, 2> 5.3 / 6.0; <8, 4> 5.3 / 6.1     1024 x 11008  <8, 4> 8.3 / 9.5; <16, 2> 8.8 / 10.1
//     512 x 16384   <16, 2> 7.0 / 8.1; <8, 4> 7.1 / 8.1     4096 x 16384  <8, 4> 31.9 / 33.9; <16, 2> 33.3 / 34.7
//     1024 x 16512  <16, 4> 11.6; <16, 8> 11.9              2048 x 32768  <16, 4> 33.9; <16, 8> 34.1
//     512 x 40960   <16, 8> 12.9; rows read twice by 16 waves 16.6.  Longer rows do not fit and are read twice.
template <bool ZP>
void fq_launch_quantize_as(const uint16_t* X, uint8_t* A, float* a_scale, int M, int K, uint16_t* planes, hipStream_t stream) {
#define FQ_QUANTIZE_IN(WPR_, CH_, REREAD_, PARTS_) \
    hipLaunchKernelGGL((fq_quantize_kernel<WPR_, CH_, ZP, REREAD_, PARTS_>), \
                       dim3((unsigned)((M + (WPR_ > 4 ? 1 : 4 / WPR_) - 1) / (WPR_ > 4 ? 1 : 4 / WPR_) * PARTS_)), \
                       dim3(WPR_ > 4 ? 64 * WPR_ : 256), 0, stream, X, A, a_scale, K, planes, M)
#define FQ_QUANTIZE(WPR_, CH_, REREAD_) FQ_QUANTIZE_IN(WPR_, CH_, REREAD_, 1)
    if constexpr (!ZP) {
        // few rows: two workgroups each, unless the second half of the chunks is empty.  One / two per row, us, inputs in turn | the same input
        // again | a copy that writes the input, then the quantiser: 1 x 4096 1.76 / 1.72 | 1.74 / 1.63 | 3.31 / 3.32, 16 x 4096 2.03 / 2.20 | 1.99 /
        // 1.84 | 3.61 / 3.81, 16 x 8192 2.53 / 2.40 | 2.20 / 2.00 | 4.11 / 3.85, 64 x 8192 2.63 / 2.66 | 2.26 / 2.14 | 4.32 / 4.29, 16 x 14336 2.84 / 2.69 |
        // 2.50 / 2.25 | 4.37 / 4.24, 64 x 14336 3.42 / 3.34 | 2.60 / 2.38 | 5.11 / 5.46; in turn 128 x 8192 2.93 / 3.14, 128 x 16384 3.59 / 3.94, 64 x 32016
        // 4.34 / 4.44
        if (M <= 64 && K > 2048 && K <= 4 * 4096) {
            if (K <= 4096) FQ_QUANTIZE_IN(4, 2, false, 2);
            else if (K <= 2 * 4096) FQ_QUANTIZE_IN(8, 2, false, 2);
            else FQ_QUANTIZE_IN(16, 2, false, 2);
            return;
        }
        // A thread holds three or four chunks: four workgroups where the fourth has some of them, or up to 16 rows where the third is
        // nearly whole, else two.  Two / four, us, inputs in turn from 600 MB | a copy that writes the input, then the quantiser: 32 x 32016
        // 4.52 / 4.33 | 6.68 / 7.15, 24 x 32016 4.37 / 4.14 | 6.31 / 6.53, 16 x 32016 3.67 / 3.49 | 5.94 / 5.90, 8 x 32016 3.62 / 3.36 | 5.54 /
        // 5.41 (the same 32 x 32016 again and again 3.38 / 3.13); 1 x 24576 3.11 / 2.86 | 4.82 / 4.65, 8 x 22528 3.17 / 3.15 | 4.88 / 4.83;
        // on the other side 24 x 24576 3.35 / 3.56 | 5.54 / 5.95, 32 x 24576 4.04 / 3.96 | 5.85 / 6.41, 16 x 20480 3.17 / 3.23 | 5.03 / 5.19
        if (M <= 32 && K > 4 * 4096 && K <= 8 * 4096) {
            if (K > 6 * 4096 || (M <= 16 && K > 22528)) FQ_QUANTIZE_IN(16, 4, false, 4);
            else FQ_QUANTIZE_IN(16, 4, false, 2);
            return;
        }
    }
    if (K > 4 * 4096) {
        if constexpr (!ZP) {                              // (no zero-point terms for rows this long)
            if (K > 16 * 4096) FQ_QUANTIZE(16, 8, true);
            else if (K > 8 * 4096) FQ_QUANTIZE(16, 8, false);
            else FQ_QUANTIZE(16, 4, false);
        }
    } else if (K > 10240) { if (M <= 512) FQ_QUANTIZE(16, 2, false); else FQ_QUANTIZE(8, 4, false); }
    else if (K > 2 * 4096) { if (M <= 256) FQ_QUANTIZE(16, 2, false); else FQ_QUANTIZE(4, 6, false); }
    else if (K > 6144 || (K > 4096 && M <= 512)) FQ_QUANTIZE(8, 2, false);
    else if (K > 4096) FQ_QUANTIZE(4, 3, false);
    else if (K > 2048 || M <= 1536) FQ_QUANTIZE(4, 2, false);
    else FQ_QUANTIZE(1, 4, false);
#undef FQ_QUANTIZE
#undef FQ_QUANTIZE_IN
}

}  // namespace

void fq_launch_quantize(const uint16_t* X, uint8_t* A, float* a_scale, int M, int K, hipStream_t stream) {
    fq_launch_quantize_as<false>(X, A, a_scale, M, K, nullptr, stream);
}

bool fq_quantize_can_write_zero_point(int K) { return (K % FQ_GROUP) == 0 && K <= 16384; }

void fq_launch_quantize_zp(const uint16_t* X, uint8_t* A, float* a_scale, int M, int K, void* workspace,
                           hipStream_t stream) {
    fq_launch_quantize_as<true>(X, A, a_scale, M, K, static_cast<uint16_t*>(workspace), stream);
}
