// Offline weight quantisation: the step that produces the GEMM's weight operands from a bf16 matrix
// W [N,K] (output channel n, input channel k; Y = X W^T).
//
//   channel-wise absmean scaling (Sec. 3.1.2, Def. 3.1)   lambda[k] = target / mean_n |W[n,k]|
//   per-tensor scaling (Def. 3.2, App. C.1)                delta = 2^n, n the smallest non-negative integer
//       for which the cumulative underflow S(W * 2^n) has reached its final value, or an element lies in
//       7 * 2^(5-n) <= |w| < 7 * 2^(6-n)
//   group-wise INT4 with an FP8 scale (Sec. 2.1 eq. 1, Sec. 3.1; App. B Lemma B.1)
//       sigma = max_group |v| / 7,  sigma8 = E4M3(sigma),  q = clamp(round(v / sigma8), -8, 7)
//
// Everywhere the weight that is worked on is v = fp32(W[n,k] * lambda[k]) (lambda may be absent),
// and the quantiser multiplies it by 2^n (exact).
#include "fq_common.h"
#include "fq_kernels.h"

namespace {

__device__ __forceinline__ float fqw_bf16(unsigned short b) { return __uint_as_float((unsigned)b << 16); }

// floor(log2(v / 7)) of a positive finite FP32 number given by its bits: v = 1.m * 2^E lies at or
// above 7 * 2^(E-2) = 1.75 * 2^E exactly when its fraction is at least 0.75.
__device__ __forceinline__ int fqw_log2_over_7(unsigned bits) {
    int e = (int)(bits >> 23);
    unsigned frac = bits & 0x7FFFFFu;
    if (e == 0) {                                         // subnormal: normalise by hand
        const int p = 31 - __builtin_clz(frac);           // frac != 0 for a positive number
        e = p - 22;                                       // value = frac * 2^-149 = 1.x * 2^(p-149); biased: p - 149 + 127
        frac = (frac << (23 - p)) & 0x7FFFFFu;
    }
    const int E = e - 127;
    return frac >= 0x600000u ? E - 2 : E - 3;
}

// Consecutive bands of `step` rows of W, one 16-byte load per lane each (`lane_off`: the lane's bytes inside a band): a wave
// keeps a ring of them in flight and asks for the next band as soon as it has used one, so that the reading never
// pauses (workgroups that fetch a batch, work on it and fetch the next do so in step, and the memory idles in between:
// 11008 x 4096 channel means from memory 40.2 us in batches, 38.1 as a ring).  Rows past N lie behind the descriptor's range and
// read as zeros.
struct fqw_bands {
    const uint16_t* p;
    long long left;                                       // bytes from p to the end of W
    long long band;                                       // bytes of a band
    __device__ __forceinline__ fqw_bands(const uint16_t* W, int N, int K, int k0, int step)
        : p(W + k0), left(((long long)N * K - k0) * 2), band((long long)step * K * 2) {}
    template <int POLICY = 0>                             // cache policy of the load (2: nontemporal)
    __device__ __forceinline__ fq_v4i next(unsigned lane_off) {
        const long long n = left < 0 ? 0 : left < 0xFFFFFF00ll ? left : 0xFFFFFF00ll;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, (int)(unsigned)n, 0x00020000);
        p += band / 2;
        left -= band;
        return __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, lane_off, 0, POLICY));
    }
};
#define FQW_OOB 0xFFFFFFF0u                               // an offset behind any range

}  // namespace

// ---- channel-wise absmean scaling ------------------------------------------------------------------
// FP64 sums over the rows of a channel, combined in a fixed order: the result does not depend on timing.  A column sum
// stays inside one workgroup here; fq_cas_partial_kernel below shares it out, where the caller has given scratch for the parts.
//
// Any W: 16 waves per 32 input channels; 16 lanes cover the 32 channels of a row (a dword = two channels each), so a
// wave reads 4 rows per instruction and the 16 waves 64; FQW_CAS_UNROLL such loads are in flight per lane.
#define FQW_CAS_UNROLL 16
#define FQW_CAS_THREADS 1024
#define FQW_CAS_LPR 16                                    // lanes per row
__global__ __launch_bounds__(FQW_CAS_THREADS) void fq_cas_scales_kernel(const uint16_t* __restrict__ W, float target,
                                                            float* __restrict__ lambda, int N, int K) {
    constexpr int FQW_CAS_ROWS = FQW_CAS_THREADS / FQW_CAS_LPR, CH = 2 * FQW_CAS_LPR;
    __shared__ double part[FQW_CAS_ROWS][CH];
    const int sub = threadIdx.x / FQW_CAS_LPR;            // which of the rows of a pass
    const int k = blockIdx.x * CH + 2 * (threadIdx.x % FQW_CAS_LPR);
    const bool two = k + 1 < K, one = k < K;              // K may be odd: the last channel then loads 2 bytes
    double s0 = 0.0, s1 = 0.0;
    for (int n0 = sub; n0 < N; n0 += FQW_CAS_ROWS * FQW_CAS_UNROLL) {
        unsigned w[FQW_CAS_UNROLL];
#pragma unroll
        for (int u = 0; u < FQW_CAS_UNROLL; ++u) {
            const int n = n0 + FQW_CAS_ROWS * u;
            w[u] = 0u;
            if (n < N && one) {
                const uint16_t* src = W + (size_t)n * K + k;
                // a dword load needs 4-byte alignment, which an odd row length breaks on every other row
                if (two && ((reinterpret_cast<uintptr_t>(src) & 3u) == 0)) w[u] = *reinterpret_cast<const unsigned*>(src);
                else w[u] = (unsigned)src[0] | (two ? (unsigned)src[1] << 16 : 0u);
            }
        }
#pragma unroll
        for (int u = 0; u < FQW_CAS_UNROLL; ++u) {
            s0 += (double)fabsf(fqw_bf16((unsigned short)(w[u] & 0xFFFFu)));
            s1 += (double)fabsf(fqw_bf16((unsigned short)(w[u] >> 16)));
        }
    }
    part[sub][2 * (threadIdx.x % FQW_CAS_LPR)] = s0;
    part[sub][2 * (threadIdx.x % FQW_CAS_LPR) + 1] = s1;
    __syncthreads();
    if (threadIdx.x < CH && blockIdx.x * CH + (int)threadIdx.x < K) {
        double t = 0.0;
#pragma unroll 16
        for (int r = 0; r < FQW_CAS_ROWS; ++r) t += part[r][threadIdx.x];
        lambda[blockIdx.x * CH + threadIdx.x] =
            t == 0.0 ? 1.0f : (float)((double)target / (t / (double)N));            // an all-zero channel keeps 1
    }
}

// Rows in 16-byte steps (K a multiple of 8, W 16-byte aligned; every weight matrix): 8 * LPR channels per workgroup, LPR
// lanes x 16 bytes per row, 64 / LPR rows per wave-level load, FQW_CASW_UNROLL of them in flight per lane.  With fewer
// than 8 lanes per row several workgroups read every 128-byte line; they are given neighbouring turns on one XCD (workgroup
// b runs on XCD b % 8), so that its L2 fetches the line once (on different XCDs the memory side moved the matrix twice
// or four times, which used to cap this at 32 channels).  |bf16| becomes FP64 by its bits alone: shifted to the top of
// the double's exponent and fraction it is the value times 2^-896, subnormals included (the double is subnormal
// then, in the same steps), so an element costs two integer instructions and an FP64 addition, no conversion; all sums
// carry that factor, which comes off exactly at the end.  Infinities and NaN go in as finite numbers of 2^128 and more that way:
// a channel with a sum from there on is read once more for them (so that finite weights pay nothing for it), and its sum
// becomes an infinity or a NaN, as FP64 addition would have made it.
#define FQW_CASW_UNROLL 8
#define FQW_CASW_THREADS 1024
template <int CTRL>
__device__ __forceinline__ double fqw_dpp_f64(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ void fqw_cas_add(double (&s)[8], const fq_v4i& v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned word = (unsigned)v[i];
        s[2 * i] += __hiloint2double((int)((word << 13) & 0x0FFFE000u), 0);
        s[2 * i + 1] += __hiloint2double((int)((word >> 3) & 0x0FFFE000u), 0);
    }
}

// A channel's sum (times 2^-896) -> its scale, by one wave that holds channel k0 + lane in lane `lane`.
__device__ __forceinline__ void fqw_cas_close(double t, bool mine, const uint16_t* __restrict__ W, float target,
                                              float* __restrict__ lambda, int k0, int lane, int N, int K) {
    t *= 0x1p+896;
    for (unsigned long long big = __ballot(mine && t >= 0x1p+128); big != 0; big &= big - 1) {
        const int c = __ffsll(big) - 1;
        bool inf = false, nan = false;
        for (int n = lane; n < N; n += 64) {
            const unsigned b = W[(size_t)n * K + k0 + c] & 0x7FFFu;
            inf |= b == 0x7F80u;
            nan |= b > 0x7F80u;
        }
        const bool any_inf = __ballot(inf) != 0, any_nan = __ballot(nan) != 0;
        if (lane == c) t = any_nan ? __builtin_nan("") : any_inf ? __builtin_inf() : t;
    }
    if (mine)
        lambda[k0 + lane] =
            t == 0.0 ? 1.0f : (float)((double)target / (t / (double)N));            // an all-zero channel keeps 1
}

template <int LPR, bool STREAM>
__global__ __launch_bounds__(FQW_CASW_THREADS) void fq_cas_scales_wide_kernel(const uint16_t* __restrict__ W, float target,
                                                                              float* __restrict__ lambda, int N, int K) {
    constexpr int ROWS = FQW_CASW_THREADS / LPR, CH = 8 * LPR, SHARE = 8 / LPR;
    __shared__ double part[64][CH];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = threadIdx.x / LPR;                    // which of the rows of a pass
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int k0 = ((j / SHARE) * 8 + x) * 64 + (j % SHARE) * CH;
    const int k = k0 + 8 * (lane % LPR);
    if (k0 >= K) return;
    const bool on = k < K;                                // (K % 8 == 0: the 8 channels are inside or outside together)
    double s[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = 0.0;
    fq_v4i w[FQW_CASW_UNROLL];
    if constexpr (LPR == 8) {
        // Whole lines per workgroup and a long row stride: all workgroups fetch a batch of bands at a time, which keeps them on
        // the same rows of W.  The ring below lets them drift apart, and memory then serves rows 22 to 57 KB apart at random:
        // 11008 x 22016 115 us in batches, 133 as a ring; 4096 x 11008, from memory, 20.5 -> 21.2 -> 21.9 (nontemporal batches,
        // these, ring), where the cached lines save the next pass over W more.
        for (int n0 = sub; n0 < N; n0 += ROWS * FQW_CASW_UNROLL) {
#pragma unroll
            for (int u = 0; u < FQW_CASW_UNROLL; ++u) {
                const int n = n0 + ROWS * u;
                w[u] = (fq_v4i){0, 0, 0, 0};
                if (n < N && on) {
                    const fq_v4i* src = reinterpret_cast<const fq_v4i*>(W + (size_t)n * K + k);
                    w[u] = STREAM ? __builtin_nontemporal_load(src) : *src;
                }
            }
#pragma unroll
            for (int u = 0; u < FQW_CASW_UNROLL; ++u) fqw_cas_add(s, w[u]);
        }
    } else {
        fqw_bands bands(W, N, K, k0, ROWS);
        const unsigned lane_off = on ? (unsigned)sub * (unsigned)K * 2u + 16u * (threadIdx.x % LPR) : FQW_OOB;
#pragma unroll
        for (int u = 0; u < FQW_CASW_UNROLL; ++u) w[u] = bands.next(lane_off);
        // A round of bands with rows in at most half of them (a small matrix has no other) is finished band by band, without the
        // work on the rest: 1024 x 1024 5.7 -> 4.0 us, 6000 x 1536 12.9 -> 12.0, 22016 x 1024 46.6 -> 42.2; a fuller one gains nothing by
        // it (11008 x 4096, from memory, 5.5 of 8 bands left: 37.5 us as a whole round, 38.0 band by band).
        int n0 = 0;
        for (; n0 + ROWS * FQW_CASW_UNROLL / 2 < N; n0 += ROWS * FQW_CASW_UNROLL) {
#pragma unroll
            for (int u = 0; u < FQW_CASW_UNROLL; ++u) {
                fqw_cas_add(s, w[u]);
                w[u] = bands.next(lane_off);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int u = 0; u < FQW_CASW_UNROLL / 2; ++u)
            if (n0 + ROWS * u < N) fqw_cas_add(s, w[u]);
    }
    // the rows of a wave are added inside its four 16-lane rows by rotations (lanes LPR apart hold the same channels; DPP:
    // shuffles through LDS took 3 us), the rest through LDS, all in a fixed order
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (LPR <= 2) s[i] += fqw_dpp_f64<0x4E>(s[i]);    // quad_perm [2,3,0,1]
        if (LPR <= 4) s[i] += fqw_dpp_f64<0x124>(s[i]);   // row_ror:4
        s[i] += fqw_dpp_f64<0x128>(s[i]);                 // row_ror:8
    }
    if ((lane & 15) < LPR) {
#pragma unroll
        for (int i = 0; i < 8; ++i) part[4 * wave + (lane >> 4)][8 * (lane & 15) + i] = s[i];
    }
    __syncthreads();
    if (wave != 0) return;
    const bool mine = lane < CH && k0 + lane < K;         // (CH <= 64: the channels' sums are lanes of the first wave)
    double t = 0.0;
    if (mine) {
#pragma unroll 16
        for (int r = 0; r < 64; ++r) t += part[r][lane];
    }
    fqw_cas_close(t, mine, W, target, lambda, k0, lane, N, K);
}

// The same with scratch, for large matrices: a workgroup sums a share of the rows of a slab of up to 512 channels (`cw` 16-byte
// columns, the slabs as even as they can be) and leaves its FP64 sums in part[share][K]; a second kernel adds the shares in their
// order.  A wave reads up to 1 KiB of a row at once, where the kernels above, whose workgroups each need all rows of their
// channels, read 32 to 128 bytes of a row, at a third of the memory's rate.  Read nontemporally: W comes from memory once, and what
// it would push out of the last-level cache has to be written back if it was written lately (11008 x 4096 after a kernel
// that wrote 320 MB: 38.5 us through the cache, 22.0 past it, 47.2 for the kernel above; all four calls of the quantiser
// in a row 82 us either way).  Back to back from memory, the kernel above and both launches here: 11008 x 4096 38.0 -> 19.9 us, 22016 x
// 4096 74.8 -> 33.3.
#define FQW_CASP_UNROLL 8
__global__ __launch_bounds__(FQW_CASW_THREADS) void fq_cas_partial_kernel(const uint16_t* __restrict__ W, double* __restrict__ part,
                                                                          int N, int K, int slabs, int cw, int rows) {
    __shared__ double red[8][FQW_CASW_THREADS];
    const int slab = blockIdx.x % slabs, share = blockIdx.x / slabs;
    const int r0 = share * rows, left = N - r0 < rows ? N - r0 : rows;
    const int c0 = slab * cw, cols = K / 8 - c0 < cw ? K / 8 - c0 : cw;      // this slab's columns
    const int par = FQW_CASW_THREADS / cw;                // rows side by side
    const int r = threadIdx.x / cw, c = threadIdx.x % cw;
    double s[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = 0.0;
    fqw_bands bands(W + (size_t)r0 * K, left, K, 8 * c0, par);
    const unsigned lane_off = r < par && c < cols ? (unsigned)r * (unsigned)K * 2u + 16u * (unsigned)c : FQW_OOB;
    fq_v4i w[FQW_CASP_UNROLL];
#pragma unroll
    for (int u = 0; u < FQW_CASP_UNROLL; ++u) w[u] = bands.next<2>(lane_off);
    int n0 = 0;
    for (; n0 + par * FQW_CASP_UNROLL <= left; n0 += par * FQW_CASP_UNROLL) {
#pragma unroll
        for (int u = 0; u < FQW_CASP_UNROLL; ++u) {
            fqw_cas_add(s, w[u]);
            w[u] = bands.next<2>(lane_off);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int u = 0; u < FQW_CASP_UNROLL; ++u)             // the bands left that hold rows
        if (n0 + par * u < left) fqw_cas_add(s, w[u]);
#pragma unroll
    for (int i = 0; i < 8; ++i) red[i][threadIdx.x] = s[i];
    __syncthreads();
    for (int j = threadIdx.x; j < 8 * cols; j += FQW_CASW_THREADS) {
        const int i = j & 7, col = j >> 3;
        double t = 0.0;
        for (int q = 0; q < par; ++q) t += red[i][q * cw + col];
        part[(size_t)share * K + 8 * c0 + j] = t;
    }
}

__global__ __launch_bounds__(256) void fq_cas_fold_kernel(const double* __restrict__ part, const uint16_t* __restrict__ W,
                                                          float target, float* __restrict__ lambda, int N, int K, int shares) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, k0 = blockIdx.x * 64;
    const bool mine = k0 + lane < K;
    double t = 0.0;
    if (mine) {
#pragma unroll 8
        for (int s = wave; s < shares; s += 4) t += part[(size_t)s * K + k0 + lane];
    }
    red[wave][lane] = t;
    __syncthreads();
    if (wave != 0) return;
    t = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    fqw_cas_close(t, mine, W, target, lambda, k0, lane, N, K);
}

// ---- per-tensor scaling: statistics, then the choice of n --------------------------------------------
// stats[0]: bits of the smallest non-zero |v| (0xFFFFFFFF: none); stats[1]: bits of the largest |v| below
// 7 * 2^6 (0: none) -- the bands of condition 2 are ordered by magnitude, so the lowest band n >= 0 that holds an
// element is the band of that element.
#define FQW_BAND0_END 0x43E00000u                         // bits of 448 = 7 * 2^6: at or above it the band index is negative
__global__ void fq_pts_init_kernel(unsigned* __restrict__ stats) {
    if (threadIdx.x < 8) stats[threadIdx.x] = threadIdx.x == 0 ? 0xFFFFFFFFu : 0u;
}

// Condition 1 holds from the n at which the smallest non-zero element reaches 7 * 2^-9 (then no
// non-zero element adds to S any more, and zeros add the same for every n); condition 2 at the
// lowest band that holds an element.  n is the smaller of the two, at most 126.
__device__ __forceinline__ int fqw_pts_resolve(unsigned vmin, unsigned vmax) {
    int n1 = 0;
    if (vmin != 0xFFFFFFFFu) {
        n1 = -9 - fqw_log2_over_7(vmin);
        n1 = n1 < 0 ? 0 : n1;
    }
    int n2 = 127;
    if (vmax != 0u) {
        n2 = 5 - fqw_log2_over_7(vmax);                   // >= 0 by the choice of vmax
        n2 = n2 > 126 ? 127 : n2;
    }
    const int n = n1 < n2 ? n1 : n2;
    return n > 126 ? 126 : n;
}

// Thread t works on the 16-byte chunk (8 weights) t % (K / 8) of the rows t / (K / 8), + rows_par, ...: its 8
// input channels never change, so their lambda sit in registers, and neighbouring threads read neighbouring
// chunks.  FQW_PTS_UNROLL rows are in flight per thread.  One workgroup per compute unit: they all end together
// and close with two atomics each, which queue up (11008 x 4096, all three launches: 24.8 us with 256 workgroups of
// 1024 threads, 29.0 with 512 of 512, 43.9 with 1024 of 256; counting the workgroups in, so that the last one resolves n
// and the third launch goes, cost 12 us more than that launch; 37 us with 512 workgroups that fetch four rows at a time).
// PARTS, with scratch: a pair of statistics per workgroup and a kernel that folds them, without the launch that presets the
// statistics and without atomics (without | with scratch: 1024 x 1024 13.0 | 8.6 us, 4096 x 4096 18.4 | 11.7, 11008 x 4096 24.2 | 20.6,
// 22016 x 11008 77.6 | 76.3).
// A small matrix (at most 32 such workgroups) takes workgroups of 256, which start and fold sooner; STREAM: a matrix
// larger than the last-level cache is read nontemporally (fq_launch_pts_exponent has the figures).
#define FQW_PTS_UNROLL 6
#define FQW_PTS_THREADS 1024
#define FQW_PTS_WGS 256
template <int THREADS, bool STREAM, bool PARTS>
__global__ __launch_bounds__(THREADS) void fq_pts_stats_kernel(const uint16_t* __restrict__ W,
                                                           const float* __restrict__ lambda,
                                                           unsigned* __restrict__ stats,
                                                           int N, int K, int rows_par) {
    __shared__ unsigned red[THREADS / 64][2];
    unsigned vmin = 0xFFFFFFFFu, vmax = 0u;               // vmin: the smallest non-zero pattern minus 1
    const int KC = K / 8;
    const unsigned t = blockIdx.x * (unsigned)THREADS + threadIdx.x;
    const int r0 = (int)(t / (unsigned)KC), cc = (int)(t % (unsigned)KC);
    float lam[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) lam[i] = lambda ? lambda[8 * cc + i] : 1.0f;
    fqw_bands bands(W, N, K, 0, rows_par);
    const unsigned lane_off = r0 < rows_par ? (unsigned)r0 * (unsigned)K * 2u + 16u * (unsigned)cc : FQW_OOB;
    fq_v4i w[FQW_PTS_UNROLL];
#pragma unroll
    for (int u = 0; u < FQW_PTS_UNROLL; ++u) w[u] = bands.template next<STREAM ? 2 : 0>(lane_off);
    const auto look = [&](const fq_v4i& x) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const unsigned word = (unsigned)x[i >> 1];
            float v = __uint_as_float((i & 1) ? (word & 0xFFFF0000u) : (word << 16));
            v *= lam[i];                                  // (exact where there is no lambda)
            const unsigned b = __float_as_uint(v) & 0x7FFFFFFFu;
            vmin = b - 1u < vmin ? b - 1u : vmin;         // (a zero wraps to the largest number)
            const unsigned below = b < FQW_BAND0_END ? b : 0u;
            vmax = below > vmax ? below : vmax;
        }
    };
    // (the last round band by band: bands without rows cost their work otherwise, 1024 x 1024 14.1 -> 12.9 us, 11008 x 4096 26.1
    // -> 25.1, all three launches)
    long long n0 = 0;
    for (; n0 + (long long)FQW_PTS_UNROLL * rows_par <= N; n0 += (long long)FQW_PTS_UNROLL * rows_par) {
#pragma unroll
        for (int u = 0; u < FQW_PTS_UNROLL; ++u) {
            look(w[u]);
            w[u] = bands.template next<STREAM ? 2 : 0>(lane_off);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int u = 0; u < FQW_PTS_UNROLL; ++u)              // the bands left that hold rows
        if (n0 + (long long)u * rows_par < N) look(w[u]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned lo = (unsigned)__shfl_xor((int)vmin, o, 64), hi = (unsigned)__shfl_xor((int)vmax, o, 64);
        vmin = lo < vmin ? lo : vmin;
        vmax = hi > vmax ? hi : vmax;
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6][0] = vmin;
        red[threadIdx.x >> 6][1] = vmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned m0 = red[0][0], m1 = red[0][1];
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) {
            m0 = red[w][0] < m0 ? red[w][0] : m0;
            m1 = red[w][1] > m1 ? red[w][1] : m1;
        }
        if (m0 != 0xFFFFFFFFu) m0 += 1u;
        if (PARTS) {                                      // stats: a pair per workgroup, folded by the next kernel
            *reinterpret_cast<uint2*>(stats + 2 * blockIdx.x) = make_uint2(m0, m1);
            return;
        }
        // only the atomics that would change a statistic (the plain reads may be stale: that costs at most an
        // atomic that changes nothing)
        const volatile unsigned* seen = stats;
        if (m0 < seen[0]) atomicMin(&stats[0], m0);
        if (m1 > seen[1]) atomicMax(&stats[1], m1);
    }
}

__global__ void fq_pts_resolve_kernel(const unsigned* __restrict__ stats, int* __restrict__ n_out) {
    if (threadIdx.x == 0) n_out[0] = fqw_pts_resolve(stats[0], stats[1]);
}

// The workgroups' pairs, at most FQW_PTS_WGS of them, one per thread.
__global__ __launch_bounds__(FQW_PTS_WGS) void fq_pts_fold_kernel(const unsigned* __restrict__ parts, int count, int* __restrict__ n_out) {
    __shared__ unsigned red[FQW_PTS_WGS / 64][2];
    uint2 v = make_uint2(0xFFFFFFFFu, 0u);
    if ((int)threadIdx.x < count) v = *reinterpret_cast<const uint2*>(parts + 2 * threadIdx.x);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned lo = (unsigned)__shfl_xor((int)v.x, o, 64), hi = (unsigned)__shfl_xor((int)v.y, o, 64);
        v.x = lo < v.x ? lo : v.x;
        v.y = hi > v.y ? hi : v.y;
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6][0] = v.x;
        red[threadIdx.x >> 6][1] = v.y;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned m0 = red[0][0], m1 = red[0][1];
#pragma unroll
        for (int w = 1; w < FQW_PTS_WGS / 64; ++w) {
            m0 = red[w][0] < m0 ? red[w][0] : m0;
            m1 = red[w][1] > m1 ? red[w][1] : m1;
        }
        n_out[0] = fqw_pts_resolve(m0, m1);
    }
}

// ---- group-wise INT4 quantisation ------------------------------------------------------------------
// 16 lanes per group of 128 weights (8 neighbouring weights = 16 bytes per lane); a thread quantises the same 8 columns of ROWS
// neighbouring rows, all of them requested before the first is worked on, so that it finds its place and fetches its lambda
// once.  3 bytes per weight, but a vector instruction per weight takes 1.1 us at 11008 x 4096, and some 22 of them (the place by
// a 64-bit modulo and lambda per row, two IEEE divisions per lane, the maximum through LDS, separate rounding, conversion and
// packing) held the reading back; with 13 it runs at 5.0 to 5.8 TB/s (from memory, us, before -> now: 11008 x 4096 33.4 -> 26.8, 4096 x 4096
// 15.5 -> 12.3, 22016 x 8192 115 -> 94, 4096 x 11008 34.0 -> 27.2, 2048 x 1024 3.6 -> 3.2; four rows per thread are even, nontemporal loads too).
// The quotient: with r = the correctly rounded 1 / sigma8, q0 = v * r, the exact residual e = fma(-q0, sigma8, v) and
// q1 = fma(e, r, q0), rint(q1) equals rint of the IEEE quotient for every FP32 v and every E4M3 sigma8 (a program on
// the host has gone through all of them, the tests go through every third v; sigma8 has four significant bits, and a power
// of two moves nothing).  The same steps by 1/7 give sigma (all significands checked there too), and r itself is the
// hardware's reciprocal after one step of Newton's: 1 / sigma8 is periodic in at most 12 bits, so never near a midpoint.
// A group whose largest weight times 2^n is infinite, or with sigma8 = 0, is cut to +-16 sigma8 first, which changes no code of a finite weight (they end
// at -8 and 7) and keeps the residual finite (with sigma8 = 0 every code is 0).  rint and the conversion are one addition:
// q1 cut to [-8, 7], plus 1.5 * 2^23, has the code in its low byte.
// 2^n multiplies sigma and divides sigma8 instead of every weight, up to 2^64, where every step stays exact (the smallest
// weights that matter are 2^-75 then, their residuals' last bits above 2^-130); beyond, the weights are multiplied.
#define FQW_MANY_PTS 64
template <int CTRL>
__device__ __forceinline__ float fqw_dpp_max(float v) {
    return fmaxf(v, __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, false)));
}

template <int ROWS>
__global__ __launch_bounds__(256) void fq_quantize_weights_kernel(const uint16_t* __restrict__ W,
                                                                  const float* __restrict__ lambda, int n_pts,
                                                                  int sigma_rne, int8_t* __restrict__ q,
                                                                  uint8_t* __restrict__ gs, int N, int K) {
    const unsigned KC = (unsigned)K / 8u, t = blockIdx.x * 256u + threadIdx.x, set = t / KC, cc = t - set * KC;
    const size_t row0 = (size_t)set * ROWS;
    if (row0 >= (size_t)N) return;                        // (K is a multiple of 128: the 16 lanes of a group stay together)
    const float p2n = __uint_as_float((unsigned)(n_pts + 127) << 23);    // 2^n, 0 <= n <= 126
    const bool many = n_pts > FQW_MANY_PTS;
    const float back = many ? 1.0f : __uint_as_float((unsigned)(127 - n_pts) << 23), up = many ? 1.0f : p2n;
    fq_v4i w[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const size_t row = row0 + u < (size_t)N ? row0 + u : (size_t)N - 1;   // (past the end: repeated, not stored)
        w[u] = *reinterpret_cast<const fq_v4i*>(W + row * (size_t)K + 8u * cc);
    }
    fq_v4f l0 = {1.f, 1.f, 1.f, 1.f}, l1 = l0;
    if (lambda) {
        l0 = *reinterpret_cast<const fq_v4f*>(lambda + 8u * cc);
        l1 = *reinterpret_cast<const fq_v4f*>(lambda + 8u * cc + 4);
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const unsigned word = (unsigned)w[u][i >> 1];
            v[i] = __uint_as_float((i & 1) ? (word & 0xFFFF0000u) : (word << 16)) * (i < 4 ? l0[i & 3] : l1[i & 3]);
        }
        if (many) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] *= p2n;
        }
        float vmax = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) vmax = fmaxf(vmax, fabsf(v[i]));
        // over the group's 16 lanes: pairs, quads, eights, sixteens
        vmax = fqw_dpp_max<0xB1>(vmax);
        vmax = fqw_dpp_max<0x4E>(vmax);
        vmax = fqw_dpp_max<0x141>(vmax);                  // row_half_mirror
        vmax = fqw_dpp_max<0x140>(vmax);                  // row_mirror
        const float vm = vmax * up, s0 = vm * (1.0f / 7.0f);
        const float sigma = fminf(fmaf(fmaf(-7.0f, s0, vm), 1.0f / 7.0f, s0), 448.0f);   // (an infinity: NaN, and so 448)
        unsigned code = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(sigma, sigma, 0, false) & 0xFFu;   // nearest even
        float s8 = __builtin_amdgcn_cvt_f32_fp8((int)code, 0);
        if (!sigma_rne && s8 > sigma) {                   // toward zero: one code down (positive codes are ordered)
            code -= 1u;
            s8 = __builtin_amdgcn_cvt_f32_fp8((int)code, 0);
        }
        const float r0 = __builtin_amdgcn_rcpf(s8);
        const float r = s8 > 0.f ? fmaf(fmaf(-s8, r0, 1.0f), r0, r0) * up : 0.f, sb = s8 * back;
        if (!(s8 > 0.f) || !(vm < __builtin_inff())) {
            const float cut = 16.0f * sb;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fminf(fmaxf(v[i], -cut), cut);
        }
        unsigned y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float q0 = v[i] * r;
            const float q1 = fmaf(fmaf(-q0, sb, v[i]), r, q0);
            y[i] = __float_as_uint(__builtin_amdgcn_fmed3f(q1, -8.f, 7.f) + 12582912.0f);
        }
        fq_v2i out;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const unsigned lo = __builtin_amdgcn_perm(y[4 * x + 1], y[4 * x], 0x0C0C0400u);
            const unsigned hi = __builtin_amdgcn_perm(y[4 * x + 3], y[4 * x + 2], 0x04000C0Cu);
            out[x] = (int)(lo | hi);
        }
        const size_t row = row0 + u;
        if (row < (size_t)N) {
            *reinterpret_cast<fq_v2i*>(q + row * (size_t)K + 8u * cc) = out;
            if ((cc & 15u) == 0) gs[row * (size_t)(K / FQ_GROUP) + (cc >> 4)] = (uint8_t)code;
        }
    }
}

namespace {

// W is larger than the last-level cache (256 MiB): read once from end to end, nothing of it is left for the next pass.
bool fqw_past_cache(int N, int K) { return (long long)N * K * 2 > (256ll << 20); }

// How the rows and channels of W are shared out over one workgroup per compute unit.
struct fqw_cas_split { int slabs, cw, rows, shares; };
fqw_cas_split fqw_split_rows(int N, int K) {
    fqw_cas_split p;
    const int cols = K / 8;
    p.slabs = (cols + 63) / 64;
    p.cw = (cols + p.slabs - 1) / p.slabs;
    const int most = fq_device_cus() > p.slabs ? fq_device_cus() / p.slabs : 1;
    p.rows = (N + most - 1) / most;
    p.shares = (N + p.rows - 1) / p.rows;
    return p;
}

}  // namespace

// Where the kernels without scratch read less than whole lines per workgroup (16 or 32 channels) of many rows; few rows or 64
// channels are served as fast without a second launch.  Without | with scratch, us, from memory: 5120 x 2048 11.8 | 9.6, 11008 x
// 1024 24.9 | 11.2, 5120 x 5120 24.6 | 15.6, 6144 x 4096 22.3 | 13.6, 11008 x 4096 38.0 | 19.9, 22016 x 4096 74.8 | 33.3, 28672 x 8192
// 120 | 76; a matrix that the last-level cache holds: 5120 x 2048 8.2 | 9.1, 11008 x 1024 11.1 | 10.3, 5120 x 5120 16.3 | 14.5, 11008 x
// 4096 24.0 | 18.8 (at the line, what it costs the smallest of them from the cache it gives from memory).  On the other side
// of the line, from memory: 4000 x 4224 13.3 | 13.5, 2000 x 8192 10.3 | 11.5, 1024 x 4096 4.7 | 7.4, 4096 x 11008 20.5 | 21.4,
// 22016 x 11008 90.8 | 89.6; 4096 x 4096 13.8 | 11.6, but 7.7 | 10.4 from the cache.
size_t fq_cas_scales_scratch(int N, int K) {
    if (K % 8 != 0 || 2 * ((K + 63) / 64) > fq_device_cus() || N < 5120 || (long long)N * K < (8ll << 20)) return 0;
    return (size_t)fqw_split_rows(N, K).shares * (size_t)K * sizeof(double);
}

void fq_launch_cas_scales_split(const uint16_t* W, float target, float* lambda, int N, int K, void* scratch, hipStream_t stream) {
    const fqw_cas_split p = fqw_split_rows(N, K);
    double* part = static_cast<double*>(scratch);
    hipLaunchKernelGGL(fq_cas_partial_kernel, dim3((unsigned)(p.slabs * p.shares)), dim3(FQW_CASW_THREADS), 0, stream, W, part, N, K, p.slabs, p.cw, p.rows);
    hipLaunchKernelGGL(fq_cas_fold_kernel, dim3((unsigned)((K + 63) / 64)), dim3(256), 0, stream, part, W, target, lambda, N, K, p.shares);
}

void fq_launch_cas_scales(const uint16_t* W, float target, float* lambda, int N, int K, hipStream_t stream) {
    if ((K % 8) == 0 && (reinterpret_cast<uintptr_t>(W) % 16) == 0) {
        // channels per workgroup: the fewest that take no second round of workgroups (N x K, in cache: 11008 x 4096 with 16 channels
        // 22.9 us, 32 24.4, 64 28.2; 11008 x 5120, 320 workgroups of 16: 42.9, 32 28.6, 64 34.0; 14336 x 8192 with 32 47.1, 64 46.3;
        // 4096 x 11008 with 64 18.4, 32 21.8).  A matrix larger than the last-level cache is read nontemporally.
        const int lines = (K + 63) / 64, rounds = (lines + 7) / 8;      // (64 channels = a 128-byte line of a row)
        const int cus = fq_device_cus();
#define FQW_CASW(LPR_, STREAM_, GRID_) \
        hipLaunchKernelGGL((fq_cas_scales_wide_kernel<LPR_, STREAM_>), dim3((unsigned)(GRID_)), dim3(FQW_CASW_THREADS), 0, stream, W, target, lambda, N, K)
        if (2 * lines > cus) {
            if (fqw_past_cache(N, K)) FQW_CASW(8, true, 8 * rounds);
            else                      FQW_CASW(8, false, 8 * rounds);
        } else if (4 * lines > cus) FQW_CASW(4, false, 16 * rounds);
        else                        FQW_CASW(2, false, 32 * rounds);
#undef FQW_CASW
        return;
    }
    constexpr int CH = 2 * FQW_CAS_LPR;
    hipLaunchKernelGGL(fq_cas_scales_kernel, dim3((unsigned)((K + CH - 1) / CH)), dim3(FQW_CAS_THREADS), 0, stream, W, target, lambda, N, K);
}

// (rows of more chunks than that many workgroups have threads take more workgroups: none for those)
size_t fq_pts_exponent_scratch(int K) { return K / 8 <= FQW_PTS_WGS * FQW_PTS_THREADS ? 2 * sizeof(unsigned) * FQW_PTS_WGS : 0; }

void fq_launch_pts_exponent(const uint16_t* W, const float* lambda, int* n_out, int N, int K, void* scratch, hipStream_t stream) {
    unsigned* stats = scratch ? static_cast<unsigned*>(scratch)
                              : reinterpret_cast<unsigned*>(n_out) + 8;     // the caller's 64 bytes: [0] = n, [8..9] statistics
    // at most FQW_PTS_WGS workgroups' worth of threads, as whole rows of K / 8 chunk columns, with the same number of rows each.
    // One workgroup more than that (the number of rows rounded up, as it used to be) has to share a compute unit: 11008 x
    // 11008, 257 workgroups, 62 us, with 256 41; 256 x 11008 19.0, 13.7.
    const int KC = K / 8;
    int rows_par = FQW_PTS_WGS * FQW_PTS_THREADS / KC;
    if (rows_par < 1) rows_par = 1;
    const int passes = (N + rows_par - 1) / rows_par;
    rows_par = (N + passes - 1) / passes;
    const size_t threads = (size_t)KC * (size_t)rows_par;
    if (!scratch) hipLaunchKernelGGL(fq_pts_init_kernel, dim3(1), dim3(64), 0, stream, stats);
#define FQW_PTS_AS(THREADS_, STREAM_, PARTS_) \
    hipLaunchKernelGGL((fq_pts_stats_kernel<THREADS_, STREAM_, PARTS_>), dim3((unsigned)((threads + THREADS_ - 1u) / THREADS_)), dim3(THREADS_), 0, \
                       stream, W, lambda, stats, N, K, rows_par)
#define FQW_PTS(THREADS_, STREAM_) \
    do { if (scratch) FQW_PTS_AS(THREADS_, STREAM_, true); else FQW_PTS_AS(THREADS_, STREAM_, false); } while (0)
    // (64 x 128 10.0 us with workgroups of 1024, 7.3 with 256; 64 x 4096, 32 of 1024: 10.8, 9.6; 64 x 8192: 11.4, 13)
    const bool narrow = threads <= 32u * FQW_PTS_THREADS;
    if (narrow) FQW_PTS(256, false);
    else if (fqw_past_cache(N, K)) FQW_PTS(FQW_PTS_THREADS, true);
    else FQW_PTS(FQW_PTS_THREADS, false);
#undef FQW_PTS
#undef FQW_PTS_AS
    const size_t wg = narrow ? 256u : FQW_PTS_THREADS;
    if (scratch) hipLaunchKernelGGL(fq_pts_fold_kernel, dim3(1), dim3(FQW_PTS_WGS), 0, stream, stats, (int)((threads + wg - 1u) / wg), n_out);
    else hipLaunchKernelGGL(fq_pts_resolve_kernel, dim3(1), dim3(64), 0, stream, stats, n_out);
}

void fq_launch_quantize_weights(const uint16_t* W, const float* lambda, int n_pts, bool sigma_rne, int8_t* q,
                                uint8_t* gs, int N, int K, hipStream_t stream) {
    const size_t groups = (size_t)N * (size_t)(K / FQ_GROUP);
#define FQW_QUANTIZE(R_) \
    hipLaunchKernelGGL((fq_quantize_weights_kernel<R_>), dim3((unsigned)(((size_t)((N + R_ - 1) / R_) * (size_t)(K / 8) + 255u) / 256u)), dim3(256), \
                       0, stream, W, lambda, n_pts, sigma_rne ? 1 : 0, q, gs, N, K)
    // one row at a time where that takes at most four workgroups per compute unit: a second one only adds its latency (512 x 4096, 16384
    // groups: 3.3 us with one, 3.8 with two; 1024 x 4096: 5.1, 5.0)
    if (groups <= 16384u) FQW_QUANTIZE(1);
    else FQW_QUANTIZE(2);
#undef FQW_QUANTIZE
}
