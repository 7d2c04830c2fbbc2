// W4A8-FP GEMM for small M (decode, M <= 64): bound by streaming the packed INT4 weights from HBM
// once (Sec. 1: memory bandwidth is what motivates 4-bit weights).  Same arithmetic as the
// large-M kernel (Sec. 3.1.1): unpack INT4 to E4M3 in registers, FP8 MFMA with FP32 accumulation,
// exact FP32 group scale, one rounding to bf16.  The packed codes carry a zero point of 8; each
// group's MFMA chain starts from -2^-6 * sum_k a_k, which one more MFMA against a constant operand
// delivers (the matrix cores are idle at these sizes).
//
// Work split (both kernels).  The output channels are dealt out evenly to one workgroup per compute
// unit; its 8 waves split K into contiguous slices of groups, so every weight byte is read once
// overall and every activation byte once per workgroup; the partial sums of the waves are added
// through LDS.  Activations (M x K bytes) come from L2, a few rows straight in MFMA operand order, more in whole pieces of rows.
#include <cstdlib>
#include <type_traits>
#include "fq_common.h"
#include "fq_kernels.h"
#include "fq_turn.h"

namespace {

__device__ __forceinline__ fq_v8i fqs_join(fq_v4i lo, fq_v4i hi) {
    fq_v8i r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return r;
}

// Byte offset of lane 4*r + c's chunk in the first half of group 0, row m0 + r; rows past M are requested out of range.
__device__ __forceinline__ unsigned fqs_a_offset(int lane, int m0, int M, int K, unsigned oob) {
    const int m = m0 + (lane >> 2);
    return m < M ? (unsigned)m * (unsigned)K + (unsigned)(lane & 3) * 16u : oob;
}

// The larger of a's two halves in lanes 0-31 and of b's in lanes 32-63; of a's neighbouring quarters in quarters 0 and 2, of b's
// in 1 and 3.
__device__ __forceinline__ unsigned fqs_swap32_max(unsigned a, unsigned b) {
    const auto h = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    return h[0] > h[1] ? h[0] : h[1];
}
__device__ __forceinline__ unsigned fqs_swap16_max(unsigned a, unsigned b) {
    const auto h = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    return h[0] > h[1] ? h[0] : h[1];
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// M <= 16: one 16-row MFMA tile (v_mfma_f32_16x16x128_f8f6f4 = exactly one group per instruction).
// The output channels are dealt out evenly, in multiples of 8, to one workgroup per compute unit
// (N = 14336 on 256 units: 56 channels each), so that every unit streams the same number of weight
// bytes and the whole matrix is requested at once.  A workgroup of 8 waves covers its channels with
// NSUB <= 7 sub-tiles of 16 channels (the last one may be partly masked; with at most 4 a layer of 28672 channels took
// 1.75 rounds of workgroups); the waves split K into
// eight contiguous slices, so each activation byte is read once per workgroup and each weight byte
// once overall.  A wave requests the packed weights of its first 4, 8, 12 or 16 groups before it computes
// anything; with K = 4096 that is its whole share.
// Every load is a raw buffer load: masked lanes carry an out-of-range offset (they fetch nothing
// and read zero), group steps travel in the scalar offset, and the code has no branches between
// the first request and the last MFMA.
// The 16x16x128 operand of lane l = 16*kq + r holds 32 consecutive k (32*kq ..) of row/channel r,
// which is one 16-byte chunk of the packed block: chunk (h = kq/2, kh = kq%2, channel % 32).
// ---------------------------------------------------------------------------------------------
#define FQS16_THREADS 512
#define FQS16_WAVES 8
#define FQS16_MAXCOLS 112                                 // channels of a workgroup (7 sub-tiles: 56 KiB of partial sums in LDS)
#define FQS16_BYROW_K 1536                                // fused: the longest K that three rows and more convert by rows
#define FQS16_OOB 0xFFFFFF00u                             // beyond any 32-bit buffer size
// byte `i` (0..3, compile-time) of a word of E4M3 codes -> float
__device__ __forceinline__ float fq_e4m3_byte_to_float(unsigned w, int i) {
    return i == 0 ? __builtin_amdgcn_cvt_f32_fp8((int)w, 0) : i == 1 ? __builtin_amdgcn_cvt_f32_fp8((int)w, 1)
         : i == 2 ? __builtin_amdgcn_cvt_f32_fp8((int)w, 2) : __builtin_amdgcn_cvt_f32_fp8((int)w, 3);
}
#define FQ_MFMA16(a, b, c) __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4((a), (b), (c), 0, 0, 0, 0, 0, 0)

// The four scale bytes of a channel that go with four consecutive slots are one 8-byte load, the two aligned words around
// them, shifted into place when they are used.  Lane quarter kq fetches them for sub-tile kq (of four) and lane exchanges
// hand them to the other quarters: every channel's scales are a place of their own, a turn of the address path for each lane
// that asks, and with every lane asking for every sub-tile (twice where rows of scales are not whole words) it took more
// turns for them than for the weights (16 x 14336 x 4096 7.5 -> 7.3 us, 16 x 4096 x 14336 10.2 -> 9.95, 1 x 4096 x 14336 8.1 -> 7.8).
// A wave keeps a ring of BATCH groups in flight (4, 8, 12 or 16: the shortest that holds a wave's slice,
// as far as the registers go): it requests the first BATCH groups of its slice at
// once and re-requests each slot, for the group BATCH further on, as soon as it has used it.  Loads
// return in order, so the ring is consumed in the order it was requested.
typedef unsigned fqs_v2u __attribute__((ext_vector_type(2)));

template <int NSUB, int BATCH_>
struct fqs16_ring {
    static constexpr int BATCH = BATCH_;
    static_assert(BATCH % 4 == 0, "scale words cover four slots");
    fq_v4i bq[BATCH][NSUB];
    fq_v4i aq[BATCH][2];
    static constexpr int NSC = (NSUB + 3) / 4;            // scale loads of four slots: four sub-tiles each
    fqs_v2u sq[BATCH / 4][NSC];

    // request group g into slot i; groups at or past g_end request nothing and read as zeros
    // (LOAD_A = false: the activations of the slot come from elsewhere)
    template <bool LOAD_A, bool TURN>
    __device__ __forceinline__ void issue(int i, __amdgpu_buffer_rsrc_t rsA, __amdgpu_buffer_rsrc_t rsW,
                                          __amdgpu_buffer_rsrc_t rsG, unsigned aoff, const unsigned (&woff)[NSUB],
                                          const unsigned (&goff)[NSC], int g, int g_end) {
        const unsigned dead = g < g_end ? 0u : FQS16_OOB;
        if (i % 4 == 0) {
#pragma unroll
            for (int j = 0; j < NSC; ++j)
                sq[i / 4][j] = __builtin_bit_cast(fqs_v2u, __builtin_amdgcn_raw_buffer_load_b64(
                    rsG, ((goff[j] + (unsigned)g) & ~3u) | dead, 0, 0));
        }
        if (LOAD_A) {                                     // (the halves of a group's 128 bytes to be turned, or of the lane's 32)
            aq[i][0] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsA, aoff | dead, g * FQ_GROUP, 0));
            aq[i][1] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsA, aoff | dead, g * FQ_GROUP + (TURN ? 64 : 16), 0));
        }
#pragma unroll
        for (int j = 0; j < NSUB; ++j)                    // streamed once: non-temporal
            bq[i][j] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsW, woff[j] | dead, g * 2048, 2));
    }

    // the scale words of slots i .. i + 3 (i a multiple of 4, group g its first) of every sub-tile; bytes of groups at or
    // past g_end, whatever they are, are cleared
    __device__ __forceinline__ void scale_words(int i, const unsigned (&goff)[NSC], int g, int g_end, unsigned (&sw)[NSUB]) const {
        const int nv = g_end - g;
        const unsigned keep = nv >= 4 ? ~0u : (nv <= 0 ? 0u : (1u << (8 * nv)) - 1u);
#pragma unroll
        for (int j = 0; j < NSC; ++j) {
            const unsigned w = __builtin_amdgcn_alignbyte(sq[i / 4][j][1], sq[i / 4][j][0], (goff[j] + (unsigned)g) & 3u) & keep;
            const auto h = __builtin_amdgcn_permlane32_swap(w, w, false, false);          // quarters 0 1 0 1 and 2 3 2 3
            const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);   // 0 0 0 0 and 1 1 1 1
            sw[4 * j] = lo[0];
            if (4 * j + 1 < NSUB) sw[4 * j + 1] = lo[1];
            if (4 * j + 2 < NSUB) {
                const auto hi = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
                sw[4 * j + 2] = hi[0];
                if (4 * j + 3 < NSUB) sw[4 * j + 3] = hi[1];
            }
        }
    }

    // slot i -> accumulators (a dead group is all zeros, its scale too, and adds nothing); `sw`: the slot's scale words, read
    // before the slot group's first slot may be re-requested
    __device__ __forceinline__ void compute(int i, fq_v4f (&acc)[NSUB], const unsigned (&sw)[NSUB]) const {
        const fq_v4f zero4 = {0.f, 0.f, 0.f, 0.f};
        const fq_v8i a = fqs_join(aq[i][0], aq[i][1]);
        fq_v8i zp;
#pragma unroll
        for (int r = 0; r < 8; ++r) zp[r] = (int)FQ_ZP_BYTES;
        const fq_v4f c0 = FQ_MFMA16(a, zp, zero4);        // zero point: -2^-6 * sum_k a_k in every column
#pragma unroll
        for (int j = 0; j < NSUB; ++j) {
            const fq_v8i b = fq_unpack_chunk(bq[i][j]);
            const float s = fq_e4m3_byte_to_float(sw[j], i % 4);
            const fq_v4f p = FQ_MFMA16(a, b, c0);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][r] = fmaf(s, p[r], acc[j][r]);
        }
    }
};

// FUSEDQ (M <= QROWS <= 8, slices no longer than the ring): `A` holds the bf16 activations X [M,K] instead of E4M3 codes, and the kernel quantises
// them itself (Sec. 2.1 eq. 2, the arithmetic of the quantiser kernel) while the weights are on their way; every workgroup
// repeats it for all of X, some eight instructions per element, which for a few rows costs less than a second kernel.
// Up to four sub-tiles a wave reads the part of every row that its own slice of K multiplies, one 16-byte load per lane, row and four groups;
// the waves exchange the parts' largest patterns through LDS, and each converts its part and turns the codes into operands through
// LDS of its own.  The weights are requested when all waves have asked for their activations: the later waves' would queue up
// behind the weights of those before them (4096 x 4096, M = 1 / 4 / 8: 3.92 / 4.54 / 5.28 us without that barrier, 3.44 / 3.84 / 4.90
// with it; 5.22 / 5.29 with the first form of the conversion, a row per wave, 6.26 with two kernels at M = 8).  BYROW: wave w reads,
// converts and leaves row w for all, which is the faster way with five sub-tiles and more, where a wave's weights alone fill the
// queues (28672 x 4096, M = 1 and 4: by slices 13.3 and 14.2 us, by rows 12.8 and 13.0), and for short slices (fq_launch_linear16).
// `a_scale` is not read.
template <int NSUB, bool ROUNDS, int BATCH_, bool TURN, int QROWS = 0, bool BYROW_ = false>
__global__ __launch_bounds__(FQS16_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void fq_gemm_small16_kernel(
    const uint8_t* __restrict__ A, const float* __restrict__ a_scale, const uint8_t* __restrict__ wp,
    const uint8_t* __restrict__ gs, float tscale, uint16_t* Y, int M, int N, int K, int cols,
    int swiglu, const uint16_t* R) {
    constexpr bool FUSEDQ = QROWS > 0;                    // rows the fused form has room for
    static_assert(!(FUSEDQ && ROUNDS) && (!BYROW_ || BATCH_ == 4) && QROWS <= 8, "the fused form: a slice is all under way; by rows K <= 4096");
    typedef fqs16_ring<NSUB, BATCH_> ring_t;
    constexpr int BATCH = ring_t::BATCH;
    __shared__ float red[FQS16_WAVES][NSUB][4][64];
    __shared__ fq_v4i turned[TURN ? FQS16_WAVES : 1][TURN ? 128 : 1];   // 2 KiB per wave: see fqs_turn
    const int G = K / FQ_GROUP;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r16 = lane & 15, kq = lane >> 4;
    const int n_first = blockIdx.x * cols;                // this workgroup owns channels [n_first, n_first + cols)
    const int per = (G + FQS16_WAVES - 1) / FQS16_WAVES;
    const int g_begin = wave * per;
    const int g_end = (g_begin + per < G) ? g_begin + per : G;

    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(A), 0, (int)((unsigned)M * (unsigned)K * (FUSEDQ ? 2u : 1u)), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(wp), 0, (int)((unsigned)((N + 31) >> 5) * (unsigned)G * 2048u), 0x00020000);
    // (range rounded up to whole words, so that the array's last word is readable when it holds fewer
    // than four scales; the array is 16-byte aligned and the surplus bytes never enter a sum)
    const __amdgpu_buffer_rsrc_t rsG = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(gs), 0, (int)(((unsigned)N * (unsigned)G + 3u) & ~3u), 0x00020000);
    // per sub-tile: byte offset of this lane's chunk in group 0 of its packed block; per four sub-tiles: of the scale row
    // of channel r16 of the sub-tile that this lane's quarter fetches
    unsigned woff[NSUB], goff[ring_t::NSC];
#pragma unroll
    for (int j = 0; j < NSUB; ++j) {
        const int c = 16 * j + r16;
        const int n = n_first + c;
        const bool on = (c < cols) && (n < N);            // masked lanes request nothing and store nothing
        woff[j] = on ? (unsigned)(n >> 5) * (unsigned)G * 2048u + (unsigned)(kq >> 1) * 1024u +
                       (unsigned)((kq & 1) * 32 + (n & 31)) * 16u
                     : FQS16_OOB;
    }
#pragma unroll
    for (int j = 0; j < ring_t::NSC; ++j) {
        const int c = 16 * (4 * j + kq) + r16;
        goff[j] = c < cols && n_first + c < N ? (unsigned)(n_first + c) * (unsigned)G : FQS16_OOB;
    }
    const unsigned aoff = TURN ? fqs_a_offset(lane, 0, M, K, FQS16_OOB)
                               : (unsigned)(r16 < M ? r16 : M - 1) * (unsigned)K + (unsigned)kq * 32u;
    // output factor of the (at most two) elements this thread writes at the end, fetched up front
    constexpr int NOUT = (NSUB * 256 + FQS16_THREADS - 1) / FQS16_THREADS;
    float osc[NOUT];
    if (!FUSEDQ) {
#pragma unroll
        for (int i = 0; i < NOUT; ++i) {
            const int idx = threadIdx.x + i * FQS16_THREADS;
            const int m = 4 * ((idx & 63) >> 4) + ((idx >> 6) & 3);
            osc[i] = a_scale[m < M ? m : M - 1];
        }
    }

    fq_v4f acc[NSUB];
#pragma unroll
    for (int j = 0; j < NSUB; ++j) acc[j] = (fq_v4f){0.f, 0.f, 0.f, 0.f};

    ring_t ring;
    constexpr bool BYROW = FUSEDQ && BYROW_;              // wave w quantises row w, else its own slice of all rows
    constexpr int CPR = BATCH_ / 4;                       // 16-byte chunks of a row's slice per lane
    constexpr int XN = !FUSEDQ ? 1 : BYROW ? 8 : QROWS * CPR;   // chunks a lane holds: of its row (K <= 4096), or of all rows' slices
    // codes: rows 16 bytes further apart than they are long, which spreads the rows of an operand over the banks
    constexpr int QSTRIDE = BYROW ? 4096 + 16 : BATCH_ * FQ_GROUP + 16;
    __shared__ __attribute__((aligned(16))) uint8_t codes[!FUSEDQ || BYROW ? 1 : FQS16_WAVES][FUSEDQ ? QROWS * QSTRIDE : 1];
    __shared__ __attribute__((aligned(16))) unsigned tops[FUSEDQ ? 16 : 1][FQS16_WAVES];   // largest pattern by row and wave
    __shared__ float srow[FUSEDQ ? FQS16_WAVES : 1];      // row scales
    fq_v4i xr[XN];
    const bool my_row = BYROW && wave < M;
    const int held = 16 * (g_end - g_begin);              // chunks of a row in the wave's slice
    if (FUSEDQ) {                                         // first in the queue: they are needed first
#pragma unroll
        for (int c = 0; c < XN; ++c) {
            const int row = BYROW ? wave : c / CPR, chunk = lane + 64 * (BYROW ? c : c % CPR);
            const unsigned off = (unsigned)row * (unsigned)K * 2u + (BYROW ? 0u : (unsigned)g_begin * (2u * FQ_GROUP)) + (unsigned)chunk * 16u;
            const bool on = BYROW ? my_row && chunk < (K >> 3) : chunk < held && row < M;
            xr[c] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsA, on ? off : FQS16_OOB, 0, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!BYROW) asm volatile("s_barrier");
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) ring.template issue<!FUSEDQ, TURN>(i, rsA, rsW, rsG, aoff, woff, goff, g_begin + i, g_end);
    __builtin_amdgcn_sched_barrier(0);                    // all requests go out before any arithmetic
    if constexpr (FUSEDQ) {
        // the largest of a wave's numbers where there are NaN among them
        auto numbers_top = [&](float amax) __attribute__((always_inline)) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
            return __float_as_uint(amax) >> 16;
        };
        uint8_t* own = codes[BYROW ? 0 : wave];
        float s_out = 0.f;                                // lane l < M: the scale of row l (BYROW: every lane the wave's row's)
        if constexpr (BYROW) {
            if (my_row) {
                fq_v2us most = {0, 0};
#pragma unroll
                for (int c = 0; c < XN; ++c) most = fq_pattern_max(most, xr[c]);
                unsigned top = fq_wave_max(most[0] > most[1] ? most[0] : most[1]);
                const bool nan = top > FQ_BF16_INF;
                if (nan) {
                    float amax = 0.f;
#pragma unroll
                    for (int c = 0; c < XN; ++c) amax = fq_absmax_numbers(amax, xr[c]);
                    top = numbers_top(amax);
                }
                const fq_row_scale sc = fq_scale_of(top);
                if (lane == 0) srow[wave] = sc.s;
                auto convert = [&](auto fast_tag) __attribute__((always_inline)) {
                    constexpr bool FAST = decltype(fast_tag)::value;
#pragma unroll
                    for (int c = 0; c < XN; ++c)
                        if (lane + 64 * c < (K >> 3))
                            *reinterpret_cast<fq_v2i*>(own + wave * QSTRIDE + (lane + 64 * c) * 8) = fq_quant8<FAST>(xr[c], sc.s, sc.rcp);
                };
                if (__builtin_amdgcn_readfirstlane((int)(sc.fast && !nan))) convert(std::true_type());
                else convert(std::false_type());
            }
            __syncthreads();
            own += g_begin * FQ_GROUP;
        } else {
            // lane l holds row l % 16's largest pattern, as the maxima of all waves make it
            auto row_top = [&]() __attribute__((always_inline)) {
                __syncthreads();
                unsigned v = 0u;
#pragma unroll
                for (int w = 0; w < FQS16_WAVES; ++w) { const unsigned o = tops[r16][w]; v = o > v ? o : v; }
                return r16 < M ? v : 0u;
            };
            unsigned v[QROWS];
#pragma unroll
            for (int m = 0; m < QROWS; ++m) {
                fq_v2us p = {0, 0};
#pragma unroll
                for (int c = 0; c < CPR; ++c) p = fq_pattern_max(p, xr[m * CPR + c]);
                v[m] = p[0] > p[1] ? p[0] : p[1];
            }
            if constexpr (QROWS == 1) {
                const unsigned o = fq_wave_max(v[0]);
                if (lane == 0) tops[0][wave] = o;
            } else {
                // four rows to a register: halves and quarters change places until quarter j of the wave holds row j
                static_assert(QROWS % 4 == 0, "whole registers of rows");
#pragma unroll
                for (int m = 0; m < QROWS; m += 4) {
                    const unsigned o = fq_row16_max(fqs_swap16_max(fqs_swap32_max(v[m], v[m + 2]), fqs_swap32_max(v[m + 1], v[m + 3])));
                    if (r16 == 0) tops[m + kq][wave] = o;
                }
            }
            unsigned top = row_top();
            const bool nan = __any(top > FQ_BF16_INF);    // the same in every wave
            if (nan) {
                __syncthreads();
#pragma unroll
                for (int m = 0; m < QROWS; ++m) {
                    float amax = 0.f;
#pragma unroll
                    for (int c = 0; c < CPR; ++c) amax = fq_absmax_numbers(amax, xr[m * CPR + c]);
                    const unsigned o = numbers_top(amax);
                    if (lane == 0) tops[m][wave] = o;
                }
                top = row_top();
            }
            const fq_row_scale sc = fq_scale_of(top);
            s_out = sc.s;
            // one choice of quotient for all rows (the full division gives the same codes), then straight-line code
            auto convert = [&](auto fast_tag) __attribute__((always_inline)) {
                constexpr bool FAST = decltype(fast_tag)::value;
#pragma unroll
                for (int m = 0; m < QROWS; ++m)
                    if (m < M) {
                        const float s = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(sc.s), m));
                        const float rcp = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(sc.rcp), m));
#pragma unroll
                        for (int c = 0; c < CPR; ++c)
                            *reinterpret_cast<fq_v2i*>(own + m * QSTRIDE + (lane + 64 * c) * 8) = fq_quant8<FAST>(xr[m * CPR + c], s, rcp);
                    }
            };
            if (!nan && __all(sc.fast)) convert(std::true_type());
            else convert(std::false_type());
            fqs_wave_order();                             // (the wave's own LDS: its accesses stay in order)
        }
        // operands of this wave's slice: row r16 (rows past M repeat the last one, as the unfused form does)
        const uint8_t* arow = own + (r16 < M ? r16 : M - 1) * QSTRIDE + kq * 32;
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            if (!BYROW || g_begin + i < g_end) {          // (a wave's own part holds zeros past its slice)
                ring.aq[i][0] = *reinterpret_cast<const fq_v4i*>(arow + i * FQ_GROUP);
                ring.aq[i][1] = *reinterpret_cast<const fq_v4i*>(arow + i * FQ_GROUP + 16);
            } else {
                ring.aq[i][0] = ring.aq[i][1] = (fq_v4i){0, 0, 0, 0};
            }
        }
#pragma unroll
        for (int i = 0; i < NOUT; ++i) {
            const int idx = threadIdx.x + i * FQS16_THREADS;
            const int m = 4 * ((idx & 63) >> 4) + ((idx >> 6) & 3), mc = m < M ? m : M - 1;
            osc[i] = BYROW ? srow[mc] : __shfl(s_out, mc, 64);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // A slot's activations are turned AHEAD slots before their use: the way through LDS takes longer than a slot's arithmetic
    // (16 x 4096 x 14336 10.5 us one slot ahead, 10.2 three; with a ring of four it is the other way round)
    constexpr int AHEAD = BATCH > 4 ? 3 : 1;
    const fqs_turn turn(lane);
    auto turn_slot = [&](int i) __attribute__((always_inline)) {
        if (TURN) turn(turned[TURN ? wave : 0], ring.aq[i]);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) turn_slot(i);
    // ROUNDS == false: no slice is longer than BATCH groups, the ring is used once and never refilled
    for (int gb = g_begin; gb < g_end; gb += BATCH) {
        unsigned sw[NSUB];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            if (ROUNDS || i + AHEAD < BATCH) turn_slot((i + AHEAD) % BATCH);
            if (i % 4 == 0) ring.scale_words(i, goff, gb + i, g_end, sw);   // (their slot may be re-requested below)
            ring.compute(i, acc, sw);
            __builtin_amdgcn_sched_barrier(0);            // slot by slot, as the data lands
            if (ROUNDS) {
                ring.template issue<!FUSEDQ, TURN>(i, rsA, rsW, rsG, aoff, woff, goff, gb + BATCH + i, g_end);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!ROUNDS) break;
    }

    // ---- sum the K-slices of the 8 waves through LDS, scale, write bf16 ----
#pragma unroll
    for (int j = 0; j < NSUB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][j][r][lane] = acc[j][r];
    __syncthreads();
    const float outer = tscale * 512.0f;                  // weights were fed in units of 2^-9
#pragma unroll
    for (int i = 0; i < NOUT; ++i) {
        const int idx = threadIdx.x + i * FQS16_THREADS;  // NSUB * 256 outputs: [sub-tile][reg][lane]
        const int l = idx & 63, r = (idx >> 6) & 3, j = idx >> 8;
        if (j < NSUB) {
            float v = 0.f, vu = 0.f;
#pragma unroll
            for (int w = 0; w < FQS16_WAVES; ++w) v += red[w][j][r][l];
            if (swiglu) {                                 // the up channel of an even (gate) channel
#pragma unroll
                for (int w = 0; w < FQS16_WAVES; ++w) vu += red[w][j][r][l | 1];
            }
            const int m = 4 * (l >> 4) + r;
            const int c = 16 * j + (l & 15);
            const int n = n_first + c;
            if (m < M && c < cols && n < N) {
                const float f = osc[i] * outer;
                if (!swiglu) {
                    fq_v2f pr = {v * f, 0.f};
                    if (R) pr[0] = fmaf(v, f, __uint_as_float((unsigned)R[(size_t)m * N + n] << 16));   // residual, one rounding
                    fq_v2bf pk = __builtin_convertvector(pr, fq_v2bf);
                    Y[(size_t)m * N + n] = __builtin_bit_cast(unsigned short, pk[0]);
                } else if ((l & 1) == 0) {                // fused epilogue: H[m, n/2] = SiLU(gate) * up
                    fq_v2f pr = {fq_silu_mul(v * f, vu * f), 0.f};
                    fq_v2bf pk = __builtin_convertvector(pr, fq_v2bf);
                    Y[(size_t)m * (N >> 1) + (n >> 1)] = __builtin_bit_cast(unsigned short, pk[0]);
                }
            }
        }
    }
}

namespace {

// Whether the activations are loaded in whole 64-byte pieces and turned (fqs_turn).  With few rows most lanes of the direct form
// repeat a row at no cost, and the way through LDS stands before a wave's first matrix instruction, which few groups do not
// win back (`per`: groups per wave; us, turned / direct; N = 4096 is one sub-tile, 8192 two, 12288 three, 14336 four):
//     per 1   16 x 4096 x 1024 3.80 / 3.79, 16 x 14336 x 256 4.20 / 3.93
//     per 2   9 x 4096 x 1408 3.72 / 3.65, 12 x 4096 x 2048 3.95 / 4.00, 16 x 4096 x 2048 3.94 / 4.10; 12 x 8192 x 2048 4.64 / 4.56
//     per 4   9 x 4096 x 4096 4.22 / 4.30, 16 rows 4.47 / 4.84; 9 x 8192 x 4096 5.45 / 5.36, 16 rows 5.62 / 5.73; 16 x 14336 x 4096
//             7.85 / 7.61
//     more    9 x 12288 x 5120 9.31 / 9.28, 16 rows 9.45 / 9.94; 9 x 8192 x 8192 8.20 / 7.91, 16 rows 8.47 / 8.71
inline bool fqs16_turns(int M, int per, int nsub) {
    if (nsub == 1) return M >= 9 && M * per >= 24;
    return M >= 12 && per >= (nsub == 2 ? 3 : 5);
}

template <int NSUB, bool ROUNDS, int BATCH>
void fq_launch_small16b(unsigned grid, hipStream_t stream, const uint8_t* A, const float* a_scale,
                        const uint8_t* wp, const uint8_t* gs, float tscale, uint16_t* Y, int M, int N, int K, int cols, int swiglu, const uint16_t* R) {
    const int per = (K / FQ_GROUP + FQS16_WAVES - 1) / FQS16_WAVES;
    auto kernel = fq_gemm_small16_kernel<NSUB, ROUNDS, BATCH, false>;
    if constexpr (NSUB <= 2 || ROUNDS || BATCH > 4) {     // (three sub-tiles and more with at most four groups never turn)
        if (fqs16_turns(M, per, NSUB)) kernel = fq_gemm_small16_kernel<NSUB, ROUNDS, BATCH, true>;
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(FQS16_THREADS), 0, stream,
                       A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
}

// The fused form (bf16 activations in, quantised by the kernel); no kernel for what fq_linear_small_serves refuses.
template <int NSUB>
auto fq_linear16_kernel(int per, int M, int K) -> decltype(&fq_gemm_small16_kernel<NSUB, false, 4, false>) {
    // by rows or by slices (see the kernel): by rows with five sub-tiles and more, and where slices are so short that most of a wave's
    // lanes would have nothing of them (by rows / by slices, us: 4 x 4096 x 1024 3.70 / 3.95, 6 rows 4.01 / 4.58, 2 rows 3.59 / 3.59;
    // 6 x 4096 x 1152 4.07 / 4.60, 6 x 12288 x 1408 6.17 / 6.29; on the other side 6 x 4096 x 2048 4.74 / 4.61, 4 rows 4.24 / 3.99)
    constexpr bool WIDE = NSUB > 4;
    if (per <= 4) {
        if (M >= 3 && K <= FQS16_BYROW_K)
            return M <= 4 ? fq_gemm_small16_kernel<NSUB, false, 4, false, 4, true> : fq_gemm_small16_kernel<NSUB, false, 4, false, 8, true>;
        return M == 1 ? fq_gemm_small16_kernel<NSUB, false, 4, false, 1, WIDE> : M <= 4 ? fq_gemm_small16_kernel<NSUB, false, 4, false, 4, WIDE>
                                                                                        : fq_gemm_small16_kernel<NSUB, false, 4, false, 8, WIDE>;
    }
    // longer slices: the rings of the unfused form (fq_launch_small16)
    if constexpr (NSUB <= 4) {
        if (per <= 8) return M == 1 ? fq_gemm_small16_kernel<NSUB, false, 8, false, 1> : fq_gemm_small16_kernel<NSUB, false, 8, false, 4>;
    }
    if constexpr (NSUB <= 2) {
        if (per <= 12) return M == 1 ? fq_gemm_small16_kernel<NSUB, false, 12, false, 1> : fq_gemm_small16_kernel<NSUB, false, 12, false, 4>;
    }
    if constexpr (NSUB == 1) {
        if (per <= 16) return M == 1 ? fq_gemm_small16_kernel<NSUB, false, 16, false, 1> : fq_gemm_small16_kernel<NSUB, false, 16, false, 4>;
    }
    return nullptr;
}

template <int NSUB>
bool fq_launch_linear16(int per, unsigned grid, hipStream_t stream, const uint16_t* X,
                        const uint8_t* wp, const uint8_t* gs, float tscale, uint16_t* Y, int M, int N, int K, int cols) {
    const auto kernel = fq_linear16_kernel<NSUB>(per, M, K);
    if (!kernel) return false;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(FQS16_THREADS), 0, stream,
                       reinterpret_cast<const uint8_t*>(X), static_cast<const float*>(nullptr), wp, gs, tscale, Y, M, N, K, cols,
                       0, static_cast<const uint16_t*>(nullptr));
    return true;
}

// Ring depth: the shortest of 4, 8, 12, 16 that holds a wave's slice of `per` groups, as far as 200 registers go (a slot
// takes 8 for the activations and 4 per sub-tile: 16 / 12 / 8 / 4 groups for 1 / 2 / 3-4 / 5-7 sub-tiles); longer slices
// go round a ring of 12 / 8 / 4 groups (ROUNDS), which exposes the latency of the refills: 16 x 4096 x 14336, 14 groups
// per wave, 15.1 us round a ring of 12, 11.7 us with all of them requested at once.  5-7 sub-tiles are only taken
// for slices of at most 4 groups (fqs_shape_of).
template <int NSUB>
void fq_launch_small16(int per, unsigned grid, hipStream_t stream, const uint8_t* A, const float* a_scale,
                       const uint8_t* wp, const uint8_t* gs, float tscale, uint16_t* Y, int M, int N, int K, int cols, int swiglu, const uint16_t* R) {
    constexpr int CAP = NSUB == 1 ? 16 : NSUB == 2 ? 12 : NSUB <= 4 ? 8 : 4, RING = NSUB == 1 ? 12 : NSUB == 2 ? 8 : 4;
    if constexpr (NSUB <= 4) {
        if (per > CAP)
            return fq_launch_small16b<NSUB, true, RING>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        if (per > 4 && per > CAP - 4)
            return fq_launch_small16b<NSUB, false, CAP>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        if constexpr (CAP >= 12) {
            if (per > CAP - 8 && per > 4)
                return fq_launch_small16b<NSUB, false, CAP - 4>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        }
        if constexpr (CAP >= 16) {
            if (per > 4)
                return fq_launch_small16b<NSUB, false, CAP - 8>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        }
    }
    fq_launch_small16b<NSUB, false, 4>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// 16 < M <= 64, general form of the kernel above: MT <= 4 row tiles of 16 rows share every unpacked
// weight operand (the weights are still read from HBM once), and the group scales of the
// workgroup's channels (cols x K/128 bytes, contiguous in memory) are copied to LDS at the start
// instead of being fetched per group.
// ---------------------------------------------------------------------------------------------
#define FQSM_MAXCOLS 64
#define FQSM_TURN_BYTES (FQS16_WAVES * 2048)             // the waves' buffers of fqs_turn
#define FQSM_LDS_BYTES (160 * 1024)

template <int MT, int NSUB>
struct fqsm_ring {
    // (deeper rings -- a whole slice of 4 groups at MT = 3 -- are no faster: 37 x 14336 x 4096 12.1 -> 12.7 us, 20 x 4096 x
    // 11008 13.2 -> 15.7)
    static constexpr int BATCH = MT >= 3 ? 2 : (MT == 2 ? 4 : (NSUB <= 2 ? 8 : 4));
    fq_v4i bq[BATCH][NSUB];
    fq_v4i aq[BATCH][MT][2];

    // request group g into slot i; groups at or past g_end request nothing and read as zeros
    template <bool TURN>
    __device__ __forceinline__ void issue(int i, __amdgpu_buffer_rsrc_t rsA, __amdgpu_buffer_rsrc_t rsW,
                                          const unsigned (&aoff)[MT], const unsigned (&woff)[NSUB], int g, int g_end) {
        const unsigned dead = g < g_end ? 0u : FQS16_OOB;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            aq[i][t][0] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsA, aoff[t] | dead, g * FQ_GROUP, 0));
            aq[i][t][1] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsA, aoff[t] | dead, g * FQ_GROUP + (TURN ? 64 : 16), 0));
        }
#pragma unroll
        for (int j = 0; j < NSUB; ++j)                    // streamed once: non-temporal
            bq[i][j] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsW, woff[j] | dead, g * 2048, 2));
    }

    // slot i (group g) -> accumulators; a dead group is all zeros and adds nothing.  `sc` points at
    // this lane's first channel in the LDS scale table [group][64 channels].
    __device__ __forceinline__ void compute(int i, fq_v4f (&acc)[MT][NSUB], const uint8_t* sc, int g) const {
        const fq_v4f zero4 = {0.f, 0.f, 0.f, 0.f};
        fq_v8i zp;
#pragma unroll
        for (int r = 0; r < 8; ++r) zp[r] = (int)FQ_ZP_BYTES;
        fq_v8i a[MT];
        fq_v4f c0[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            a[t] = fqs_join(aq[i][t][0], aq[i][t][1]);
            c0[t] = FQ_MFMA16(a[t], zp, zero4);           // zero point: -2^-6 * sum_k a_k in every column
        }
        const uint8_t* scg = sc + g * FQSM_MAXCOLS;
#pragma unroll
        for (int j = 0; j < NSUB; ++j) {
            const fq_v8i b = fq_unpack_chunk(bq[i][j]);
            const float s = __builtin_amdgcn_cvt_f32_fp8((int)scg[16 * j], 0);
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const fq_v4f p = FQ_MFMA16(a[t], b, c0[t]);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[t][j][r] = fmaf(s, p[r], acc[t][j][r]);
            }
        }
    }
};

// TURN: the activations come in whole 64-byte pieces and are turned (fqs_turn); fq_launch_smallm has the rule.
template <int MT, int NSUB, bool ROUNDS, bool TURN>
__global__ __launch_bounds__(FQS16_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void fq_gemm_smallm_kernel(
    const uint8_t* __restrict__ A, const float* __restrict__ a_scale, const uint8_t* __restrict__ wp,
    const uint8_t* __restrict__ gs, float tscale, uint16_t* Y, int M, int N, int K, int cols,
    int swiglu, const uint16_t* R) {
    typedef fqsm_ring<MT, NSUB> ring_t;
    constexpr int BATCH = ring_t::BATCH;
    // LDS: first the waves' buffers of fqs_turn, if any, and the scale table [G][64] bytes, later (after a barrier) the partial
    // sums [wave][row tile][sub-tile][reg][lane] floats
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_bytes[];
    float* red = reinterpret_cast<float*>(lds_bytes);
    uint8_t* const smem = lds_bytes + (TURN ? FQSM_TURN_BYTES : 0);
    const int G = K / FQ_GROUP;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    fq_v4i* const turned = reinterpret_cast<fq_v4i*>(lds_bytes) + wave * 128;
    const int r16 = lane & 15, kq = lane >> 4;
    const int n_first = blockIdx.x * cols;                // this workgroup owns channels [n_first, n_first + cols)
    const int per = (G + FQS16_WAVES - 1) / FQS16_WAVES;
    const int g_begin = wave * per;
    const int g_end = (g_begin + per < G) ? g_begin + per : G;

    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(A), 0, (int)((unsigned)M * (unsigned)K), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(wp), 0, (int)((unsigned)((N + 31) >> 5) * (unsigned)G * 2048u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsG = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(gs), 0, (int)((unsigned)N * (unsigned)G), 0x00020000);
    // the scale bytes of this workgroup: (channel c, group g) at gs[(n_first + c) * G + g]; up to 8 per thread now,
    // the rest (K > 8192) after the ring has been requested.  Where rows of scales are whole words (K a multiple of
    // 512) a thread fetches words, two instead of eight loads ahead of the weights in the queue: a load costs the
    // address path the same whatever its width.
    const int nsc = FQSM_MAXCOLS * G;
    const bool scw = (G & 3) == 0;
    unsigned scb[8];
    if (scw) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int idx = 4 * (threadIdx.x + x * FQS16_THREADS);    // idx = c * G + g
            const int c = idx / G;
            const bool on = idx < nsc && c < cols && n_first + c < N;
            scb[x] = __builtin_amdgcn_raw_buffer_load_b32(rsG, on ? (unsigned)(n_first * G + idx) : FQS16_OOB, 0, 0);
        }
    } else {
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int idx = threadIdx.x + x * FQS16_THREADS;
            const int c = idx / G;
            const bool on = idx < nsc && c < cols && n_first + c < N;
            scb[x] = __builtin_amdgcn_raw_buffer_load_b8(rsG, on ? (unsigned)(n_first * G + idx) : FQS16_OOB, 0, 0);
        }
    }
    // per sub-tile: byte offset of this lane's chunk in group 0 of its packed block
    unsigned woff[NSUB];
#pragma unroll
    for (int j = 0; j < NSUB; ++j) {
        const int c = 16 * j + r16;
        const int n = n_first + c;
        const bool on = (c < cols) && (n < N);            // masked lanes request nothing and store nothing
        woff[j] = on ? (unsigned)(n >> 5) * (unsigned)G * 2048u + (unsigned)(kq >> 1) * 1024u +
                       (unsigned)((kq & 1) * 32 + (n & 31)) * 16u
                     : FQS16_OOB;
    }
    unsigned aoff[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int m = 16 * t + r16;
        aoff[t] = TURN ? fqs_a_offset(lane, 16 * t, M, K, FQS16_OOB) : (unsigned)(m < M ? m : M - 1) * (unsigned)K + (unsigned)kq * 32u;
    }
    // output factors of the elements this thread writes at the end, fetched up front
    constexpr int NOUT = (MT * NSUB * 256 + FQS16_THREADS - 1) / FQS16_THREADS;
    float osc[NOUT];
#pragma unroll
    for (int i = 0; i < NOUT; ++i) {
        const int idx = threadIdx.x + i * FQS16_THREADS;
        const int m = 16 * (idx / (256 * NSUB)) + 4 * ((idx & 63) >> 4) + ((idx >> 6) & 3);
        osc[i] = a_scale[m < M ? m : M - 1];
    }

    fq_v4f acc[MT][NSUB];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < NSUB; ++j) acc[t][j] = (fq_v4f){0.f, 0.f, 0.f, 0.f};

    ring_t ring;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) ring.template issue<TURN>(i, rsA, rsW, aoff, woff, g_begin + i, g_end);
    __builtin_amdgcn_sched_barrier(0);                    // all requests go out before anything else
    // scale table: transposed to [group][channel] so that a lane's sub-tiles are 16 bytes apart
    if (scw) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int idx = 4 * (threadIdx.x + x * FQS16_THREADS);
            const int c = idx / G, g = idx - c * G;       // (G % 4 == 0: the word's four groups belong to one channel)
            if (idx < nsc) {
#pragma unroll
                for (int e = 0; e < 4; ++e) smem[(g + e) * FQSM_MAXCOLS + c] = (uint8_t)(scb[x] >> (8 * e));
            }
        }
        for (int idx = 4 * (threadIdx.x + 2 * FQS16_THREADS); idx < nsc; idx += 4 * FQS16_THREADS) {
            const int c = idx / G, g = idx - c * G;
            const bool on = c < cols && n_first + c < N;
            const unsigned w = __builtin_amdgcn_raw_buffer_load_b32(rsG, on ? (unsigned)(n_first * G + idx) : FQS16_OOB, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) smem[(g + e) * FQSM_MAXCOLS + c] = (uint8_t)(w >> (8 * e));
        }
    } else {
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int idx = threadIdx.x + x * FQS16_THREADS;
            const int c = idx / G, g = idx - c * G;
            if (idx < nsc) smem[g * FQSM_MAXCOLS + c] = (uint8_t)scb[x];
        }
        for (int idx = threadIdx.x + 8 * FQS16_THREADS; idx < nsc; idx += FQS16_THREADS) {
            const int c = idx / G, g = idx - c * G;
            const bool on = c < cols && n_first + c < N;
            smem[g * FQSM_MAXCOLS + c] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(
                rsG, on ? (unsigned)(n_first * G + idx) : FQS16_OOB, 0, 0);
        }
    }
    __syncthreads();
    const uint8_t* sc = smem + r16;
    const fqs_turn turn(lane);
    auto turn_slot = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
            if (TURN) turn(turned, ring.aq[i][t]);
    };
    // ROUNDS == false: no slice is longer than BATCH groups, the ring is used once and never refilled
    for (int gb = g_begin; gb < g_end; gb += BATCH) {
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const int g = gb + i < G ? gb + i : G - 1;    // (a dead slot may read any scale: its sums are zero)
            turn_slot(i);
            ring.compute(i, acc, sc, g);
            __builtin_amdgcn_sched_barrier(0);            // slot by slot, as the data lands
            if (ROUNDS) {
                ring.template issue<TURN>(i, rsA, rsW, aoff, woff, gb + BATCH + i, g_end);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!ROUNDS) break;
    }

    // ---- sum the K-slices of the 8 waves through LDS (over the scale table), scale, write bf16 ----
    __syncthreads();                                      // every wave is done with the scale table
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < NSUB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(((wave * MT + t) * NSUB + j) * 4 + r) * 64 + lane] = acc[t][j][r];
    __syncthreads();
    const float outer = tscale * 512.0f;                  // weights were fed in units of 2^-9
#pragma unroll
    for (int i = 0; i < NOUT; ++i) {
        const int idx = threadIdx.x + i * FQS16_THREADS;  // MT * NSUB * 256 outputs: [row tile][sub-tile][reg][lane]
        const int l = idx & 63, r = (idx >> 6) & 3, j = (idx >> 8) % NSUB, t = idx / (256 * NSUB);
        if (t < MT) {
            float v = 0.f, vu = 0.f;
#pragma unroll
            for (int w = 0; w < FQS16_WAVES; ++w) v += red[w * (MT * NSUB * 256) + idx];
            if (swiglu) {                                 // the up channel of an even (gate) channel
#pragma unroll
                for (int w = 0; w < FQS16_WAVES; ++w) vu += red[w * (MT * NSUB * 256) + (idx | 1)];
            }
            const int m = 16 * t + 4 * (l >> 4) + r;
            const int c = 16 * j + (l & 15);
            const int n = n_first + c;
            if (m < M && c < cols && n < N) {
                const float f = osc[i] * outer;
                if (!swiglu) {
                    fq_v2f pr = {v * f, 0.f};
                    if (R) pr[0] = fmaf(v, f, __uint_as_float((unsigned)R[(size_t)m * N + n] << 16));   // residual, one rounding
                    fq_v2bf pk = __builtin_convertvector(pr, fq_v2bf);
                    Y[(size_t)m * N + n] = __builtin_bit_cast(unsigned short, pk[0]);
                } else if ((l & 1) == 0) {                // fused epilogue: H[m, n/2] = SiLU(gate) * up
                    fq_v2f pr = {fq_silu_mul(v * f, vu * f), 0.f};
                    fq_v2bf pk = __builtin_convertvector(pr, fq_v2bf);
                    Y[(size_t)m * (N >> 1) + (n >> 1)] = __builtin_bit_cast(unsigned short, pk[0]);
                }
            }
        }
    }
}

namespace {

template <int MT, int NSUB, bool ROUNDS, bool TURN>
void fq_launch_smallm_as(unsigned grid, hipStream_t stream, const uint8_t* A, const float* a_scale,
                         const uint8_t* wp, const uint8_t* gs, float tscale, uint16_t* Y, int M, int N, int K, int cols, int swiglu, const uint16_t* R) {
    const size_t red_bytes = (size_t)FQS16_WAVES * MT * NSUB * 256 * sizeof(float);
    const size_t sc_bytes = (size_t)FQSM_MAXCOLS * (K / FQ_GROUP) + (TURN ? FQSM_TURN_BYTES : 0);
    const size_t lds = red_bytes > sc_bytes ? red_bytes : sc_bytes;
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fq_gemm_smallm_kernel<MT, NSUB, ROUNDS, TURN>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((fq_gemm_smallm_kernel<MT, NSUB, ROUNDS, TURN>), dim3(grid), dim3(FQS16_THREADS), lds, stream,
                       A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
}

// The activations are turned where slices go round the ring and LDS has room for the buffers beside the scale table (K up to
// 294912): 64 x 4096 x 4096 10.8 -> 8.6 us, 64 x 4096 x 14336 30 -> 21, 48 x 8192 x 8192 16 -> 13.2, 24 x 4096 x 11008 13.6 -> 12.2.
// A slice that is all under way at once wins back the way through LDS only with three or four row tiles and two groups, from the
// rows below on (turned / direct: 33 x 4096 x 1408 1.07, 40 x 4096 x 2048 0.965, 48 1.00 and 0.92; 56 x 8192 x 2048 1.04, 64 x 6144 x
// 1408 0.97; 40 x 28672 x 2048 1.03, 49 1.02, 64 0.97; one group: 33 x 8192 x 1024 1.10, 48 1.08; two row tiles: 32 x 14336 x 4096 1.03).
template <int MT, int NSUB>
void fq_launch_smallm(int per, unsigned grid, hipStream_t stream, const uint8_t* A, const float* a_scale,
                      const uint8_t* wp, const uint8_t* gs, float tscale, uint16_t* Y, int M, int N, int K, int cols, int swiglu, const uint16_t* R) {
    if (per <= fqsm_ring<MT, NSUB>::BATCH) {
        if constexpr (MT >= 3) {
            if (per == 2 && M >= (NSUB == 1 ? 40 : 57))
                return fq_launch_smallm_as<MT, NSUB, false, true>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        }
        fq_launch_smallm_as<MT, NSUB, false, false>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
    } else if (FQSM_MAXCOLS * (K / FQ_GROUP) + FQSM_TURN_BYTES <= FQSM_LDS_BYTES)
        fq_launch_smallm_as<MT, NSUB, true, true>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
    else
        fq_launch_smallm_as<MT, NSUB, true, false>(grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
}

template <int MT>
void fq_launch_smallm_mt(int nsub, int per, unsigned grid, hipStream_t stream, const uint8_t* A, const float* a_scale,
                         const uint8_t* wp, const uint8_t* gs, float tscale, uint16_t* Y, int M, int N, int K, int cols, int swiglu, const uint16_t* R) {
    switch (nsub) {
        case 1: return fq_launch_smallm<MT, 1>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        case 2: return fq_launch_smallm<MT, 2>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        case 3: return fq_launch_smallm<MT, 3>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
        default: return fq_launch_smallm<MT, 4>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R);
    }
}

}  // namespace

namespace {

// How a small-M problem is cut up: channels per workgroup (an even share of N over the compute units,
// a multiple of 8, at most `max_cols`, or 64 where a wave's slice is longer than 4 groups; more channels than that go in
// several even rounds: 16 x 28672 x 4096 15.0 us in 448 workgroups of 64 channels, 13.3 us in 256 of 112; 64 x 18432 x 4096 27.0 us in
// 288 of 64, 25.3 in 461 of 40.  With more than 16 rows an even round of 49 to 63 channels has as many sub-tiles as one of 64 and more
// workgroups: 64 stay, 64 x 28672 x 4096 with the residual 30.7 us, in 512 of 56 32.3), workgroups, groups per wave and sub-tiles of 16 channels.
struct fqs_shape {
    int cols;
    unsigned grid;
    int per, nsub, rounds;
};

fqs_shape fqs_shape_of(int M, int N, int K, int max_cols) {
    const int cus = fq_device_cus();
    fqs_shape sh;
    const int G = K / FQ_GROUP;
    sh.per = (G + FQS16_WAVES - 1) / FQS16_WAVES;
    if (sh.per > 4 && max_cols > 64) max_cols = 64;
    sh.rounds = (int)(((long long)N + (long long)cus * max_cols - 1) / ((long long)cus * max_cols));
    const long long wgs = (long long)sh.rounds * cus;
    sh.cols = (int)((N + wgs - 1) / wgs + 7) & ~7;
    sh.cols = sh.cols < 8 ? 8 : (sh.cols > max_cols ? max_cols : sh.cols);
    if (M > 16 && sh.rounds > 1 && sh.cols > max_cols - 16) sh.cols = max_cols;
    sh.grid = (unsigned)((N + sh.cols - 1) / sh.cols);
    sh.nsub = (sh.cols + 15) / 16;
    return sh;
}

}  // namespace

// Where quantising inside the GEMM kernel pays (one kernel / quantiser and GEMM, us, replayed from graphs, weights in turn from 600 MB).
// One round of the compute units only, beyond six rows or K = 4096: every further round reads and converts X again (7 x 28680 x 4096
// 17.0 / 15.0, 8 x 32000 x 4096 18.3 / 15.6, 2 x 16640 x 8192 19.0 / 17.4, 1 x 128256 x 8192 98.4 / 91.9; 1 x 22016 x 5120 17.1 / 17.2).
// Slices of at most four groups, 7 and 8 rows: up to three sub-tiles (8 rows: 4096 x 4096 5.0 / 6.0, 8192 x 4096 6.7 / 7.3, 12288 x 4096 8.4 /
// 8.6, 12288 x 2048 7.3 / 7.3), with four only where it converts by rows (14336 x 1024 6.8 / 7.3, 16384 x 1536 7.4 / 7.6; by slices
// 14336 x 2048 8.3 / 8.0, 16384 x 3072 9.3 / 8.9); 12 rows, an earlier form: 4096 x 4096 7.2 / 6.5.
// Longer slices, all under way at once: the more channels a workgroup has, the less time for a wave's conversions, rows x groups:
//     8 channels    48   4 x 1024 x 11264 7.8 / 8.4, 4 x 2048 x 12288 8.2 / 9.0 (four rows and 12 groups, the kernels' most)
//     16            36   4 x 3072 x 9216 8.70 / 8.67, 3 x 4096 x 12288 9.06 / 8.95, 3 x 4096 x 8320 8.3 / 8.7; 4 x 4096 x 11008 9.6 / 9.1
//     24            24   2 x 5120 x 12288 10.3 / 10.7, 2 x 6144 x 12288 11.0 / 11.0; 3 x 6144 x 9216 11.2 / 10.7, 4 x 5120 x 9216 11.1 / 10.4
//     32            20   2 x 8192 x 10240 12.0 / 11.9, 3 x 8192 x 6144 8.7 / 8.9; 2 x 8192 x 12288 12.9 / 12.2, 4 x 8192 x 8192 10.1 / 9.8
//     up to 64      16   two rows: 9216 x 6144 9.8 / 10.1, 12288 x 8192 12.9 / 12.8, 16384 x 8192 17.7 / 17.7, 13824 x 8192 14.6 / 14.3; 4 x 14336 x 5120
//                        12.75 / 12.56
// and beyond 12 groups two rows (4096 x 14336 10.3 / 10.5, 4096 x 16384 10.95 / 10.56; 3 rows 11.3 / 11.1).
bool fq_linear_small_serves(int M, int N, int K) {
    if (M < 1 || M > 8) return false;
    if (M <= 6 && K <= 4 * FQS16_WAVES * FQ_GROUP) return true;
    const fqs_shape sh = fqs_shape_of(M, N, K, FQS16_MAXCOLS);
    if (sh.rounds > 1) return false;
    if (sh.per <= 4) return sh.nsub <= 3 || (sh.nsub == 4 && K <= FQS16_BYROW_K);
    if (sh.nsub > 4 || sh.per > (sh.nsub == 1 ? 16 : sh.nsub == 2 ? 12 : 8)) return false;
    if (M > (sh.nsub > 2 || sh.per > 12 ? 2 : 4)) return false;
    return M * sh.per <= (sh.cols <= 8 ? 48 : sh.cols <= 16 ? 36 : sh.cols <= 24 ? 24 : sh.cols <= 32 ? 20 : 16);
}

bool fq_launch_linear_small(const uint16_t* X, const uint8_t* wp, const uint8_t* gs, float tscale,
                            uint16_t* Y, int M, int N, int K, hipStream_t stream) {
    if (!fq_linear_small_serves(M, N, K)) return false;
    const fqs_shape sh = fqs_shape_of(M, N, K, FQS16_MAXCOLS);
    switch (sh.nsub) {
        case 1: return fq_launch_linear16<1>(sh.per, sh.grid, stream, X, wp, gs, tscale, Y, M, N, K, sh.cols);
        case 2: return fq_launch_linear16<2>(sh.per, sh.grid, stream, X, wp, gs, tscale, Y, M, N, K, sh.cols);
        case 3: return fq_launch_linear16<3>(sh.per, sh.grid, stream, X, wp, gs, tscale, Y, M, N, K, sh.cols);
        case 4: return fq_launch_linear16<4>(sh.per, sh.grid, stream, X, wp, gs, tscale, Y, M, N, K, sh.cols);
        case 5: return fq_launch_linear16<5>(sh.per, sh.grid, stream, X, wp, gs, tscale, Y, M, N, K, sh.cols);
        case 6: return fq_launch_linear16<6>(sh.per, sh.grid, stream, X, wp, gs, tscale, Y, M, N, K, sh.cols);
        default: return fq_launch_linear16<7>(sh.per, sh.grid, stream, X, wp, gs, tscale, Y, M, N, K, sh.cols);
    }
}

// M <= 64: the scale table of the kernel for more than 16 rows has to fit LDS (K <= 327680)
bool fq_gemm_small_serves(int M, int K) {
    return M <= 16 || (M <= 64 && (long long)FQSM_MAXCOLS * (K / FQ_GROUP) <= FQSM_LDS_BYTES);
}

bool fq_launch_gemm_small(const uint8_t* A, const float* a_scale, const uint8_t* wp, const uint8_t* gs,
                          float tscale, uint16_t* Y, int M, int N, int K, bool swiglu_epilogue, const uint16_t* R, hipStream_t stream) {
    if (!fq_gemm_small_serves(M, K)) return false;
    const int swiglu = swiglu_epilogue ? 1 : 0;
    const fqs_shape sh = fqs_shape_of(M, N, K, M <= 16 ? FQS16_MAXCOLS : FQSM_MAXCOLS);
    const int cols = sh.cols, per = sh.per, nsub = sh.nsub;
    const unsigned grid = sh.grid;
    if (M <= 16) {
        switch (nsub) {
            case 1: fq_launch_small16<1>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
            case 2: fq_launch_small16<2>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
            case 3: fq_launch_small16<3>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
            case 4: fq_launch_small16<4>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
            case 5: fq_launch_small16<5>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
            case 6: fq_launch_small16<6>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
            default: fq_launch_small16<7>(per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
        }
        return true;
    }
    switch ((M + 15) / 16) {
        case 2: fq_launch_smallm_mt<2>(nsub, per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
        case 3: fq_launch_smallm_mt<3>(nsub, per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
        default: fq_launch_smallm_mt<4>(nsub, per, grid, stream, A, a_scale, wp, gs, tscale, Y, M, N, K, cols, swiglu, R); break;
    }
    return true;
}
