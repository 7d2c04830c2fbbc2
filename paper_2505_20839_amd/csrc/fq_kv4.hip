// Attention operands with an INT4 key/value cache and FP8 queries (Sec. 3.2.1: queries FP8, keys and
// values INT4 with one scaling factor per token; Sec. 2.1: those factors are FP8; Sec. 3.1.1: the
// INT4 x FP8 product also forms S = Q K^T and O = P V).  Heads are 128 wide, so one token of one head is
// exactly one quantisation group, and both caches are kept in the packed layout of the linear layers
// (fq_common.h), one matrix per head:
//     keys    N = tokens (padded to 32), K = 128 head dimensions   (one group per token)
//     values  N = 128 head dimensions,   K = tokens (padded to 128, padding = code of q = 0)
// so that in both products the contraction index runs along the 32 consecutive codes a lane holds.
//
// Scores: the M <= 16 GEMM's arithmetic with a single group -- unpack to E4M3 (mask and shift; the
// zero point of 8 comes out again through one more MFMA against a constant operand, computed once per
// query tile), v_mfma_f32_16x16x128_f8f6f4, and the token's scale applied in FP32 to the finished sum.
// Output: the token's scale sits on the contraction index, so it cannot multiply a finished sum.  It is
// applied exactly all the same: P[r,t] * sigma[t] has at most 8 significant bits and q at most 4, both
// are exact bf16 numbers, and v_mfma_f32_16x16x32_bf16 forms exact products and adds them in FP32.
#include "fq_common.h"
#include "fq_kernels.h"

#define FQK_HEAD 128
#define FQK_OOB 0xFFFFFF00u

namespace {

typedef __bf16 fqk_v8bf __attribute__((ext_vector_type(8)));

// packed-cache bytes of one head
__host__ __device__ inline size_t fqk_key_bytes(int T) { return (size_t)((T + 31) / 32) * 32u * (FQK_HEAD / 2); }
__host__ __device__ inline size_t fqk_value_bytes(int T) { return (size_t)FQK_HEAD * (size_t)((T + 127) / 128 * 128) / 2u; }

// A key cache is the linear layers' packing of each head's [T,128] matrix (fq_launch_pack_many).  A value cache is packed
// transposed: n = dimension, k = token; tokens past T hold q = 0.  One wave per head and group of 128 tokens: lane
// 16 * s + d reads dimensions 8 d .. 8 d + 7 of the 32 tokens of segment s, 8 bytes each (a wave-level load is four whole
// rows of 128 bytes), packs pairs of tokens 16 apart, and turns four tokens x four dimensions round in registers at a
// time (byte permutes); the 16-byte chunks then change lanes through LDS (8 KiB of the wave's own, slots swizzled so that
// both accesses spread over the banks), so that a store writes runs of 512 bytes instead of 16 bytes here and
// there.  Bound by HBM, 1.5 bytes per code: 128 heads x 2000 tokens (49 MB) 9.8 us (5.0 TB/s); 16.2 with a branch per load, 19.8
// without the change of lanes, 62.8 with one thread per packed byte and its two byte loads 128 bytes apart.
typedef unsigned fqk_v2u_a1 __attribute__((ext_vector_type(2), aligned(1)));
__global__ __launch_bounds__(256) void fqk_pack_values_kernel(const int8_t* __restrict__ codes, uint8_t* __restrict__ packed,
                                                              int T, int G) {
    __shared__ fq_v4i turn[4][512];
    const int g = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (g >= G) return;
    const int8_t* src = codes + (size_t)blockIdx.y * T * FQK_HEAD + 8 * (lane & 15);
    const int t0 = 128 * g + 32 * (lane >> 4);
    unsigned w[32][2];
#pragma unroll
    for (int t = 0; t < 32; ++t) {
        // (tokens past T: the last one again, cleared below -- no branch between the 32 requests)
        const int tt = t0 + t < T ? t0 + t : T - 1;
        const fqk_v2u_a1 v = *reinterpret_cast<const fqk_v2u_a1*>(src + (size_t)tt * FQK_HEAD);
        w[t][0] = v[0];
        w[t][1] = v[1];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (128 * g + 128 > T) {
#pragma unroll
        for (int t = 0; t < 32; ++t) {
            w[t][0] = t0 + t < T ? w[t][0] : 0u;
            w[t][1] = t0 + t < T ? w[t][1] : 0u;
        }
    }
    fq_v4i* own = turn[threadIdx.x >> 6];                 // chunk [segment][dimension]
#pragma unroll
    for (int y = 0; y < 2; ++y) {                         // dimensions 4 y .. 4 y + 3 of the lane's eight
        fq_v4i out[4];                                    // [dimension]: bytes 0..15 = token pairs (j, 16 + j)
#pragma unroll
        for (int x = 0; x < 4; ++x) {                     // token pairs 4 x .. 4 x + 3
            unsigned p[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                p[i] = ((w[4 * x + i][y] & 0x0F0F0F0Fu) | ((w[16 + 4 * x + i][y] & 0x0F0F0F0Fu) << 4)) ^ 0x88888888u;
            // p[i] holds the four dimensions of pair i -> out[dimension][x] holds pairs 0..3
            const unsigned a0 = __builtin_amdgcn_perm(p[1], p[0], 0x05010400u), a1 = __builtin_amdgcn_perm(p[3], p[2], 0x05010400u);
            const unsigned b0 = __builtin_amdgcn_perm(p[1], p[0], 0x07030602u), b1 = __builtin_amdgcn_perm(p[3], p[2], 0x07030602u);
            out[0][x] = (int)__builtin_amdgcn_perm(a1, a0, 0x05040100u);
            out[1][x] = (int)__builtin_amdgcn_perm(a1, a0, 0x07060302u);
            out[2][x] = (int)__builtin_amdgcn_perm(b1, b0, 0x05040100u);
            out[3][x] = (int)__builtin_amdgcn_perm(b1, b0, 0x07060302u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = 8 * lane + 4 * y + i;
            own[p ^ ((p >> 4) & 7)] = out[i];
        }
    }
    // (other lanes' chunks are read back: the wave's own LDS accesses stay in order, which the fence holds the compiler to)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint8_t* dst = packed + (size_t)blockIdx.y * fqk_value_bytes(T) + (size_t)g * 2048u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int p = 64 * i + lane, n = p & 127, seg = p >> 7;
        *reinterpret_cast<fq_v4i*>(dst + (size_t)(n >> 5) * G * 2048u + (seg >> 1) * 1024 + ((seg & 1) * 32 + (n & 31)) * 16) =
            own[p ^ ((p >> 4) & 7)];
    }
}

// The same with a thread per packed byte, for a few groups (fq_launch_kv4_pack): bound by latency, which is that of two byte
// loads here and of 32 loads, a transposition and a change of lanes there.
__global__ __launch_bounds__(256) void fqk_pack_values_few_kernel(const int8_t* __restrict__ codes, uint8_t* __restrict__ packed,
                                                                  int T, int G) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x; // byte of the head's cache, a whole number of workgroups
    const int8_t* src = codes + (size_t)blockIdx.y * T * FQK_HEAD;
    const int blk = (int)(idx >> 11), in = (int)(idx & 2047u), lane = (in >> 4) & 63;
    const int n = (blk / G) * 32 + (lane & 31);           // dimension
    const int t = (blk % G) * 128 + 64 * (in >> 10) + 32 * (lane >> 5) + (in & 15);   // low nibble; the high one: 16 tokens on
    const unsigned lo = t < T ? fq_code_from_q(src[(size_t)t * FQK_HEAD + n]) : 8u;
    const unsigned hi = t + 16 < T ? fq_code_from_q(src[(size_t)(t + 16) * FQK_HEAD + n]) : 8u;
    packed[(size_t)blockIdx.y * fqk_value_bytes(T) + idx] = (uint8_t)(lo | (hi << 4));
}

template <bool VALUES>
__global__ __launch_bounds__(256) void fqk_unpack_kernel(const uint8_t* __restrict__ packed, int8_t* __restrict__ codes,
                                                         int T, size_t per_head) {
    const size_t idx = (size_t)blockIdx.x * 256u + threadIdx.x;   // element (t, c) of the head
    if (idx >= (size_t)T * FQK_HEAD) return;
    const int h = blockIdx.y;
    const int t = (int)(idx / FQK_HEAD), c = (int)(idx % FQK_HEAD);
    int hi;
    const size_t off = VALUES ? fq_weight_byte(c, t, (T + 127) / 128, &hi) : fq_weight_byte(t, c, 1, &hi);
    const unsigned byte = packed[(size_t)h * per_head + off];
    codes[(size_t)h * T * FQK_HEAD + idx] = (int8_t)fq_q_from_code(hi ? (byte >> 4) : (byte & 0xFu));
}

#define FQ_MFMA16(a, b, c) __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4((a), (b), (c), 0, 0, 0, 0, 0, 0)

__device__ __forceinline__ fq_v8i fqk_join(fq_v4i lo, fq_v4i hi) {
    fq_v8i r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return r;
}

// ---- S = Q K^T ------------------------------------------------------------------------------------------
// grid (token chunks, heads); a workgroup of 4 waves covers 4 * NSUB * 16 tokens, wave w the sub-tiles
// w * NSUB .. of 16 tokens each.  Lane l = 16 * kq + r holds, of the A operand, dimensions 32 kq .. of query
// row r, and of the B operand the same dimensions of token r of the sub-tile: one 16-byte chunk of the
// packed cache.  MT row tiles of 16 queries share every unpacked operand.
// A lane ends up with 4 rows x 1 token; the four lanes of a quad hold the same rows of four neighbouring tokens, and a
// 4 x 4 transpose of bf16 pairs inside the quad (two DPP exchanges) leaves each lane with one row x four tokens = one
// 8-byte store instead of four 2-byte ones, which cost the address path four times as much.  Rows of S start at any
// multiple of 2 bytes (T is whatever the cache has grown to): STORE 0, rows in 8-byte steps; 1, 8-byte stores of 2-byte
// alignment, the last, partial quad of a row token by token; 2, 2-byte stores without the transpose, where the memory side pays
// more for split lines than the address path saves (fq_launch_kv4_scores says where).
#define FQK_S_NSUB 4
typedef int fqk_v2i_a2 __attribute__((ext_vector_type(2), aligned(2)));
template <int MT, int STORE>
__global__ __launch_bounds__(256) void fq_kv4_scores_kernel(
    const uint8_t* __restrict__ Q, const float* __restrict__ q_scale, const uint8_t* __restrict__ kp,
    const uint8_t* __restrict__ ks, float out_scale, uint16_t* __restrict__ S, int R, int T) {
    const int h = blockIdx.y;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
    const int t_first = (blockIdx.x * 4 + wave) * (FQK_S_NSUB * 16);
    if (t_first >= T) return;
    const size_t kbytes = fqk_key_bytes(T);
    const __amdgpu_buffer_rsrc_t rsK = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(kp) + (size_t)h * kbytes, 0, (int)kbytes, 0x00020000);
    // all of this wave's cache chunks are requested before anything else (streamed once: non-temporal)
    fq_v4i bq[FQK_S_NSUB];
    float sig[FQK_S_NSUB];
#pragma unroll
    for (int j = 0; j < FQK_S_NSUB; ++j) {
        const int t = t_first + 16 * j + r16;
        const unsigned off = t < T ? (unsigned)(t >> 5) * 2048u + (unsigned)(kq >> 1) * 1024u +
                                     (unsigned)((kq & 1) * 32 + (t & 31)) * 16u
                                   : FQK_OOB;
        bq[j] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsK, off, 0, 2));
    }
    // token scales: lane (kq, r) fetches the one of token r of sub-tile kq, and the four lanes with the same r pass
    // them round (one byte load per lane instead of four: a load costs the address path the same whatever its width)
    {
        const int t = t_first + 16 * kq + r16;
        const float own = t < T ? fq_e4m3_to_float(ks[(size_t)h * T + t]) : 0.f;
        static_assert(FQK_S_NSUB == 4, "one sub-tile per lane quarter");
#pragma unroll
        for (int j = 0; j < FQK_S_NSUB; ++j) sig[j] = __shfl(own, 16 * j + r16, 64);
    }
    fq_v8i a[MT];
    fq_v4f c0[MT];
    float rs[MT][4];
    fq_v8i zp;
#pragma unroll
    for (int r = 0; r < 8; ++r) zp[r] = (int)FQ_ZP_BYTES;
    const fq_v4f zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = 16 * m + r16;
        const fq_v4i* qrow = reinterpret_cast<const fq_v4i*>(Q + ((size_t)h * R + (row < R ? row : R - 1)) * FQK_HEAD + 32 * kq);
        a[m] = fqk_join(qrow[0], qrow[1]);
        c0[m] = FQ_MFMA16(a[m], zp, zero4);               // -2^-6 * sum_c Q[r, c] in every column
#pragma unroll
        for (int i = 0; i < 4; ++i) {                     // output rows of this lane: 16 m + 4 kq + i
            const int orow = 16 * m + 4 * kq + i;
            rs[m][i] = q_scale[(size_t)h * R + (orow < R ? orow : R - 1)] * (out_scale * 512.0f);   // codes were fed in units of 2^-9
        }
    }
#pragma unroll
    for (int j = 0; j < FQK_S_NSUB; ++j) {
        const fq_v8i b = fq_unpack_chunk(bq[j]);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const fq_v4f p = FQ_MFMA16(a[m], b, c0[m]);
            if constexpr (STORE == 2) {
                const int t = t_first + 16 * j + r16;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int orow = 16 * m + 4 * kq + i;
                    const fq_v2f pr = {(sig[j] * p[i]) * rs[m][i], 0.f};
                    if (orow < R && t < T)
                        S[((size_t)h * R + orow) * T + t] = __builtin_bit_cast(unsigned short, __builtin_convertvector(pr, fq_v2bf)[0]);
                }
                continue;
            }
            const fq_v2f pr0 = {(sig[j] * p[0]) * rs[m][0], (sig[j] * p[1]) * rs[m][1]};
            const fq_v2f pr1 = {(sig[j] * p[2]) * rs[m][2], (sig[j] * p[3]) * rs[m][3]};
            const unsigned pk0 = __builtin_bit_cast(unsigned, __builtin_convertvector(pr0, fq_v2bf));   // rows 0, 1
            const unsigned pk1 = __builtin_bit_cast(unsigned, __builtin_convertvector(pr1, fq_v2bf));   // rows 2, 3
            const bool oddl = lane & 1, upper = (lane & 2) != 0;
            const unsigned sel = oddl ? 0x03020706u : 0x05040100u;   // even: (own.lo, partner.lo); odd: (partner.hi, own.hi)
            const unsigned n0 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)pk0, 0xB1, 0xF, 0xF, false);
            const unsigned n1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)pk1, 0xB1, 0xF, 0xF, false);
            const unsigned a0 = __builtin_amdgcn_perm(n0, pk0, sel);  // row 0 (even lane) / 1 (odd), the pair's two tokens
            const unsigned a1 = __builtin_amdgcn_perm(n1, pk1, sel);  // row 2 / 3
            const unsigned give = upper ? a0 : a1;
            const unsigned got = (unsigned)__builtin_amdgcn_update_dpp(0, (int)give, 0x4E, 0xF, 0xF, false);
            const fq_v2i out = upper ? (fq_v2i){(int)got, (int)a1} : (fq_v2i){(int)a0, (int)got};
            const int orow = 16 * m + 4 * kq + (lane & 3);            // the row this lane now holds, for tokens t4 .. t4 + 3
            const int t4 = t_first + 16 * j + (r16 & 12);
            if (orow < R && t4 < T) {
                uint16_t* dst = S + ((size_t)h * R + orow) * T + t4;
                if (STORE == 0) {
                    *reinterpret_cast<fq_v2i*>(dst) = out;
                } else if (t4 + 4 <= T) {
                    *reinterpret_cast<fqk_v2i_a2*>(dst) = out;
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (t4 + i < T) dst[i] = (uint16_t)((unsigned)out[i >> 1] >> (16 * (i & 1)));
                }
            }
        }
    }
}

// ---- O = P V --------------------------------------------------------------------------------------------
// A workgroup per head and slice of DT of the 8 dimension tiles (grid: heads x 8 / DT; fewer tiles per workgroup when
// there are few heads, so that the grid still covers the chip); its NW waves take the 128-token groups w, w + NW, ...
// and their partial results are added through LDS.  Lane l = 16 * kq + r fetches, per dimension tile, the 16-byte
// chunk of tokens 32 kq .. 32 kq + 31 of dimension r (one packed chunk), and the 32 probability codes (of query row r)
// and 32 scales of the same tokens: wide loads only, since a load costs the address path the same whatever its width.
// Four matrix instructions use a group up: number j4 takes, in every lane, tokens 32 kq + 8 j4 .. + 7 (the order of the
// summation index is free as long as both operands agree), i.e. bytes 8 j4 .. of the codes and scales and, of the
// chunk, the low (j4 < 2) or high nibbles of bytes 8 (j4 % 2) ...  A' = bf16(P * sigma) is the A operand.  A 4-bit code
// c = q + 8 becomes the bf16 number 16 + c in a byte shuffle (low byte 0x80 | c << 3, high byte 0x41: the binade [16, 32)
// has a spacing of 1/8).  The matrix cores therefore sum A' * (q + 24); one more MFMA against an all-ones operand
// delivers sum A', and 24 times that is taken off at the end (all products are exact; the offset costs a few FP32
// roundings of the larger intermediate sum, far below the tolerance).
// A wave keeps DEPTH groups in flight: what bounds a long cache is the latency of a group's loads times the groups a
// wave takes one after the other (8 heads x 32001 tokens: 394 us with byte loads and one block of 32 tokens ahead, 26.7
// us in this form on one workgroup per head and tile).
// CROWD: there are workgroups enough for two and more on every compute unit, and what counts is that they fit: at most 128
// registers, two groups in flight with up to 16 rows, one with up to 32 (256 heads x 32 rows x 2048 tokens 16.1 us with a ring of two,
// 160 registers and so one workgroup per compute unit; 12.3 in this form).
// ALIGNED: rows of P and of the scales start at multiples of 16 bytes and T is one (16-byte loads as they are; the steps past T
// are not fetched).  Otherwise -- a cache that grows by a token per step has any length -- the aligned words around the 32 bytes are
// fetched (one more 4-byte load each) and shifted into place; what lies past T in the last group is cleared, in the
// scales and in the codes, since neither the next row's bytes nor a padding's need be finite numbers.
//
// The waves' partial sums (DT dimension tiles and the row sums of A') are added through LDS in the order of the waves,
// the offset of 24 per code comes off, the row's scale goes on, one rounding to bf16.
// SPLIT: the workgroup has seen one slice of the tokens only; its sums go to `part` ([slice][head][row][128] FP32, offset
// already off) and fqk_output_combine_kernel adds the slices in their order.
template <int MT, int DT, int NW, bool SPLIT>
__device__ __forceinline__ void fqk_output_finish(const fq_v4f (&acc)[MT][DT + 1], float* red, const float* __restrict__ p_scale,
                                                  uint16_t* __restrict__ O, float* __restrict__ part, int h, int d0, int R, int r0, int rows) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int d = 0; d < DT + 1; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) red[(((wave * MT + m) * (DT + 1) + d) * 4 + i) * 64 + lane] = acc[m][d][i];
    __syncthreads();
    for (int idx = threadIdx.x; idx < MT * DT * 4 * 64; idx += 64 * NW) {
        const int l = idx & 63, i = (idx >> 6) & 3, d = (idx >> 8) % DT, m = (idx >> 8) / DT;
        const int row = 16 * m + 4 * (l >> 4) + i, dim = 16 * (d0 + d) + (l & 15);
        if (row < rows) {
            float v = 0.f, s1 = 0.f;                      // fixed order: deterministic
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                v += red[(((w * MT + m) * (DT + 1) + d) * 4 + i) * 64 + l];
                s1 += red[(((w * MT + m) * (DT + 1) + DT) * 4 + i) * 64 + l];
            }
            const size_t orow = (size_t)h * R + r0 + row;
            const float o = fmaf(-24.0f, s1, v);
            if (SPLIT) {
                part[((size_t)blockIdx.z * gridDim.x * R + orow) * FQK_HEAD + dim] = o;
                continue;
            }
            const fq_v2f pr = {o * p_scale[orow], 0.f};
            const fq_v2bf pk = __builtin_convertvector(pr, fq_v2bf);
            O[orow * FQK_HEAD + dim] = __builtin_bit_cast(unsigned short, pk[0]);
        }
    }
}

// Adds the slices' partial sums in the order of the slices (a fixed order: the result does not depend on timing).
__global__ __launch_bounds__(256) void fqk_output_combine_kernel(const float* __restrict__ part, const float* __restrict__ p_scale,
                                                                 uint16_t* __restrict__ O, unsigned n4, int slices) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x;   // four dimensions of one row
    if (i >= n4) return;
    fq_v4f v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int s = 0; s < slices; ++s) v += reinterpret_cast<const fq_v4f*>(part)[(size_t)s * n4 + i];
    const float ps = p_scale[i >> 5];
    const fq_v2bf lo = __builtin_convertvector((fq_v2f){v[0] * ps, v[1] * ps}, fq_v2bf);
    const fq_v2bf hi = __builtin_convertvector((fq_v2f){v[2] * ps, v[3] * ps}, fq_v2bf);
    uint16_t* dst = O + (size_t)i * 4;
    *reinterpret_cast<fqk_v2i_a2*>(dst) = (fq_v2i){__builtin_bit_cast(int, lo), __builtin_bit_cast(int, hi)};
}

// Rows r0 .. r0 + rows - 1 (at most 16 * MT) of the R query rows of every head; SPLIT: the token groups of slice blockIdx.z,
// `gper` of them.
template <int MT, int DT, int NW, int DEPTH, bool ALIGNED, bool SPLIT, bool CROWD>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(CROWD ? 4 : 1)))
void fq_kv4_output_kernel(
    const uint8_t* __restrict__ P, const float* __restrict__ p_scale, const uint8_t* __restrict__ vp,
    const uint8_t* __restrict__ vs, uint16_t* __restrict__ O, float* __restrict__ part, int R, int r0, int rows, int T, int ldp,
    int gper) {
    extern __shared__ float red[];                        // [NW][MT][DT + 1][4][64]
    constexpr int NWD = ALIGNED ? 8 : 9;                  // words fetched per 32 bytes
    const int d0 = blockIdx.y * DT;                       // first dimension tile of this workgroup
    const int h = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
    const int G = (T + 127) / 128;                        // 128-token groups of the packed value cache
    const int g_begin = SPLIT ? (int)blockIdx.z * gper : 0;
    const int g_end = SPLIT && g_begin + gper < G ? g_begin + gper : G;
    const size_t vbytes = fqk_value_bytes(T);
    const __amdgpu_buffer_rsrc_t rsV = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(vp) + (size_t)h * vbytes, 0, (int)vbytes, 0x00020000);
    // descriptors of the head's scales and probability rows: from the aligned word that holds the first byte to the one
    // that holds the last (bytes of those words outside the arrays never enter a sum)
    const uint8_t* s_base = vs + (size_t)h * T;
    const uint8_t* p_base = P + ((size_t)h * R + r0) * ldp;
    const unsigned s_off = ALIGNED ? 0u : (unsigned)(reinterpret_cast<uintptr_t>(s_base) & 3u);
    const unsigned p_off = ALIGNED ? 0u : (unsigned)(reinterpret_cast<uintptr_t>(p_base) & 3u);
    const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(s_base) - s_off, 0, (int)((s_off + (unsigned)T + 3u) & ~3u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsP = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(p_base) - p_off, 0, (int)((p_off + (unsigned)rows * (unsigned)ldp + 3u) & ~3u), 0x00020000);
    fq_v4f acc[MT][DT + 1];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int d = 0; d < DT + 1; ++d) acc[m][d] = (fq_v4f){0.f, 0.f, 0.f, 0.f};
    fqk_v8bf ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = __builtin_bit_cast(__bf16, (unsigned short)0x3F80);
    unsigned prow[MT];                                    // byte offset of this lane's 32 codes of group 0, per row tile
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = 16 * m + r16;
        prow[m] = p_off + (unsigned)(row < rows ? row : rows - 1) * (unsigned)ldp + 32u * kq;
    }
    const unsigned srow = s_off + 32u * kq;               // the same of its scales
    unsigned vlane[DT];                                   // this lane's chunk inside a 2048-byte block, per dimension tile
#pragma unroll
    for (int d = 0; d < DT; ++d) {
        const int dim = 16 * (d0 + d) + r16;
        vlane[d] = (unsigned)(dim >> 5) * (unsigned)G * 2048u + (unsigned)(kq >> 1) * 1024u +
                   (unsigned)((kq & 1) * 32 + (dim & 31)) * 16u;
    }
    struct fqk_raw { fq_v4i vq[DT]; unsigned ws[NWD]; unsigned wp[MT][NWD]; };
    // 32 bytes from `off` on, of which the first `nv` are valid (none if nv <= 0).  ALIGNED: nv is a multiple of 16, and the
    // 16-byte steps past it read zeros
    auto fetch32 = [&](__amdgpu_buffer_rsrc_t rs, unsigned off, int nv, unsigned (&w)[NWD]) __attribute__((always_inline)) {
        const unsigned o = nv > 0 ? (off & ~3u) : FQK_OOB;   // (steps in the per-lane offset: the range check sees only that)
        const fq_v4i lo = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
        const fq_v4i hi = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, !ALIGNED || nv > 16 ? o + 16u : FQK_OOB, 0, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) { w[i] = (unsigned)lo[i]; w[4 + i] = (unsigned)hi[i]; }
        if (!ALIGNED) w[NWD - 1] = __builtin_amdgcn_raw_buffer_load_b32(rs, o + 32u, 0, 0);
    };
    auto fetch = [&](int g, fqk_raw& raw) __attribute__((always_inline)) {
        const unsigned dead = g < g_end ? 0u : FQK_OOB;       // (a group past the end: zeros, which add nothing; no branch)
#pragma unroll
        for (int d = 0; d < DT; ++d)                      // (streamed once: non-temporal)
            raw.vq[d] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(
                rsV, (vlane[d] + (unsigned)g * 2048u) | dead, 0, 2));
        // (32 tokens that start past T hold nothing: not fetched)
        const int nv = g < g_end ? T - (128 * g + 32 * kq) : 0;
        fetch32(rsS, srow + 128u * (unsigned)g, nv, raw.ws);
#pragma unroll
        for (int m = 0; m < MT; ++m) fetch32(rsP, prow[m] + 128u * (unsigned)g, nv, raw.wp[m]);
    };
    // the 8 words of 32 bytes as fetched -> the bytes themselves; `nv` of them are valid
    auto settle = [&](unsigned (&w)[NWD], unsigned off, int nv, bool ragged) __attribute__((always_inline)) {
        if (!ALIGNED) {
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = __builtin_amdgcn_alignbyte(w[i + 1 < NWD ? i + 1 : NWD - 1], w[i], off & 3u);
        }
        if (ragged) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int n = nv - 4 * i;
                w[i] &= n >= 4 ? 0xFFFFFFFFu : n <= 0 ? 0u : (1u << (8 * n)) - 1u;
            }
        }
    };
    auto work = [&](int g, fqk_raw& cur) __attribute__((always_inline)) {
        const bool ragged = !ALIGNED && g == G - 1 && (T & 127) != 0;
        const int nv = T - (128 * g + 32 * kq);
        settle(cur.ws, srow, nv, ragged);
#pragma unroll
        for (int m = 0; m < MT; ++m) settle(cur.wp[m], prow[m], nv, ragged);
#pragma unroll
        for (int j4 = 0; j4 < 4; ++j4) {
            const int x = j4 >> 1, w0 = 2 * (j4 & 1);     // which 8 bytes of the 16-byte chunk
            float sg[8];                                  // sigma of the lane's 8 tokens (zero past T)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int w = (int)cur.ws[4 * x + w0 + y];
                const fq_v2f lo = __builtin_amdgcn_cvt_pk_f32_fp8(w, false), hi = __builtin_amdgcn_cvt_pk_f32_fp8(w, true);
                sg[4 * y] = lo[0]; sg[4 * y + 1] = lo[1]; sg[4 * y + 2] = hi[0]; sg[4 * y + 3] = hi[1];
            }
            fqk_v8bf a[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                float pv[8];
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const int w = (int)cur.wp[m][4 * x + w0 + y];
                    const fq_v2f lo = __builtin_amdgcn_cvt_pk_f32_fp8(w, false), hi = __builtin_amdgcn_cvt_pk_f32_fp8(w, true);
                    pv[4 * y] = lo[0]; pv[4 * y + 1] = lo[1]; pv[4 * y + 2] = hi[0]; pv[4 * y + 3] = hi[1];
                }
                // P * sigma: at most 8 significant bits, exact in FP32 and in bf16 (the conversion's rounding never acts)
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    const fq_v2f pr = {pv[j] * sg[j], pv[j + 1] * sg[j + 1]};
                    const fq_v2bf pb = __builtin_convertvector(pr, fq_v2bf);
                    a[m][j] = pb[0];
                    a[m][j + 1] = pb[1];
                }
                acc[m][DT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], ones, acc[m][DT], 0, 0, 0);   // sum_t A'[r, t], every column
            }
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                fq_v4i bw;
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const unsigned w = (unsigned)cur.vq[d][w0 + y];
                    const unsigned c3 = (((j4 >> 1) ? (w >> 1) : (w << 3)) & 0x78787878u) | 0x80808080u;   // 0x80 | c << 3, 4 tokens
                    bw[2 * y] = (int)__builtin_amdgcn_perm(0x41414141u, c3, 0x04010400u);
                    bw[2 * y + 1] = (int)__builtin_amdgcn_perm(0x41414141u, c3, 0x04030402u);
                }
                const fqk_v8bf b = __builtin_bit_cast(fqk_v8bf, bw);
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[m][d], 0, 0, 0);
            }
        }
    };
    if constexpr (CROWD && MT == 1) {
        fqk_raw cur, nxt;
        fetch(g_begin + wave, cur);
        for (int g = g_begin + wave; g < g_end; g += NW) {
            fetch(g + NW, nxt);
            __builtin_amdgcn_sched_barrier(0);
            work(g, cur);
            g += NW;
            if (g >= g_end) break;
            __builtin_amdgcn_sched_barrier(0);
            fetch(g + NW, cur);
            __builtin_amdgcn_sched_barrier(0);
            work(g, nxt);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (CROWD) {
        fqk_raw cur;
        for (int g = g_begin + wave; g < g_end; g += NW) {
            fetch(g, cur);
            __builtin_amdgcn_sched_barrier(0);
            work(g, cur);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        fqk_raw ring[DEPTH];
    #pragma unroll
        for (int i = 0; i < DEPTH; ++i) fetch(g_begin + wave + i * NW, ring[i]);
        __builtin_amdgcn_sched_barrier(0);                    // all requests go out before any arithmetic
        int g = g_begin + wave;
        for (; g + (DEPTH - 1) * NW < g_end; g += DEPTH * NW) {   // whole rounds of the ring
    #pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                work(g + i * NW, ring[i]);
                __builtin_amdgcn_sched_barrier(0);
                fetch(g + (i + DEPTH) * NW, ring[i]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    #pragma unroll
        for (int i = 0; i < DEPTH - 1; ++i)                   // the last, partial one
            if (g + i * NW < g_end) work(g + i * NW, ring[i]);
    }
    fqk_output_finish<MT, DT, NW, SPLIT>(acc, red, p_scale, O, part, h, d0, R, r0, rows);
}

}  // namespace

size_t fq_kv4_key_bytes(int T) { return fqk_key_bytes(T); }
size_t fq_kv4_value_bytes(int T) { return fqk_value_bytes(T); }

void fq_launch_kv4_pack(const int8_t* codes, uint8_t* packed, int H, int T, bool values, hipStream_t stream) {
    if (!values) {
        fq_launch_pack_many(codes, packed, H, T, FQK_HEAD, stream);
        return;
    }
    const int G = (T + 127) / 128;
    // few groups: 8 heads x 333 tokens (24 groups) 2.4 us with a thread per byte, 3.1 with a wave per group; 8 x 512 (32) 2.6, 3.1; 32
    // x 100 2.65, 2.8; 8 x 1000 (64) 3.5, 3.3
    if ((long long)H * G <= 32) {
        hipLaunchKernelGGL(fqk_pack_values_few_kernel, dim3((unsigned)G * 32u, (unsigned)H), dim3(256), 0, stream, codes, packed, T, G);
        return;
    }
    hipLaunchKernelGGL(fqk_pack_values_kernel, dim3((unsigned)(G + 3) / 4u, (unsigned)H), dim3(256), 0, stream, codes, packed, T, G);
}

void fq_launch_kv4_unpack(const uint8_t* packed, int8_t* codes, int H, int T, bool values, hipStream_t stream) {
    const size_t per_head = values ? fqk_value_bytes(T) : fqk_key_bytes(T);
    const dim3 grid((unsigned)(((size_t)T * FQK_HEAD + 255u) / 256u), (unsigned)H);
    if (values) hipLaunchKernelGGL(fqk_unpack_kernel<true>, grid, dim3(256), 0, stream, packed, codes, T, per_head);
    else        hipLaunchKernelGGL(fqk_unpack_kernel<false>, grid, dim3(256), 0, stream, packed, codes, T, per_head);
}

void fq_launch_kv4_scores(const uint8_t* Q, const float* q_scale, const uint8_t* kp, const uint8_t* ks, float out_scale,
                          uint16_t* S, int H, int R, int T, hipStream_t stream) {
    const dim3 grid((unsigned)((T + 4 * FQK_S_NSUB * 16 - 1) / (4 * FQK_S_NSUB * 16)), (unsigned)H);
    // rows in 8-byte steps; else, by rows at odd multiples of 2 bytes or even ones (128 heads, T = 4095 and 8190, 8-byte / 2-byte
    // stores, us: 4 rows 8.3 / 9.1 and 14.7 / 16.8; 8 rows 10.7 / 10.3 and 17.9 / 19.5; 16 rows 15.8 / 13.9 and 25.3 / 25.2; 24 rows
    // 23.6 / 19.1 and 33.4 / 33.9; 64 rows 46.5 / 40.8 and 78.1 / 72.1)
    const uintptr_t at = reinterpret_cast<uintptr_t>(S);
    const int store = (T % 4) == 0 && (at % 8) == 0 ? 0 : R > ((T & 1) != 0 || (at & 2u) != 0 ? 4 : 32) ? 2 : 1;
#define FQK_SCORES(MT_) \
    do { \
        if (store == 0)      hipLaunchKernelGGL((fq_kv4_scores_kernel<MT_, 0>), grid, dim3(256), 0, stream, Q, q_scale, kp, ks, out_scale, S, R, T); \
        else if (store == 1) hipLaunchKernelGGL((fq_kv4_scores_kernel<MT_, 1>), grid, dim3(256), 0, stream, Q, q_scale, kp, ks, out_scale, S, R, T); \
        else                 hipLaunchKernelGGL((fq_kv4_scores_kernel<MT_, 2>), grid, dim3(256), 0, stream, Q, q_scale, kp, ks, out_scale, S, R, T); \
    } while (0)
    switch ((R + 15) / 16) {
        case 1: FQK_SCORES(1); break;
        case 2: FQK_SCORES(2); break;
        case 3: FQK_SCORES(3); break;
        default: FQK_SCORES(4); break;
    }
#undef FQK_SCORES
}

namespace {

template <int MT, int DT, int NW, int DEPTH, bool ALIGNED, bool SPLIT, bool CROWD = false>
void fqk_launch_output(const uint8_t* P, const float* p_scale, const uint8_t* vp, const uint8_t* vs, uint16_t* O, float* part,
                       int H, int R, int r0, int rows, int T, int ldp, int slices, int gper, hipStream_t stream) {
    constexpr size_t lds = (size_t)NW * MT * (DT + 1) * 4 * 64 * sizeof(float);
    static fq_device_once attr_once;                      // (one per template instance)
    fq_once_per_device(attr_once, [] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fq_kv4_output_kernel<MT, DT, NW, DEPTH, ALIGNED, SPLIT, CROWD>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    });
    hipLaunchKernelGGL((fq_kv4_output_kernel<MT, DT, NW, DEPTH, ALIGNED, SPLIT, CROWD>), dim3((unsigned)H, 8 / DT, (unsigned)slices),
                       dim3(64 * NW), lds, stream, P, p_scale, vp, vs, O, part, R, r0, rows, T, ldp, gper);
}

template <int MT, bool ALIGNED>
void fqk_launch_output_dt(int dt, const uint8_t* P, const float* p_scale, const uint8_t* vp, const uint8_t* vs, uint16_t* O, float* part,
                          int H, int R, int r0, int rows, int T, int ldp, int slices, int gper, hipStream_t stream) {
#define FQK_OUT(DT_, NW_, DEPTH_, CROWD_) \
    fqk_launch_output<MT, DT_, NW_, DEPTH_, ALIGNED, false, CROWD_>(P, p_scale, vp, vs, O, nullptr, H, R, r0, rows, T, ldp, 1, 0, stream)
    if (slices > 1) fqk_launch_output<MT, 4, 8, 2, ALIGNED, true>(P, p_scale, vp, vs, O, part, H, R, r0, rows, T, ldp, slices, gper, stream);
    // more than a workgroup per compute unit (rows in 16-byte steps; without, the form has no advantage): 256 heads x 4 rows x 4096
    // tokens 14.4 us with the ring, 13.9; x 24 rows 21.7, 19.6; 512 heads x 24 rows x 2048 tokens 29.4, 22.8
    else if (ALIGNED && dt == 4 && 2 * H > fq_device_cus() && (MT == 2 || T > 1024)) FQK_OUT(4, 8, 2, ALIGNED);
    // a group per wave at most, nothing to keep in flight behind it (8 heads x 4 rows x 128 tokens 2.65 us with a ring of four, 2.38; x
    // 1000 3.7, 2.95); with 4 tiles and 32 rows in 16-byte steps the ring is as good and takes fewer registers
    else if (T <= 1024) {
        if (dt == 4) FQK_OUT(4, 8, (MT == 2 && ALIGNED ? 2 : 1), false);
        else if (dt == 2) FQK_OUT(2, 8, 1, false);
        else FQK_OUT(1, 8, 1, false);
    } else if (dt == 4) FQK_OUT(4, 8, 2, false);
    else if (dt == 2) FQK_OUT(2, 8, 2, false);
    // (8 heads x 4 rows x 4096 tokens 4.45 us with a ring of two, 4.95 with four; x 32 rows 7.0, 8.1; 16 waves instead: 8 x 4 x 2048
    // 5.6 us against 3.3)
    else if (T <= 4096) FQK_OUT(1, 8, 2, false);
    else FQK_OUT(1, 16, (MT == 1 ? 3 : 2), false);
#undef FQK_OUT
}

// Dimension tiles per workgroup without slices: the most (of 4) that still give a workgroup per compute unit.  Every
// workgroup of a head converts the same P * sigma, so fewer tiles mean more redundant conversions, more of them fewer
// workgroups (4 rows x 4096 tokens, us with 4 / 2 / 1 tiles: 32 heads 7.0 / 5.4 / 4.6; 64 heads 7.1 / 5.6 / 7.0; 128 heads 7.7 / 9.1
// / 12.4; x 24 rows 9.6 / 7.4 / 6.6, 9.7 / 7.6 / 11.2, 11.2 / 13.5 / 21.2.  Between the powers of two the next larger number is
// already the faster one: 48 heads 7.1 / 5.5 / 6.8, 96 heads 7.4 / 8.6 / 9.4).
int fqk_output_tiles(int H, int cus) {
    int dt = 4;
    while (dt > 1 && (long)H * (8 / dt) < (long)cus) dt >>= 1;
    return dt;
}

// Token slices of an output product that is given a workspace, and the groups of each: as many as fill the device with
// workgroups of 4 dimension tiles, every wave with at least one group.  A group costs a wave about 1 us (the conversions
// of its two to four waves per SIMD), slices with their second kernel 4.5 us before the first group, so slices are taken where they
// save a wave three groups or more.  Measured without -> with (4 rows): 8 heads x 32001 tokens 23.0 -> 8.4 us, x 16384 10.9 -> 6.2, x
// 8192 7.1 -> 5.6, x 4096 4.4 -> 6.0 (not taken); 1 head x 32768 19.1 -> 6.3; 32 heads x 16384 12.7 -> 10.9, x 8192 7.3 -> 7.9 (not
// taken); 64 heads x 16384 16.4 -> 15.8, x 8192 8.9 -> 10.1 (taken: there the line lies too low), x 4096 5.5 -> 7.5 (not taken).
// 24 rows: 8 heads x 8192 10.9 -> 7.0; 64 heads 12.9 -> 14.4.
int fqk_output_slices(int H, int T, int cus, int* gper) {
    const int G = (T + 127) / 128;
    *gper = G;
    int S = H > 0 ? cus / (2 * H) : 1;
    if (S > G / 8) S = G / 8;
    if (S < 2) return 1;
    const int per = (G + S - 1) / S;
    const int waves = fqk_output_tiles(H, cus) == 1 ? 16 : 8;
    if ((G + waves - 1) / waves - (per + 7) / 8 < 3) return 1;
    *gper = per;
    return (G + per - 1) / per;                           // (none of them empty)
}

}  // namespace

size_t fq_kv4_output_scratch_bytes(int H, int R, int T) {
    int gper;
    const int S = fqk_output_slices(H, T, fq_device_cus(), &gper);
    return S > 1 ? (size_t)S * (size_t)H * (size_t)R * FQK_HEAD * sizeof(float) : 0;
}

void fq_launch_kv4_output(const uint8_t* P, const float* p_scale, const uint8_t* vp, const uint8_t* vs, uint16_t* O,
                          int H, int R, int T, int ldp, void* scratch, hipStream_t stream) {
    const uintptr_t all = reinterpret_cast<uintptr_t>(P) | reinterpret_cast<uintptr_t>(vs) | (uintptr_t)T | (uintptr_t)ldp;
    const bool aligned = (all % 16) == 0;
    const int cus = fq_device_cus();
    int slices = 1, gper = 0;
    if (scratch) slices = fqk_output_slices(H, T, cus, &gper);
    float* part = static_cast<float*>(scratch);
    const int dt = fqk_output_tiles(H, cus);
    // rows of a head are addressed through 32-bit buffer offsets: all of them at once, unless rows are so long that
    // fewer fit (a row has less than 2^31 codes)
    const unsigned long long fit = 0xFFFFFF00ull / (unsigned long long)ldp;
    const int step = (unsigned long long)R <= fit ? R : (int)fit;
    for (int r0 = 0; r0 < R; r0 += step) {
        const int rows = R - r0 < step ? R - r0 : step;
#define FQK_OUTPUT(MT_) \
        do { \
            if (aligned) fqk_launch_output_dt<MT_, true>(dt, P, p_scale, vp, vs, O, part, H, R, r0, rows, T, ldp, slices, gper, stream); \
            else         fqk_launch_output_dt<MT_, false>(dt, P, p_scale, vp, vs, O, part, H, R, r0, rows, T, ldp, slices, gper, stream); \
        } while (0)
        if (rows <= 16) FQK_OUTPUT(1);
        else            FQK_OUTPUT(2);
#undef FQK_OUTPUT
    }
    if (slices > 1) {
        const unsigned n4 = (unsigned)H * (unsigned)R * (FQK_HEAD / 4);
        hipLaunchKernelGGL(fqk_output_combine_kernel, dim3((n4 + 255u) / 256u), dim3(256), 0, stream, part, p_scale, O, n4, slices);
    }
}
