// Offline weight packing and its inverse (Sec. 3.1: INT4 weights, groups of 128 along K).
// The byte order is described in fq_common.h.
#include "fq_common.h"
#include "fq_kernels.h"

// One wave per block (32 channels x 128 input channels): lane 32 * kh + n holds, for each half h, the 32 consecutive codes
// of its channel that one 16-byte chunk packs, fetches them with two 16-byte loads and writes the chunk with one store
// (a block is 2 KiB of consecutive chunks).  The four waves of a workgroup take neighbouring groups, so that a
// workgroup reads runs of 512 bytes.  Bound by HBM: 1.5 bytes per code.  Measured on 11008 x 4096 codes (68 MB): 10.8 us,
// 6.3 TB/s (partly from the last-level cache); one thread per packed byte, with two byte loads each, took 41 us.  blockIdx.y counts independent matrices
// of the same shape (the heads of a key cache).  q needs no alignment: rows start where the caller's array does.
typedef int fqp_v4i_a1 __attribute__((ext_vector_type(4), aligned(1)));
__global__ __launch_bounds__(256) void fq_pack_kernel(const int8_t* __restrict__ q, uint8_t* __restrict__ wp,
                                                      int N, int K, unsigned blocks) {
    const unsigned blk = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (blk >= blocks) return;
    const int G = K / FQ_GROUP, lane = threadIdx.x & 63;
    const int nt = (int)(blk / (unsigned)G), g = (int)(blk - (unsigned)nt * (unsigned)G);
    const int n = nt * 32 + (lane & 31);
    fq_v4i c[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) c[h][0] = c[h][1] = (fq_v4i){0, 0, 0, 0};
    if (n < N) {
        const int8_t* row = q + ((size_t)blockIdx.y * N + n) * K + (size_t)g * FQ_GROUP + 32 * (lane >> 5);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int x = 0; x < 2; ++x) c[h][x] = *reinterpret_cast<const fqp_v4i_a1*>(row + 64 * h + 16 * x);
    }
    uint8_t* out = wp + ((size_t)blockIdx.y * blocks + blk) * 2048u + lane * 16;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        fq_v4i o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned packed = (((unsigned)c[h][0][i] & 0x0F0F0F0Fu) | (((unsigned)c[h][1][i] & 0x0F0F0F0Fu) << 4)) ^ 0x88888888u;
            o[i] = n < N ? (int)packed : 0;               // code = (q + 8) mod 16; channels past N hold code 0
        }
        *reinterpret_cast<fq_v4i*>(out + h * 1024) = o;
    }
}

// One thread per weight.
__global__ __launch_bounds__(256) void fq_unpack_kernel(const uint8_t* __restrict__ wp, int8_t* __restrict__ q,
                                                        int N, int K, size_t total) {
    size_t idx = (size_t)blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    int n = (int)(idx / (size_t)K), k = (int)(idx % (size_t)K);
    int hi;
    size_t off = fq_weight_byte(n, k, K / FQ_GROUP, &hi);
    unsigned byte = wp[off];
    q[idx] = (int8_t)fq_q_from_code(hi ? (byte >> 4) : (byte & 0xFu));
}

void fq_launch_pack_many(const int8_t* q, uint8_t* wp, int matrices, int N, int K, hipStream_t stream) {
    const unsigned blocks = (unsigned)((size_t)((N + 31) / 32) * (size_t)(K / FQ_GROUP));
    hipLaunchKernelGGL(fq_pack_kernel, dim3((blocks + 3u) / 4u, (unsigned)matrices), dim3(256), 0, stream, q, wp, N, K, blocks);
}

void fq_launch_pack(const int8_t* q, uint8_t* wp, int N, int K, hipStream_t stream) {
    fq_launch_pack_many(q, wp, 1, N, K, stream);
}

void fq_launch_unpack(const uint8_t* wp, int8_t* q, int N, int K, hipStream_t stream) {
    size_t total = (size_t)N * (size_t)K;
    unsigned blocks = (unsigned)((total + 255u) / 256u);
    hipLaunchKernelGGL(fq_unpack_kernel, dim3(blocks), dim3(256), 0, stream, wp, q, N, K, total);
}
