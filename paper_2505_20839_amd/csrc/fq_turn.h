// Activations of one group of 16 rows, on their way to an operand of the 16x16x128 MFMA.  The operand of lane 16*kq + r
// is 32 bytes of row r: neighbouring lanes hold different rows, so a wave that loads it as such touches 64 places of 16
// bytes, each of which takes the address path as long as four lanes that share 64 bytes.  So lane 4*r + c loads bytes
// 16*c .. of each 64-byte half of row r (two loads), and the halves change lanes through LDS: 2 KiB per wave, row-major,
// 16-byte slot x of row r at x ^ fqs_swizzle(r / 2), which spreads writes and reads over the banks.
//
// The buffer is the wave's own and the hardware keeps a wave's LDS accesses in order, so nothing is waited for and one buffer is
// enough for any number of groups in a row.  The compiler sees one lane only, whose reads and writes it may reorder where their
// places differ: fqs_wave_order holds it to the order that the other lanes need, the reads behind the writes that they read and
// the next group's writes behind these reads.  It is no instruction: a compiler barrier, and the mark that the wave meets there.
// (A wavefront fence over LDS in its place keeps the requests of the whole ring ahead of the first exchange, where the weights
// hold up the activations: 16 x 4096 x 14336 10.2 -> 10.9 us, 16 x 28672 x 4096 13.3 -> 13.5, 16 x 8192 x 8192 8.4 -> 8.7.)
#pragma once

// (fq_v4i: fq_common.h)
__device__ __forceinline__ int fqs_swizzle(int h) { return h ^ ((h & 2) << 1); }

__device__ __forceinline__ void fqs_wave_order() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

struct fqs_turn {
    int wr, rd;                                           // this lane's chunk in a row tile: to write (first half) and to read
    __device__ __forceinline__ fqs_turn(int lane) {
        const int rw = lane >> 2, rr = lane & 15;
        wr = 8 * rw + ((lane & 3) ^ fqs_swizzle(rw >> 1));
        rd = 8 * rr + ((2 * (lane >> 4)) ^ fqs_swizzle(rr >> 1));
    }
    __device__ __forceinline__ void operator()(fq_v4i* buf, fq_v4i (&half)[2]) const {   // the two halves as loaded -> the operand
        buf[wr] = half[0];
        buf[wr ^ 4] = half[1];
        fqs_wave_order();
        half[0] = buf[rd];
        half[1] = buf[rd ^ 1];
        fqs_wave_order();
    }
};
