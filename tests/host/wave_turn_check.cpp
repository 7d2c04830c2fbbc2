// The lane exchange of csrc/fq_turn.h with the 64 lanes of a wave run one after the other, each as far as it is free to run: up to
// the next place where the source orders the wave's accesses.  That is the farthest apart a compiler that sees one lane only may
// move them.  Several groups in a row, each checked against the operand that the matrix instruction defines.
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <ucontext.h>

#define LANES 64
#define GROUPS 3

typedef int fq_v4i __attribute__((ext_vector_type(4)));
#define __device__
#define __forceinline__ inline
static void lanes_meet();
#define __builtin_amdgcn_wave_barrier() ((void)0)         // (no order of memory accesses by itself)
#define asm
#define volatile(...) lanes_meet()                        // the compiler barrier: asm volatile("" ::: "memory")
#include "fq_turn.h"
#undef asm
#undef volatile

static ucontext_t here[LANES], back;
static char stacks[LANES][65536];
static int at;
static bool done[LANES];
static fq_v4i buffer[128], got[GROUPS][LANES][2];

static void lanes_meet() { swapcontext(&here[at], &back); }

static uint8_t code(int group, int row, int k) { return (uint8_t)(group * 97 + row * 13 + k * 7 + (k >> 5)); }

static void run_lane() {
    const int lane = at;
    const fqs_turn turn(lane);
    for (int g = 0; g < GROUPS; ++g) {
        fq_v4i half[2];
        for (int h = 0; h < 2; ++h)                       // lane 4 * r + c: bytes 16 * c .. of each 64-byte half of row r
            for (int b = 0; b < 16; ++b) ((uint8_t*)&half[h])[b] = code(g, lane >> 2, 64 * h + 16 * (lane & 3) + b);
        turn(buffer, half);
        got[g][lane][0] = half[0];
        got[g][lane][1] = half[1];
    }
    done[lane] = true;
}

int main() {
    memset(buffer, 0xEE, sizeof buffer);
    for (int l = 0; l < LANES; ++l) {
        getcontext(&here[l]);
        here[l].uc_stack.ss_sp = stacks[l];
        here[l].uc_stack.ss_size = sizeof stacks[l];
        here[l].uc_link = &back;
        makecontext(&here[l], run_lane, 0);
    }
    // every lane in turn to its next meeting place, from the first lane to the last and back again, until all are done
    int left = LANES;
    for (int round = 0; left > 0; ++round)
        for (int i = 0; i < LANES; ++i) {
            at = round & 1 ? LANES - 1 - i : i;
            if (done[at]) continue;
            swapcontext(&back, &here[at]);
            if (done[at]) --left;
        }
    int wrong = 0;
    for (int g = 0; g < GROUPS; ++g)
        for (int l = 0; l < LANES; ++l)
            for (int b = 0; b < 32; ++b)                  // lane 16 * kq + r: bytes 32 * kq .. of row r
                wrong += ((uint8_t*)got[g][l])[b] != code(g, l & 15, 32 * (l >> 4) + b);
    printf("wrong bytes %d\n", wrong);
    return wrong != 0;
}
