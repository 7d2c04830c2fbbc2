// W4A8-FP GEMM for problems with too few output tiles to fill the chip (Sec. 3.1.1; same arithmetic and
// operand formats as fq_gemm_large.hip): a workgroup of 8 waves owns one tile of 32 * NMT rows x 32 * NW
// channels and splits K over KS = 8 / NW groups of NW waves.  Each K split streams its own A tiles through
// its own two LDS stages and its own packed weights (128- and 64-row tiles: both through registers, several groups
// ahead), with two chained v_mfma_f32_32x32x64_f8f6f4 per row tile and group and the group scale applied in FP32 to each
// group's partial sum, as in the large-M kernel; the splits' partial tiles are then added through LDS, each wave taking
// over NMT / KS row tiles, and the zero-point update, whose operands travel from the start, and the epilogue finish those.  The shapes:
//     NMT = 4, NW = 4, KS = 2   128 x 128 tiles, K halved: wherever these tiles fit one round of the compute units
//     NMT = 4, NW = 2, KS = 4   128 x 64 tiles, K quartered: where even these do (batched decode, chunked prefill,
//                               narrow layers)
//     NMT = 2, NW = 2, KS = 4   64 x 64 tiles, the zero point through the matrix cores (no workspace): M just
//                               below 64 with many channels, where the M <= 64 kernel is slowest
//     NMT = 8, NW = 4, KS = 2   256 x 128 tiles, K halved, only on request (fq_test_force_kernel)
// One workgroup per compute unit (64 to 160 KiB of LDS, two waves per SIMD).
//
// K slices: when even these tiles are fewer than the compute units, S workgroups share a tile, each taking a
// contiguous 1/S of the groups (and splitting that among its waves as above).  A workgroup's loop is bound by
// what one compute unit can pull from L2 (about 110 GB/s measured, and every step of a 128 x 64 tile moves
// 80 KiB for 8 matrix instructions per wave), so a tile finishes S times sooner.  Each slice writes its folded
// partial tile (FP32, in the accumulators' own layout) to the workspace and counts itself in; the workgroup that
// arrives last adds the S partial tiles in the order of the slices -- a fixed order, so the result does not
// depend on which one that is -- and goes on to the epilogue (each slice has made the zero-point update for its own groups);
// it leaves the counter at zero for the next call.  The S workgroups of a tile run on the same XCD, so the partial tiles stay in its L2.
#include <type_traits>
#include "fq_common.h"
#include "fq_kernels.h"
#include "fq_gemm_large_common.h"

#define FQK_WAVES 8
#define FQK_THREADS (64 * FQK_WAVES)

namespace {

// LDS: KS * 2 stages of 32 * NMT rows x 128 bytes, then (256 x 128 shape) 8 x 4 KiB of packed weights; reused for the fold
// (8 waves x NMT tiles of 4 KiB, all at once where they fit, else half of them at a time), the zero-point units and the output tile.
template <int NMT, int NW, int KS, bool ZPM>
struct fqk_cfg {
    static constexpr int BM = 32 * NMT, BN = 32 * NW;
    static constexpr int STG = 8 * BM;                    // 16-byte chunks per A stage
    static constexpr int OUT_STRIDE = BN * 2 + 16;        // bytes per row of the output tile staged in LDS
    static constexpr bool WREG = NMT <= 4;                // packed weights through registers instead of LDS
    static constexpr int LOOP_LDS = KS * 2 * STG * 16 + (WREG ? 0 : FQK_WAVES * 4096);
    // row tiles that go through LDS at a time when the K splits' partial tiles are added: all of them where the
    // stages have room for 8 waves x NMT tiles of 4 KiB, else half
    static constexpr int HALF = FQK_WAVES * NMT * 4096 <= (WREG ? 128 * 1024 : LOOP_LDS) ? NMT : (NMT / 2 > 0 ? NMT / 2 : 1);
    static constexpr int FOLD_LDS = FQK_WAVES * HALF * 4096;
    static constexpr int EPI_LDS = BM * OUT_STRIDE + 1024;
    static constexpr int WORK_LDS = LOOP_LDS > FOLD_LDS ? (LOOP_LDS > EPI_LDS ? LOOP_LDS : EPI_LDS)
                                                        : (FOLD_LDS > EPI_LDS ? FOLD_LDS : EPI_LDS);
    // zero-point units: rounds of 8 units of BM rows; the first two have a place of their own and travel from the start
    // (256 x 128 shape: no room)
    static constexpr int ZROUND = 8 * BM;                 // chunks
    static constexpr bool ZPRE = WREG && !ZPM;
    static constexpr int LDS = WORK_LDS + (ZPRE ? 2 * ZROUND * 16 : 0);
    static constexpr int ZBATCH = WORK_LDS / (ZROUND * 16) < 4 ? WORK_LDS / (ZROUND * 16) : 4;   // later rounds that travel together
    static_assert(NW * KS == FQK_WAVES && (NMT % KS == 0 || KS % NMT == 0) && (4 * NMT) % NW == 0 && 8 % NMT == 0, "shape");
    static_assert(LDS <= 160 * 1024, "LDS");
};

// ZPM: the zero point comes out through one more matrix instruction per operand half against a constant operand
// (every byte -2^-6), as in the small-M kernels, instead of the Z planes of a workspace: for problems that have none.
template <int NMT, int NW, int KS, bool ZPM = false>
__global__ __launch_bounds__(FQK_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void fq_gemm_ksplit_kernel(
    const uint8_t* __restrict__ A, const float* __restrict__ a_scale, const uint8_t* __restrict__ wp,
    const uint8_t* __restrict__ gs, float tscale, uint16_t* Y, int M, int N, int K,
    int tiles_m, int tiles_n, int pm, const uint16_t* __restrict__ planes, const uint16_t* R,
    int S, unsigned* counters, float* partials) {
    typedef fqk_cfg<NMT, NW, KS, ZPM> cfg;
    constexpr int NT = 4 * NMT / NW;                      // A transfers (8 rows each) per wave and stage
    constexpr int OWN = NMT >= KS ? NMT / KS : 1;         // row tiles a wave finishes (fewer row tiles than splits:
                                                          // the first NMT splits finish one each, the others none)
    extern __shared__ fq_v4i lds[];
    const int G = K / FQ_GROUP;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nw = wave % NW, kw = wave / NW;             // position along the channels / which K split
    // which tile: XCD x = blockIdx % 8 runs a contiguous range of the tiles, panels of `pm` row tiles, row
    // tile fastest inside a panel, so that the tiles an XCD runs at one time share rows of A and channels of W
    // (with K slices: workgroup j of an XCD is slice j % S of the XCD's tile j / S)
    int m0, n0, tile, slice;
    {
        const int x = blockIdx.x % FQL_XCDS, js = blockIdx.x / FQL_XCDS;
        const int j = js / S;
        slice = js - j * S;
        const int ntiles = tiles_m * tiles_n, base = ntiles / FQL_XCDS, rem = ntiles % FQL_XCDS;
        if (j >= base + (x < rem ? 1 : 0)) return;
        const int t = x * base + (x < rem ? x : rem) + j;
        tile = t;
        const int per_panel = pm * tiles_n;
        const int panel = t / per_panel, rest = t - panel * per_panel;
        const int ph = tiles_m - panel * pm < pm ? tiles_m - panel * pm : pm;
        const int tn = rest / ph, tm = panel * pm + (rest - tn * ph);
        m0 = tm * cfg::BM;
        n0 = tn * cfg::BN;
    }
    // the scale of row m0 + threadIdx.x, fetched now so that the epilogue does not wait for it (and not touched until then:
    // its product formed here held every other request back for the time of one load)
    static_assert(cfg::BM <= FQK_THREADS, "one row scale per thread");
    const float row_scale = a_scale[m0 + (int)threadIdx.x < M ? m0 + (int)threadIdx.x : M - 1];
    const int nw0 = n0 + nw * 32;                         // first output channel of this wave
    const bool wave_on = nw0 < N;                         // waves past N compute a duplicate tile and store nothing
    const int n = nw0 + (lane & 31);
    const bool n_ok = n < N;
    const int nt = wave_on ? (nw0 >> 5) : ((N - 1) >> 5);
    const unsigned wblk = (unsigned)nt * (unsigned)G * 2048u;
    const unsigned lane16 = (unsigned)lane * 16u;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(A), 0, (int)((unsigned)M * (unsigned)K), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(wp), 0, (int)((unsigned)((N + 31) >> 5) * (unsigned)G * 2048u), 0x00020000);
    const int C2 = fql_c2(G), ZU = FQL_ZPLANES * C2;
    const __amdgpu_buffer_rsrc_t rsZ = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(planes), 0, (int)((unsigned)ZU * (unsigned)M * 16u), 0x00020000);
    const unsigned abase = fql_a_lane_base(nw, lane, K, NT);
    [[maybe_unused]] const uint8_t* gsrow = gs + (size_t)(n_ok ? n : N - 1) * G;
    // this workgroup's slice of the groups: [sb, se); this split's groups: [gb, ge); every split runs `gper`
    // steps, the surplus ones as ghosts with scale 0
    const int sper = (G + S - 1) / S;
    const int sb = slice * sper < G ? slice * sper : G;
    const int se = sb + sper < G ? sb + sper : G;
    const int gper = (se - sb + KS - 1) / KS;
    const int gb = sb + kw * gper < se ? sb + kw * gper : se;
    const int ge = gb + gper < se ? gb + gper : se;
    const int glast = G - 1;
    auto gclamp = [&](int j) { const int g = gb + j; return g < ge ? g : (ge > gb ? ge - 1 : glast); };
    // ghost steps request their operands out of range: zeros arrive at once and nothing is fetched
    auto ghost = [&](int j) { return gb + j < ge ? 0u : FQL_OOB; };

    // ---- zero-point units of this slice's groups ----
    // Plane 0's units, then plane 1's (fql_c2), `znp` places each (an even number: places 2 i, 2 i + 1 are the two lane halves of one
    // matrix instruction), those past the slice's last unit empty.  Round r is places 8 r .. 8 r + 7.
    const int zu0 = sb >> 3, zun = ((se + 7) >> 3) - zu0, znp = (zun + 1) & ~1;
    const int rounds = ZPM ? 0 : (2 * znp + 7) >> 3;
    auto issue_z = [&](fq_v4i* dst, int r) __attribute__((always_inline)) {
        constexpr int SUBS = cfg::BM / 64;
#pragma unroll
        for (int t = 0; t < 8 * SUBS / FQK_WAVES; ++t) {
            const int q = wave + FQK_WAVES * t, slot = q / SUBS, sub = q - slot * SUBS;
            const int i = 8 * r + slot, plane = i >= znp ? 1 : 0, k = i - plane * znp;
            // (rows past M are masked too: the range check sees the per-lane offset only)
            const int row = m0 + 64 * sub + lane;
            const unsigned v = k < zun && row < M ? (unsigned)row * 16u : FQL_OOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsZ, (fql_lds_ptr)(dst + slot * cfg::BM + 64 * sub), 16, v,
                                                     (int)((unsigned)(plane * C2 + zu0 + k) * (unsigned)M * 16u), 0, 0);
        }
    };
    // their factors: 8 groups of this lane's channel per place, the aligned words around them (see fql_scales_issue)
    const int hl = lane >> 5;
    const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(gs), 0, (int)(((unsigned)N * (unsigned)G + 3u) & ~3u), 0x00020000);
    auto zgroup = [&](int r, int ci) __attribute__((always_inline)) {    // first group of this lane's place of chunk ci
        const int i = 8 * r + 2 * ci;
        return 8 * (zu0 + (i >= znp ? i - znp : i) + hl);
    };
    auto issue_sig = [&](int r, fql_raw_scales& raw) __attribute__((always_inline)) {
        typedef unsigned v3u __attribute__((ext_vector_type(3)));
#pragma unroll
        for (int ci = 0; ci < 4; ++ci) {
            const int g0 = zgroup(r, ci);
            const unsigned o = 8 * r + 2 * ci < 2 * znp && n_ok && g0 < se ? ((unsigned)n * (unsigned)G + (unsigned)g0) & ~3u : FQL_OOB;
            const v3u t = __builtin_bit_cast(v3u, __builtin_amdgcn_raw_buffer_load_b96(rsS, o, 0, 0));
            raw.d[ci][0] = t[0]; raw.d[ci][1] = t[1]; raw.d[ci][2] = t[2];
        }
    };

    const int r32 = lane & 31, sw = (r32 >> 1) & 7;
    const int o00 = r32 * 8 + ((2 * (lane >> 5)) ^ sw);
    const int o01 = o00 ^ 1, o10 = o00 ^ 4, o11 = o00 ^ 5;

    fq_v16f acc[NMT];
#pragma unroll
    for (int t = 0; t < NMT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    fq_v16f zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
    fq_v8i zpb;
#pragma unroll
    for (int r = 0; r < 8; ++r) zpb[r] = (int)FQ_ZP_BYTES;

    fq_v4i* stages = lds + kw * (2 * cfg::STG);           // this split's two A stages
    fq_v16f pprev = zero;
    float sprev = 0.f;
    if constexpr (cfg::WREG) {
        // ---- main loop, operands through registers ----
        // A step (one group) of a workgroup is 16 matrix instructions per SIMD, 1024 cycles, and measured 2500 with all of
        // its requests issued at its start: the 48 to 80 requests of the eight waves occupy the address path for 800 to 1300
        // cycles, and no wave gets past its own to its next MFMA.  Spread over the step's MFMAs it is 2100 (200 x 4096 x 11008
        // with two slices 27.5 -> 25.4 us, 512 x 4096 x 11008 40.3 -> 36.1; the compiler keeps transfers straight into
        // LDS from being spread, so A goes through registers).  Without any loads a step takes 1650 cycles, without LDS
        // reads as well 1150 (all three from copies of the loop without them).  More groups in flight change nothing.  Where a step has fewer requests it gives little (128 x 14336 x 4096
        // 16.6 -> 15.9 us, 64 x 14336 x 4096 10.7 -> 10.4), and with K = 1024 its longer start costs 0.35 us.
        // A(g) sits in register set g % RA until the middle of step g - 1, when it goes to LDS stage g & 1; W(g) in slot
        // g % 4 until it is unpacked during step g - 1; a word holds the group scales of four steps.
        constexpr int RA = 2;
        fq_v4i ra[RA][NT], wr[4][2];
        auto load_a = [&](int set, int j, int i) __attribute__((always_inline)) {
            unsigned ab = abase;
            if (NT > 4) asm volatile("" : "+v"(ab));      // (opaque, or the offsets of all transfers stay in registers)
            const unsigned v = (ab ^ ((i & 1) ? 64u : 0u)) + (unsigned)(m0 + 8 * i) * (unsigned)K;
            ra[set][i] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsA, v | ghost(j), gclamp(j) * FQ_GROUP, 0));
        };
        auto load_w = [&](int slot, int j, int h) __attribute__((always_inline)) {
            wr[slot][h] = __builtin_bit_cast(fq_v4i, __builtin_amdgcn_raw_buffer_load_b128(
                rsW, lane16 | ghost(j), wblk + (unsigned)gclamp(j) * 2048u + 1024u * (unsigned)h, 0));
        };
        auto put_a = [&](int set, int stage, int i) __attribute__((always_inline)) {
            stages[stage * cfg::STG + nw * (64 * NT) + lane + 64 * i] = ra[set][i];
        };
        // group scales: the word of steps 4 p .. 4 p + 3 from the aligned words around its bytes
        const __amdgpu_buffer_rsrc_t rsG = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t*>(gs), 0, (int)(((unsigned)N * (unsigned)G + 3u) & ~3u), 0x00020000);
        const unsigned goff = (unsigned)(n_ok ? n : N - 1) * (unsigned)G + (unsigned)gb;
        auto load_s = [&](int p) __attribute__((always_inline)) {
            return __builtin_amdgcn_raw_buffer_load_b32(rsG, (goff & ~3u) + 4u * (unsigned)p, 0, 0);
        };
        unsigned sw0 = load_s(0), sw1 = load_s(1), sw2 = 0u;
        // requested in the order of the steady state (the waits are timed for the shortest path into the loop)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i >= 4 - RA)
#pragma unroll
                for (int x = 0; x < NT; ++x) load_a(i - (4 - RA), i - (4 - RA), x);
            load_w(i, i, 0);
            load_w(i, i, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (cfg::ZPRE) {
            issue_z(lds + cfg::WORK_LDS / 16, 0);
            issue_z(lds + cfg::WORK_LDS / 16 + cfg::ZROUND, 1);   // (past the last round: nothing is fetched)
        }
        __builtin_amdgcn_sched_barrier(0);
        fq_v8i b0[2], b1[2];
        b0[0] = fq_unpack_chunk(wr[0][0]);
        b1[0] = fq_unpack_chunk(wr[0][1]);
        b0[1] = b0[0]; b1[1] = b1[0];
#pragma unroll
        for (int x = 0; x < NT; ++x) put_a(0, 0, x);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        fq_v8i an = fql_join(stages[o00], stages[o01]);
        // Step 4 p + u of this split (group gb + 4 p + u); `sw`: the scale bytes of steps 4 p .. 4 p + 3.
        auto step = [&](const int p, const unsigned sw, auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                const int j = 4 * p + u;
                const fq_v4i* cur = stages + (u & 1) * cfg::STG;
                const float t = u == 0 ? __builtin_amdgcn_cvt_f32_fp8((int)sw, 0) : u == 1 ? __builtin_amdgcn_cvt_f32_fp8((int)sw, 1)
                              : u == 2 ? __builtin_amdgcn_cvt_f32_fp8((int)sw, 2) : __builtin_amdgcn_cvt_f32_fp8((int)sw, 3);
                const float s = gb + j < ge ? t : 0.f;
                fq_v4i q = wr[(u + 1) & 3][0];
                fq_v16f pt;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    const int tp = (mt + NMT - 1) % NMT;
                    const float sp = (mt == 0) ? sprev : s;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        // The step's requests are spread over its MFMAs (see above).  A(j + 1) goes to the other stage (last read before the previous barrier) in the second half;
                        // the barrier stands before the step's last MFMA, when all of its operands have been read, so
                        // that this MFMA covers the next step's first reads.
                        constexpr int SLOTS = 2 * NMT;
                        const int sl = 2 * mt + h;
#pragma unroll
                        for (int x = 0; x < NT; ++x)
                            if (x * SLOTS / NT == sl) load_a(u % RA, j + RA, x);
                        if (sl == SLOTS / 2) load_w(u, j + 4, 0);
                        if (sl == SLOTS - 2) load_w(u, j + 4, 1);
                        if (u == 0 && sl == SLOTS - 1) sw2 = load_s(p + 2);
#pragma unroll
                        for (int x = 0; x < NT; ++x)
                            if (SLOTS / 2 - 1 + x * (SLOTS / 2) / NT == sl) put_a((u + 1) % RA, (u & 1) ^ 1, x);
                        const fq_v8i ac = an;
                        if (h == 0) {
                            an = fql_join(cur[mt * 256 + o10], cur[mt * 256 + o11]);
                        } else if (mt + 1 < NMT) {
                            an = fql_join(cur[(mt + 1) * 256 + o00], cur[(mt + 1) * 256 + o01]);
                        } else {
                            __builtin_amdgcn_sched_barrier(0);
                            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                            const fq_v4i* nxs = stages + ((u & 1) ^ 1) * cfg::STG;
                            an = fql_join(nxs[o00], nxs[o01]);
                        }
                        if (ZPM) pt = FQ_MFMA(ac, zpb, h == 0 ? zero : pt);   // -2^-6 * sum_k a_k in every column
                        if (h == 0) pt = FQ_MFMA(ac, b0[u & 1], ZPM ? pt : zero);
                        else        pt = FQ_MFMA(ac, b1[u & 1], pt);
#pragma unroll
                        for (int r = 8 * h; r < 8 * h + 8; ++r) acc[tp][r] = fmaf(sp, pprev[r], acc[tp][r]);
#pragma unroll
                        for (int e = 0; e < 8 / NMT; ++e) {
                            const int slot = (8 / NMT) * mt + e;
                            const unsigned w = (unsigned)q[slot & 3];
                            const int ev = (int)((h == 0 ? w : (w >> 4)) & 0x0F0F0F0Fu);
                            if (slot < 4) b0[(u & 1) ^ 1][4 * h + (slot & 3)] = ev;
                            else          b1[(u & 1) ^ 1][4 * h + (slot & 3)] = ev;
                        }
                        if (mt == NMT / 2 - 1 && h == 1) q = wr[(u + 1) & 3][1];
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x008, ZPM ? 2 : 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x020, 3, 0);
                        __builtin_amdgcn_sched_group_barrier(0x200, 4, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 24, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    pprev = pt;
                }
                sprev = s;
        };
        // Whole rounds of four steps, then the rest (the same number for all splits), the loop left at its end only: where a step
        // in its middle could leave it, the compiler timed the waits of its start for that way round and let hardly a request be
        // under way at the end of each round; and where the loop alone used the requests above, it put them behind its first
        // test, where the prologue paid their latency on top of the first operands' (200 x 4096 x 11008 25.5 -> 24.3 us,
        // 128 x 14336 x 4096 17.1 -> 16.2, 1500 x 2048 x 8192 34.2 -> 32.8, 64 x 14336 x 4096 12.1 -> 11.5).
        int p = 0;
        for (; 4 * p + 4 <= gper; ++p) {
            const unsigned sw = __builtin_amdgcn_alignbyte(sw1, sw0, goff & 3u);
            step(p, sw, std::integral_constant<int, 0>());
            step(p, sw, std::integral_constant<int, 1>());
            step(p, sw, std::integral_constant<int, 2>());
            step(p, sw, std::integral_constant<int, 3>());
            sw0 = sw1; sw1 = sw2;
        }
        if (4 * p < gper) {
            const unsigned sw = __builtin_amdgcn_alignbyte(sw1, sw0, goff & 3u);
            step(p, sw, std::integral_constant<int, 0>());
            if (4 * p + 1 < gper) {
                step(p, sw, std::integral_constant<int, 1>());
                if (4 * p + 2 < gper) step(p, sw, std::integral_constant<int, 2>());
            }
        }
    } else {
        // ---- prologue ----
        fq_v4i* wbuf = lds + KS * 2 * cfg::STG + wave * 256;  // this wave's two weight buffers
        // (both A stages are free at the start: the second group's tile travels with the first instead of one step later)
        fql_issue_a<NT>(rsA, abase, m0, K, stages, nw, gclamp(0), ghost(0));
        fql_issue_b(rsW, wbuf, lane16 | ghost(0), wblk + (unsigned)gclamp(0) * 2048u);
        fql_issue_b(rsW, wbuf + 128, lane16 | ghost(1), wblk + (unsigned)gclamp(1) * 2048u);
        fql_issue_a<NT>(rsA, abase, m0, K, stages + cfg::STG, nw, gclamp(1), ghost(1));
        unsigned psb[2];
        psb[0] = gsrow[gclamp(0)];
        psb[1] = gsrow[gclamp(1)];
        fq_v8i b0[2], b1[2];
        float sc[2];
        __builtin_amdgcn_s_waitcnt(FQL_WAIT_VM(0));
        b0[0] = fq_unpack_chunk(wbuf[lane]);
        b1[0] = fq_unpack_chunk(wbuf[64 + lane]);
        sc[0] = gb < ge ? __builtin_amdgcn_cvt_f32_fp8((int)psb[0], 0) : 0.f;
        b0[1] = b0[0]; b1[1] = b1[0]; sc[1] = 0.f;
        __syncthreads();

        const int npairs = (gper + 1) >> 1;
        fq_v8i an = fql_join(stages[o00], stages[o01]);
        for (int p = 0; p < npairs; ++p) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int j = 2 * p + u;                      // step of this split; group gb + j
                const fq_v4i* cur = stages + u * cfg::STG;
                if (j > 0) fql_issue_a<NT>(rsA, abase, m0, K, stages + (u ^ 1) * cfg::STG, nw, gclamp(j + 1), ghost(j + 1));
                const unsigned qs = psb[u ^ 1];
                fql_issue_b(rsW, wbuf + u * 128, lane16 | ghost(j + 2), wblk + (unsigned)gclamp(j + 2) * 2048u);
                psb[u] = gsrow[gclamp(j + 2)];
                __builtin_amdgcn_s_waitcnt(FQL_WAIT_VM(NT + 3));
                const fq_v4i* nxt = wbuf + (u ^ 1) * 128 + lane;
                const float s = sc[u];
                fq_v4i q = nxt[0];
                fq_v16f pt;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    const int tp = (mt + NMT - 1) % NMT;
                    const float sp = (mt == 0) ? sprev : s;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const fq_v8i ac = an;
                        if (h == 0) {
                            an = fql_join(cur[mt * 256 + o10], cur[mt * 256 + o11]);
                        } else if (mt + 1 < NMT) {
                            an = fql_join(cur[(mt + 1) * 256 + o00], cur[(mt + 1) * 256 + o01]);
                        }
                        if (ZPM) pt = FQ_MFMA(ac, zpb, h == 0 ? zero : pt);   // -2^-6 * sum_k a_k in every column
                        if (h == 0) pt = FQ_MFMA(ac, b0[u], ZPM ? pt : zero);
                        else        pt = FQ_MFMA(ac, b1[u], pt);
#pragma unroll
                        for (int r = 8 * h; r < 8 * h + 8; ++r) acc[tp][r] = fmaf(sp, pprev[r], acc[tp][r]);
#pragma unroll
                        for (int e = 0; e < 8 / NMT; ++e) {
                            const int slot = (8 / NMT) * mt + e;
                            const unsigned w = (unsigned)q[slot & 3];
                            const int ev = (int)((h == 0 ? w : (w >> 4)) & 0x0F0F0F0Fu);
                            if (slot < 4) b0[u ^ 1][4 * h + (slot & 3)] = ev;
                            else          b1[u ^ 1][4 * h + (slot & 3)] = ev;
                        }
                        if (mt == NMT / 2 - 1 && h == 1) q = nxt[64];
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x008, ZPM ? 2 : 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 24, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    pprev = pt;
                }
                sprev = s;
                {
                    const float t = __builtin_amdgcn_cvt_f32_fp8((int)qs, 0);
                    sc[u ^ 1] = (gb + j + 1 < ge) ? t : 0.f;
                }
                __builtin_amdgcn_s_waitcnt(FQL_WAIT_VM(3));
                __syncthreads();
                {
                    const fq_v4i* nxs = stages + (u ^ 1) * cfg::STG;
                    an = fql_join(nxs[o00], nxs[o01]);
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[NMT - 1][r] = fmaf(sprev, pprev[r], acc[NMT - 1][r]);

    // The first zero-point units, older than any request of the loop, and ghost requests, which fetch nothing, have landed
    // (waited for here, or the compiler makes the barrier below wait for the residual and the scale words too).
    if (cfg::ZPRE) __builtin_amdgcn_s_waitcnt(FQL_WAIT_VM(0));

    // ---- residual tile: requested now, used in the epilogue ----
    // (step `it` of the epilogue: rows 8 * it + 4 * (lane / 32) + 0..3 of the wave's own rows; the even lane of a pair
    // fetches both channels' bf16 of rows 0, 1 as dwords, the odd lane those of rows 2, 3.  Rows past M lie behind the
    // descriptor's range and read zero, channels past N wrap into the next row and are never stored.  A slice that
    // does not finish the tile fetches values it never uses.)
    const int mrows = M - m0 < cfg::BM ? M - m0 : cfg::BM;   // rows of the tile that exist
    const bool wide_rows = (N & 7) == 0;                  // rows of Y and R in 16-byte steps: whole-row stores
    const bool add_wide = R != nullptr && wide_rows;
    unsigned rres[4 * OWN][2];
    if (add_wide && kw * OWN < NMT) {
        const __amdgpu_buffer_rsrc_t rsR = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(R) + (size_t)m0 * N + n0, 0, (int)(((unsigned)mrows * (unsigned)N - (unsigned)n0) * 2u), 0x00020000);
        const unsigned rlane = ((unsigned)(kw * (32 * OWN) + 4 * (lane >> 5) + 2 * (lane & 1)) * (unsigned)N +
                                (unsigned)(nw * 32 + ((lane & 31) & ~1))) * 2u;
#pragma unroll
        for (int it = 0; it < 4 * OWN; ++it)
#pragma unroll
            for (int x = 0; x < 2; ++x)
                rres[it][x] = __builtin_amdgcn_raw_buffer_load_b32(rsR, rlane + (unsigned)(8 * it + x) * (unsigned)N * 2u, 0, 0);
    }

    fql_raw_scales zraw[2];
    if (cfg::ZPRE) {
        issue_sig(0, zraw[0]);
        issue_sig(1, zraw[1]);
    }

    // ---- fold: add the K splits' partial tiles through LDS ----
    // Row tiles are handed out in blocks: split kw finishes row tiles kw * OWN .. kw * OWN + OWN - 1 (for its
    // NW waves' channels).  All row tiles go through LDS at once where they fit, else half of them at a time: every
    // wave writes its partial tiles of the pass ([wave][tile of the pass][4 x 4 registers][64 lanes], 16 bytes per lane and access), and
    // the waves that own one of them add up the KS partials in the order of the splits (a fixed order: the result
    // is deterministic).
    if (!cfg::WREG) __builtin_amdgcn_s_waitcnt(FQL_WAIT_VM(0));   // ghost transfers have landed: the stages can be reused
    __syncthreads();
    fq_v16f fin[OWN];
    const bool owner = kw * OWN < NMT;                    // this wave finishes row tiles kw * OWN ..
#pragma unroll
    for (int i = 0; i < OWN; ++i) fin[i] = zero;
    {
        fq_v4f* fold = reinterpret_cast<fq_v4f*>(lds);
        constexpr int HALF = cfg::HALF;                   // row tiles per pass
        constexpr int PASSES = NMT / HALF;
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
#pragma unroll
            for (int t = 0; t < HALF; ++t)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const fq_v16f& a = acc[pass * HALF + t];
                    fold[((wave * HALF + t) * 4 + r4) * 64 + lane] = (fq_v4f){a[4 * r4], a[4 * r4 + 1], a[4 * r4 + 2], a[4 * r4 + 3]};
                }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                const int mt = kw * OWN + i;              // (runtime: only used for addresses)
                if (mt / HALF == pass) {
                    const int t = mt - pass * HALF;
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        fq_v4f v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int k2 = 0; k2 < KS; ++k2) v += fold[(((k2 * NW + nw) * HALF + t) * 4 + r4) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 4; ++e) fin[i][4 * r4 + e] = v[e];
                    }
                }
            }
            __syncthreads();
        }
    }

    // ---- zero point: fin += Z * gscale^T over the slice's groups, on the fp16 matrix cores ----
    // (per slice, its units under way since the start: with all groups' units fetched and applied by the workgroup that
    // finishes the tile, behind the hand-over, 200 x 4096 x 11008 took 24.4 us, 22.4 now; 128 x 4096 x 11008 20.6, 18.5; without
    // slices 1000 x 1024 x 8192 23.3, 22.5)
    if (!ZPM) {
        auto apply = [&](const fq_v4i* stage, int r, const fql_raw_scales& raw) __attribute__((always_inline)) {
#pragma unroll
            for (int ci = 0; ci < 4; ++ci) {
                if (8 * r + 2 * ci < 2 * znp) {
                    const int g0 = zgroup(r, ci);
                    const unsigned sh = ((unsigned)n * (unsigned)G + (unsigned)g0) & 3u;
                    unsigned long long w = (unsigned long long)__builtin_amdgcn_alignbyte(raw.d[ci][1], raw.d[ci][0], sh) |
                                           (unsigned long long)__builtin_amdgcn_alignbyte(raw.d[ci][2], raw.d[ci][1], sh) << 32;
                    // bytes of groups outside [sb, se) are another slice's, or another channel's
                    const int lo = sb - g0 < 0 ? 0 : sb - g0, hi = se - g0;      // lo is at most 7
                    if (hi < 8) w &= hi <= 0 ? 0ull : (1ull << (8 * hi)) - 1ull;
                    w &= ~0ull << (8 * lo);
                    fq_v4i pk;
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        const int v = (int)(x == 0 ? (unsigned)w : (unsigned)(w >> 32));
                        pk[2 * x]     = __builtin_bit_cast(int, __builtin_amdgcn_cvt_pkrtz(
                            __builtin_amdgcn_cvt_f32_fp8(v, 0), __builtin_amdgcn_cvt_f32_fp8(v, 1)));
                        pk[2 * x + 1] = __builtin_bit_cast(int, __builtin_amdgcn_cvt_pkrtz(
                            __builtin_amdgcn_cvt_f32_fp8(v, 2), __builtin_amdgcn_cvt_f32_fp8(v, 3)));
                    }
                    const fq_v4i* unit = stage + (2 * ci + hl) * cfg::BM + kw * (32 * OWN) + (lane & 31);
#pragma unroll
                    for (int i = 0; i < OWN; ++i)
                        fin[i] = FQ_MFMA_F16(__builtin_bit_cast(fql_v8h, unit[32 * i]), __builtin_bit_cast(fql_v8h, pk), fin[i]);
                }
            }
        };
        // rounds past the first two (K beyond 8192 in one slice) travel through the stages, which the fold is done with
        constexpr int PRE = cfg::ZPRE ? 2 : 0;
        auto issue_batch = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < cfg::ZBATCH; ++t)
                if (r0 + t < rounds) issue_z(lds + t * cfg::ZROUND, r0 + t);
        };
        if (PRE < rounds) issue_batch(PRE);
        if (cfg::ZPRE) {
            apply(lds + cfg::WORK_LDS / 16, 0, zraw[0]);
            if (rounds > 1) apply(lds + cfg::WORK_LDS / 16 + cfg::ZROUND, 1, zraw[1]);
        }
        for (int r0 = PRE; r0 < rounds; r0 += cfg::ZBATCH) {
            fql_raw_scales raw;
            if (r0 > PRE) issue_batch(r0);
            issue_sig(r0, raw);
            __builtin_amdgcn_s_waitcnt(FQL_WAIT_VM(0));
            __syncthreads();
            for (int t = 0; t < cfg::ZBATCH && r0 + t < rounds; ++t) {
                const fql_raw_scales cur = raw;
                if (r0 + t + 1 < rounds) issue_sig(r0 + t + 1, raw);
                apply(lds + t * cfg::ZROUND, r0 + t, cur);
            }
            __syncthreads();                              // read: LDS is free again
        }
    }

    // ---- K slices: hand the partial tile over; the workgroup that arrives last adds them up and goes on ----
    // The partial tiles and the counter are written and read with device-scope accesses (the sc1 bit: they go to
    // the level at which all XCDs agree and bypass the caches on the way back), and a wave's stores have been
    // acknowledged there (vmcnt = 0) before its workgroup counts itself in: a device-scope fence would do the same
    // by writing back the whole L2, once per workgroup, which cost more than the GEMM.  A tile's partial sums are
    // laid out [slice][wave][own row tile][4 x 4 registers][64 lanes], 16 bytes per lane and access.
    if (!ZPM && S > 1) {
        constexpr int SC1 = 16;                           // cache policy of the buffer builtins: device scope
        constexpr unsigned WAVE_BYTES = (unsigned)OWN * 4096u;
        const __amdgpu_buffer_rsrc_t rsP = __builtin_amdgcn_make_buffer_rsrc(
            partials + (size_t)tile * S * FQK_WAVES * (WAVE_BYTES / 4), 0, (int)((unsigned)S * FQK_WAVES * WAVE_BYTES), 0x00020000);
#pragma unroll
        for (int i = 0; i < OWN; ++i)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const fq_v4f v = {fin[i][4 * r4], fin[i][4 * r4 + 1], fin[i][4 * r4 + 2], fin[i][4 * r4 + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(fq_v4i, v), rsP, lane16,
                                                       (unsigned)(slice * FQK_WAVES + wave) * WAVE_BYTES + (unsigned)(i * 4 + r4) * 1024u, SC1);
            }
        __builtin_amdgcn_s_waitcnt(FQL_WAIT_VM(0));       // this wave's partial sums have arrived ...
        __syncthreads();
        unsigned* flag = reinterpret_cast<unsigned*>(lds + cfg::LDS / 16 - 1);
        if (threadIdx.x == 0)                             // ... before the workgroup counts itself in
            flag[0] = __hip_atomic_fetch_add(&counters[tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        // (one value for the whole wave, said so: else the addresses below count as each lane's own and every load becomes a loop)
        const unsigned arrived = (unsigned)__builtin_amdgcn_readfirstlane((int)*reinterpret_cast<volatile unsigned*>(flag));
        if (arrived != (unsigned)(S - 1)) return;
        if (threadIdx.x == 0)                             // every slice has counted: ready for the next call
            __hip_atomic_store(&counters[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // four slices' worth of loads are in flight at a time; the sum runs in the order of the slices
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) fin[i][r] = 0.f;
            for (int sl0 = 0; sl0 < S; sl0 += 4) {
                fq_v4f part[4][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int sl = sl0 + q < S ? sl0 + q : S - 1;       // (a repeat of the last slice, dropped below)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4)
                        part[q][r4] = __builtin_bit_cast(fq_v4f, __builtin_amdgcn_raw_buffer_load_b128(
                            rsP, lane16, (unsigned)(sl * FQK_WAVES + wave) * WAVE_BYTES + (unsigned)(i * 4 + r4) * 1024u, SC1));
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (sl0 + q < S) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) fin[i][r] += part[q][r >> 2][r & 3];
                    }
            }
        }
    }

    // ---- epilogue: per-token and per-tensor factors, the residual if any, one rounding to bf16, store ----
    float* osc = reinterpret_cast<float*>(reinterpret_cast<char*>(lds) + cfg::BM * cfg::OUT_STRIDE);
    if ((int)threadIdx.x < cfg::BM) osc[threadIdx.x] = row_scale * (tscale * 512.0f);   // x 2^9: the weights were fed in units of 2^-9
    __syncthreads();
    if (wide_rows) {
        // transpose through LDS so that every store instruction writes whole rows of the tile
        char* tile = reinterpret_cast<char*>(lds);
        char* wcol = tile + (kw * (32 * OWN) + 4 * (lane >> 5)) * cfg::OUT_STRIDE + (nw * 32 + (lane & 31)) * 2;
        const float* oscl = osc + kw * (32 * OWN) + 4 * (lane >> 5);
#pragma unroll
        for (int it = 0; it < (owner ? 4 * OWN : 0); ++it) {   // step it: rows 8 * it + 4 * (lane / 32) + 0..3 of the wave's own rows
            const int i = it >> 2, jj = it & 3;
            const fq_v4f sc4 = *reinterpret_cast<const fq_v4f*>(&oscl[8 * it]);
            fq_v4f res = {0.f, 0.f, 0.f, 0.f};
            if (add_wide) {                               // this lane's four residual values: the pair of lanes swaps halves
                const bool oddl = lane & 1;
                const unsigned d0 = rres[it][0], d1 = rres[it][1];
                const unsigned p0 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)d0, 0xB1, 0xF, 0xF, false);
                const unsigned p1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)d1, 0xB1, 0xF, 0xF, false);
                const unsigned a[4] = {oddl ? p0 : d0, oddl ? p1 : d1, oddl ? d0 : p0, oddl ? d1 : p1};
                const unsigned sh = oddl ? 0u : 16u;
#pragma unroll
                for (int e = 0; e < 4; ++e) res[e] = __uint_as_float((a[e] << sh) & 0xFFFF0000u);
            }
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                const fq_v2f pr = add_wide ? (fq_v2f){fmaf(fin[i][4 * jj + e], sc4[e], res[e]),
                                                      fmaf(fin[i][4 * jj + e + 1], sc4[e + 1], res[e + 1])}
                                           : (fq_v2f){fin[i][4 * jj + e] * sc4[e], fin[i][4 * jj + e + 1] * sc4[e + 1]};
                const unsigned pk = __builtin_bit_cast(unsigned, __builtin_convertvector(pr, fq_v2bf));
                char* dst = wcol + (8 * it + e) * cfg::OUT_STRIDE;
                *reinterpret_cast<unsigned short*>(dst) = (unsigned short)pk;
                *reinterpret_cast<unsigned short*>(dst + cfg::OUT_STRIDE) = (unsigned short)(pk >> 16);
            }
        }
        __syncthreads();                                  // (all residual reads of the tile precede all of its stores)
        constexpr int RPW = cfg::BM / FQK_WAVES, LPR = cfg::BN / 8, RPI = 64 / LPR;
        // (rows past M lie behind the descriptor's range, 16-byte steps past N get an offset out of range)
        const __amdgpu_buffer_rsrc_t rsY = __builtin_amdgcn_make_buffer_rsrc(
            Y + (size_t)m0 * N + n0, 0, (int)(((unsigned)mrows * (unsigned)N - (unsigned)n0) * 2u), 0x00020000);
        const unsigned ylane = (unsigned)(wave * RPW + lane / LPR) * (unsigned)N * 2u + (unsigned)(lane % LPR) * 16u;
        const bool col_ok = n0 + (lane % LPR) * 8 < N;
        const char* rd = tile + (wave * RPW + (lane / LPR)) * cfg::OUT_STRIDE + (lane % LPR) * 16;
#pragma unroll
        for (int j = 0; j < RPW / RPI; ++j) {
            const fq_v4i v = *reinterpret_cast<const fq_v4i*>(rd + RPI * j * cfg::OUT_STRIDE);
            __builtin_amdgcn_raw_buffer_store_b128(v, rsY, col_ok ? ylane + (unsigned)(RPI * j) * (unsigned)N * 2u : FQL_OOB, 0, 0);
        }
        return;
    }
    // rows not in 16-byte steps: element-wise, with bounds checks.  (In-place residual: an element is read and written by the
    // same lane, and nobody else touches it.)
    if (!wave_on || !n_ok || !owner) return;
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ml = kw * (32 * OWN) + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (m0 + ml < M) {
                float v = fin[i][r] * osc[ml];
                if (R) v = fmaf(fin[i][r], osc[ml], __uint_as_float((unsigned)R[(size_t)(m0 + ml) * N + n] << 16));
                const fq_v2f pr = {v, 0.f};
                const fq_v2bf pk = __builtin_convertvector(pr, fq_v2bf);
                Y[(size_t)(m0 + ml) * N + n] = __builtin_bit_cast(unsigned short, pk[0]);
            }
        }
    }
}

template <int NMT, int NW, int KS, bool ZPM = false>
void fqk_launch(const uint8_t* A, const float* a_scale, const uint8_t* wp, const uint8_t* gs, float tscale, uint16_t* Y,
                int M, int N, int K, const uint16_t* planes, const uint16_t* R, int S, unsigned* counters, float* partials,
                hipStream_t stream) {
    typedef fqk_cfg<NMT, NW, KS, ZPM> cfg;
    static fq_device_once attr_once;                      // (one per template instance)
    fq_once_per_device(attr_once, [] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fq_gemm_ksplit_kernel<NMT, NW, KS, ZPM>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, cfg::LDS);
    });
    const int tiles_m = (M + cfg::BM - 1) / cfg::BM, tiles_n = (N + cfg::BN - 1) / cfg::BN;
    const int ntiles = tiles_m * tiles_n;
    const int pm = tiles_m < 4 ? tiles_m : 4;
    const unsigned grid = (unsigned)((ntiles + FQL_XCDS - 1) / FQL_XCDS * FQL_XCDS * S);
    hipLaunchKernelGGL((fq_gemm_ksplit_kernel<NMT, NW, KS, ZPM>), dim3(grid), dim3(FQK_THREADS), cfg::LDS, stream,
                       A, a_scale, wp, gs, tscale, Y, M, N, K, tiles_m, tiles_n, pm, planes, R, S, counters, partials);
}

}  // namespace

// Which shape of this kernel, if any, serves the problem better than the large-M kernel's own tiles: 0 = none,
// 2 = 128 x 64 tiles with K quartered, 3 = 128 x 128 tiles with K halved (1 = 256 x 128 tiles is never chosen).
// A shape wins where its tiles fit one round of the compute units, the smaller one first; GEMM alone with a prepared
// workspace, large-M kernel -> 128 x 128 -> 128 x 64, us: 256 x 14336 x 4096 27.2 -> 22.9 -> 33.9 (two rounds); 700 x 4096 x 4096
// 21.9 -> 19.1 -> 28.1; 1000 x 4096 x 11008 68.4 -> 49.4 -> 67.6; 1024 x 4096 x 14336 87.6 -> 62.0 -> 84.5; 1500 x 2048 x
// 8192 39.6 -> 31.6 -> 45.3; 1000 x 2048 x 4096 19.6 -> 18.3 -> 16.2; 1000 x 1024 x 8192 34.4 -> 29.1 -> 23.3; beyond one round
// both lose (2048 x 4096 x 11008, 512 tiles: 85.5 -> 99.4; 512 x 14336 x 4096: 33.6 -> 42.9).  A single row tile with K >= 5120 is
// given two rounds of 128 x 64 tiles all the same: that line was drawn before there were 128 x 128 tiles, which would take
// these problems otherwise and in two thirds of the time: 128 x 20480 x 5120 42.3 -> 26.6 -> 40.2, 128 x 28672 x 8192
// 62.6 -> 41.9 -> 58.7, 80 x 22016 x 8192 50.9 -> 33.7 -> 46.0.
// With a short K the large-M kernel is the better one where its 128-row halves are one round too (large-M -> 128 x 128: 256
// x 11008 x 1024 9.8 -> 10.5 us, 512 x 6144 x 1024 9.7 -> 10.5, 1280 x 3000 x 1024 10.9 -> 11.1, but 200 x 8200 x 1536 11.8 -> 11.4; 256
// x 14336 x 2048 13.4 -> 14.3, x 3072 22.7 -> 18.8); two rounds of halves lose at any K (300 x 8200 x 1024 11.7 -> 10.4).
int fq_gemm_ksplit_choice(int M, int N, int K, int cus) {
    const int G = K / FQ_GROUP;
    if (M <= 64 || G < 8) return 0;
    const long long rows = (M + 127) / 128, rounds = (M <= 128 && G >= 40) ? 2 : 1;
    if (rows * ((N + 63) / 64) <= rounds * cus) return 2;
    const long long cols = (N + 127) / 128, halves = 2 * (long long)((M + 255) / 256) * cols;
    return rows * cols <= cus && (G >= 16 || halves > cus) ? 3 : 0;
}

// K slices of the 128 x 64 shape: as many as fill the compute units, each with at least two groups per K split
// of its workgroup, none of them empty, at most 8; 1 where the shape is not the 128 x 64 one or the tiles exceed
// the counters.
int fq_gemm_ksplit_slices(int choice, int M, int N, int K, int cus) {
    if (choice != 2 || M > FQ_KSPLIT_MAX_M) return 1;
    const int G = K / FQ_GROUP;
    const long long tiles = (long long)((M + 127) / 128) * ((N + 63) / 64);
    if (tiles > FQ_KSPLIT_COUNTERS) return 1;
    int S = (int)(cus / tiles);
    if (S > G / 8) S = G / 8;
    if (S > 8) S = 8;
    if (S < 1) S = 1;
    while (S > 1 && (long long)((G + S - 1) / S) * (S - 1) >= G) --S;
    return S;
}

size_t fq_gemm_ksplit_partial_bytes(int choice, int M, int N, int K, int cus) {
    const int S = fq_gemm_ksplit_slices(choice, M, N, K, cus);
    if (S <= 1) return 0;
    return (size_t)S * (size_t)((M + 127) / 128) * (size_t)((N + 63) / 64) * (128u * 64u * sizeof(float));
}

void fq_launch_gemm_ksplit(int choice, const uint8_t* A, const float* a_scale, const uint8_t* wp, const uint8_t* gs,
                           float tscale, uint16_t* Y, int M, int N, int K, void* workspace, bool prepared,
                           const uint16_t* R, hipStream_t stream) {
    if (!prepared) fq_launch_zero_point(A, workspace, M, K, stream);
    const uint16_t* planes = static_cast<const uint16_t*>(workspace);
    // behind the planes: the tiles' arrival counters (zeroed by whatever prepared the workspace), then the partial tiles
    const size_t plane_bytes = fq_gemm_plane_bytes(M, K);
    unsigned* counters = reinterpret_cast<unsigned*>(static_cast<char*>(workspace) + plane_bytes);
    float* partials = reinterpret_cast<float*>(counters + FQ_KSPLIT_COUNTERS);
    const int S = fq_gemm_ksplit_slices(choice, M, N, K, fq_device_cus());
    if (choice == 3) fqk_launch<4, 4, 2>(A, a_scale, wp, gs, tscale, Y, M, N, K, planes, R, 1, counters, partials, stream);
    else if (choice == 1) fqk_launch<8, 4, 2>(A, a_scale, wp, gs, tscale, Y, M, N, K, planes, R, 1, counters, partials, stream);
    else             fqk_launch<4, 2, 4>(A, a_scale, wp, gs, tscale, Y, M, N, K, planes, R, S, counters, partials, stream);
}

// 16 < M <= 64 without a workspace: 64 x 64 tiles, K quartered, the zero point through the matrix cores; its time hardly
// depends on M.  Against the M <= 64 kernel, M <= 64 -> this, us, at M = 64, 57, 48 and 33: 14336 x 4096 14.3 -> 13.3, 13.9 -> 13.1,
// 12.2 -> 12.7, 11.6 -> 12.3; 11008 x 4096 12.6 -> 12.2, 12.3 -> 12.0, 10.7 -> 11.7, 10.2 -> 11.4; 12288 x 2048 8.7 -> 8.3, 8.7 -> 8.2, 7.6 ->
// 8.2, 7.1 -> 8.1; 8192 x 8192 15.7 -> 18.7, 15.6 -> 18.4, 13.5 -> 17.8, 12.3 -> 17.1; 8192 x 1024 6.1 -> 6.4, 6.0 -> 6.4, 5.2 -> 6.3, 5.0 ->
// 6.2; outside the line 6144 x 4096 10.6 -> 10.4 at 64, 8.8 -> 10.2 at 48; 4096 x 4096 8.7 -> 10.2; 14336 x 11008 28.8 -> 27.0 at 64, even
// at 48.  So: the top of the range, at least half a round of tiles, K up to 8192; drawn when the M <= 64 kernel took
// 19.3 us for 64 x 8192 x 8192, the line now holds from 11008 channels on and is too low for 8192.
bool fq_gemm_ksplit64_serves(int M, int N, int K, int cus) {
    const int tiles = (N + 63) / 64;
    return M > FQ_KSPLIT64_MIN_M && M <= 64 && K / FQ_GROUP >= 8 && K <= 8192 && tiles <= cus && 2 * tiles >= cus;
}

void fq_launch_gemm_ksplit64(const uint8_t* A, const float* a_scale, const uint8_t* wp, const uint8_t* gs, float tscale,
                             uint16_t* Y, int M, int N, int K, const uint16_t* R, hipStream_t stream) {
    fqk_launch<2, 2, 4, true>(A, a_scale, wp, gs, tscale, Y, M, N, K, nullptr, R, 1, nullptr, nullptr, stream);
}
