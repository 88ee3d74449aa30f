// INT8 MatMul for many tokens: persistent workgroups that stream K steps through LDS without stopping at tile boundaries.
// Arithmetic and epilogue are those of gemm_kernel.h (W as [N,K], bias, dyadic requantization, optional residual or
// GELU, clamp); what differs is how the work is laid out in time.
//
//   * One workgroup of eight wavefronts (2 x 4; 4 x 2 on 192 columns) per CU owns a BM x BN tile at a time and walks over several tiles.
//   * A K step is 128 bytes (whole cache lines: requests of 64-byte row pieces run at half the rate, 17 against 28-32 TB/s
//     measured chip-wide).  LDS holds two steps.  A step is four phases, one per quadrant of the wavefront's tile, over its whole K:
//         1: A top x W first   (reads W second)      3: A bottom x W first   (reads A top of the next step)
//         2: A top x W second  (reads A bottom)      4: A bottom x W second  (reads W first of the next step)
//     so that no operand needs a second set of registers (96 in all), and the LDS regions fall free one after the other: A top
//     and W first of a step have been read by everybody at the barrier that ends the step before, W second and A bottom at the barrier
//     after phase 2.  Their refills -- for the step after next -- are requested in the half step after that, and are not
//     needed for two half steps more: the requests are spread evenly over all wavefronts and all of the time (32 B/clk of the
//     50 the path does), each has some 2000 cycles to arrive, and there are two barriers per step.
//     (With a step as one unit all its requests fall into the half after the barrier and take longer than the MFMAs.)
//   * The stream of steps runs on into the next tile: while the epilogue of a tile runs, the first two steps of the next
//     one arrive.  The GELU table is built once per workgroup.
//   * What bounds it: a 256x256 step takes about 2500 cycles for 2048 of MFMA (the rest is barriers and waiting for the address
//     unit), at a clock that the denser loop itself brings down (sclk read during [32768,1024] x K 4096: 1.91 GHz; 1.98 when a step took
//     2900 cycles; 3.7-4.0 POP/s is MFMA alone on random data).  What the loop issues beside the MFMAs counts: operands addressed as
//     buffers, with the step as the scalar offset, in place of 64-bit addresses with a row minimum and a test for every request: a third
//     of the scalar instructions (1.24e7 -> 4.1e6 for 8.4e6 MFMAs), us: [32768,1024] x K 4096 INT8 117.6 -> 108.9, [32768,4096] x
//     K 1024 + GELU 150.6 -> 141.5, 256x192: [32768,768] x K 3072 INT8 77.3 -> 67.7, INT16 83.5 -> 79.0, [4096,3072] x K 768 + GELU 17.9 -> 17.1.
//     (Requests of the two wavefronts of a SIMD half a slot apart, behind a branch each, gave all of it back.)
//   * With many rows it is power that bounds it: the same launches on zeros take the same cycles and 14 to 24 % less time (2.2 GHz
//     against 1.75 to 1.95; [32768,3072] x K 1024 105 -> 80 us).  A loop of nothing but the step's MFMAs sustains 4.05 POP/s on random
//     operands, with its LDS reads 3.5, with its requests 3.0 -- 1425 ns a step, about what a step takes here.
//   * An epilogue is what the address unit, then the ALU, make of it.  Rows leave and residuals come with neighbouring lanes on neighbouring
//     bytes, through LDS (see `turn`; with GELU as they are), one unit of rows at a time while the next is being made; the MFMA's first operand are
//     the rows of A, so that a lane has the same few channels for all its tokens and their constants are made once.  Cycles of a launch, thousands, with
//     lane swaps in place of LDS and stores that left together at the end / as it is: [32768,1024] x K 1024 INT16 + residual 84.0 / 73.5,
//     [32768,768] x K 768 63 / 56.5, x K 3072 133 / 125, [32768,3072] x K 1024 INT8 175 / 166, [32768,4096] x K 1024 + GELU 250 / 237; us: 45.3 /
//     41.9, 35.6 / 32.0, 76.7 / 71.3, 104 / 101, 134 / 130.  Tried and not kept: the next tile's first operands held in registers over
//     the epilogue, so that requests go on in its first half step (they queue behind the stores: 176 k -> 199 k cycles); a barrier at a tile's
//     head in place of that (equal).
//   * A 256x192 INT8 tile of K 768 took 18.8 thousand cycles (stamps): first step 2.1, five more 9.7 (7.7 of MFMA), clearing accumulators and requesting
//     constants 0.7, head of the epilogue 1.1, values and stores 2.8 for the first wavefront of a SIMD, 4.7 for the second; 256x256 + GELU 25.8: 2.5, 12.5, 1.1,
//     1.5, 6.3 / 7.6.  What stands between loop and values is gone or shorter since: the first step's MFMAs add to zero, constants are requested a
//     tile ahead (at a tile's head they stood behind the stores), the tests of the head are minima and maxima.  us: [32768,3072] x K 1024 INT8 104.5 ->
//     101.0, [32768,4096] x K 1024 + GELU 141.1 -> 137.3, [32768,768] x K 768 INT16 + residual 33.1 -> 32.4 (a card that power binds).
//   * Measured against one workgroup per tile, us, W cold, when it came: [32768,4096] x K 1024 with GELU 212 -> 142, [15311,3072] x K 768
//     with GELU 115 -> 45 (any M: tiles may be ragged), [32768,1024] x K 1024 + residual 62 -> 44.
//   * The vector registers must hold everything: with one of them spilled the loop takes 1.6 times as long, even where no scratch is
//     touched.  None is (224 at most of 256x192, 239 of 256x256): what an epilogue derives from the lane's index is made there.
//   * Rows past M (any M is allowed) are computed from zeros and not stored: operands, residual and output are addressed as buffers
//     that end with the last row.
#pragma once
#include "gemm_kernel.h"

namespace ibert {

struct StreamArgs {
    const int8_t* A;
    const int8_t* W;
    const int32_t* bias;
    const int32_t* mult;
    const int32_t* shift;
    const int8_t* R;
    void* C;
    int32_t M, nk;             // nk: K steps (K / 128)
    int32_t lda, ldw, ldc, ldr;
    int32_t tiles_m, bn;       // tile rows; tile columns of an XCD's share
    uint32_t bn_magic;         // see udiv_fix
    int32_t xs, gs;            // log2 of the shares side by side (columns) and above each other (rows): xs + gs = 3
    int32_t per_xcd;           // workgroups per XCD
    int32_t per_channel, dy_m, dy_s;
    int32_t out_clamp;
    int32_t res_m, res_s, res_fast;
    int64_t res_rnd;
    ResShort res_short;        // see residual_short
    int32_t k_fast;            // K * 127^2 < 2^30
    int32_t gelu_fast, gelu_lut_lo, gelu_lut_n;
    GeluConst gelu;
    uint32_t* path_word;
};

// Workgroups are dealt round-robin to the 8 XCDs.  XCD x works on the tile columns of share x % 2^xs and, of those tiles in
// row-major order, on the (x >> xs)-th of 2^gs runs; its workgroups take the tiles of the run in turn.
struct StreamRun {
    int first_col, first, count;   // the share's first tile column; the run's first tile, its tiles
};
__host__ __device__ __forceinline__ StreamRun stream_run(const StreamArgs& g, int x)
{
    const int group = g.tiles_m * g.bn, xm = x >> g.xs, t0 = (int)(((int64_t)xm * group) >> g.gs);
    return StreamRun{(x & ((1 << g.xs) - 1)) * g.bn, t0, (int)(((int64_t)(xm + 1) * group) >> g.gs) - t0};
}
__host__ __device__ __forceinline__ void stream_tile(const StreamArgs& g, const StreamRun& run, int l, int& tm, int& tn)
{
    const int t = run.first + l;
    tm = udiv_fix(t, g.bn, g.bn_magic);
    tn = run.first_col + t - tm * g.bn;
}

template <int BM, int BN, int NW, bool OUT_I8, bool GELU>
struct StreamLayout {
    static constexpr int STAGE = (BM + BN) * 128;
    static constexpr int PAR = 2 * STAGE;                          // two buffers of 3 x BN constants
    static constexpr int TURN = PAR + 2 * 3 * BN * 4;              // rows on their way out, see `turn` (none with GELU)
    static constexpr int TURN_WAVE = GELU ? 0 : BN % 128 == 0 ? (OUT_I8 ? 1280 : 2560) : 3584;     // bytes per wavefront
    static constexpr int LUT = TURN + NW * TURN_WAVE;
    static constexpr int ROOM = 163840 - LUT;                      // for the GELU table
};

// The channel of its wavefront's tile that lane r of 16 holds in block column i.  An MFMA block is 16 rows of W, and which ones is free: chosen
// so, a lane's channels are neighbours over the block columns: four in the first 64, two in 32 further ones.
template <int FN>
__host__ __device__ constexpr int lane_channel(int i, int r)
{
    return i < 4 ? 4 * r + i : 64 + 2 * r + (i - 4);
}

// OUT_I8: INT8 output (no residual), with GELU if GELU; else INT16 output with or without residual.
template <int BM, int BN, int NW, bool OUT_I8, bool GELU>
__global__ __launch_bounds__(64 * NW) void gemm_stream_kernel(StreamArgs g)
{
    using SL = StreamLayout<BM, BN, NW, OUT_I8, GELU>;
    static_assert(!GELU || OUT_I8, "the GELU epilogue writes INT8");
    constexpr int NT = 64 * NW, WR = BN % 128 == 0 ? 2 : 4, WC = NW / WR;     // wavefronts in WR rows of WC
    constexpr int WM = BM / WR, WN = BN / WC, FM = WM / 16, FN = WN / 16;
    constexpr int FMH = FM / 2, FN0 = FN / 4 * 2 + FN % 4, FN1 = FN - FN0;    // MFMA blocks: A top and A bottom, W first and W second
    // 1 KB requests (8 rows x 128 bytes) per wavefront and region: A top, A bottom, W first, W second
    constexpr int QA = FMH * 2 * WR / NW, QW0 = FN0 * 2 * WC / NW, QW1 = FN1 * 2 * WC / NW;
    constexpr int N0 = QA + QW0, N1 = QW1 + QA;                    // requested together: group 0 (A top, W first), group 1
    static_assert(FM % 2 == 0 && (FN == 4 || FN == 6) && FMH * 2 * WR % NW == 0 && FN0 * 2 * WC % NW == 0 && FN1 * 2 * WC % NW == 0, "tile shape");
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = wave % WR * WM, wn0 = wave / WR * WN;
    const int frow = lane & 15, fch = lane >> 4;

    // ---- the workgroup's tiles ------------------------------------------------------------------
    const StreamRun run = stream_run(g, blockIdx.x & 7);
    const int count = run.count;
    const uint32_t kbytes = (uint32_t)g.nk * 128u;                 // bytes of a row that the K steps cover
    int lt = blockIdx.x >> 3;                                      // index inside the run
    if (lt >= count) return;
    auto tile_at = [&](int l, int& m0, int& n0) {
        int tm, tn;
        stream_tile(g, run, l, tm, tn);
        m0 = tm * BM;
        n0 = tn * BN;
    };

    // ---- requests -------------------------------------------------------------------------------
    // lane l of a request brings, for row l / 8 of its 8, the chunk that the swizzle (row / 2 mod 8) puts at byte 16 l.  Request k
    // of a wavefront in a region whose wavefront tiles have nb blocks of 8 rows there: block (wave + NW k) % nb of tile
    // (wave + NW k) / nb -- its parity is the wavefront's, so the lane's chunk is the same in all of them, and the next request of
    // the region is a fixed number of rows on.
    // The operands of the tile are buffers: their descriptors hold the tile's first row and its bytes, the lanes' row offsets stay
    // the same from tile to tile, and the K step is the scalar offset.  Rows past M, and whole steps past the last tile, lie outside
    // the buffer and read as zeros, so a request is one addition for its place in LDS and the load, with no test and no minimum.
    const int r8 = lane >> 3;
    const uint32_t chunk = (uint32_t)(((lane & 7) ^ (((wave & 1) << 2) | (r8 >> 1))) << 4);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)lds;
    static_assert(FMH * 2 % NW == 0 || NW % (FMH * 2) == 0, "rows of the requests of a region at a fixed distance");
    auto first_row = [&](int nb, int rows) { return wave / nb * rows + wave % nb * 8; };
    constexpr int SA = NW / (FMH * 2) * WM, SW0 = NW / (FN0 * 2) * WN, SW1 = NW / (FN1 * 2) * WN;     // rows from request to request
    const int pa = first_row(FMH * 2, WM), pw0 = first_row(FN0 * 2, WN), pw1 = first_row(FN1 * 2, WN) + FN0 * 16;
    // Rows of W go into LDS in the order that gives every lane neighbouring channels in the end: row 16 i + q of a wavefront's
    // tile there is its channel lane_channel(i, q).
    auto w_row = [&](int p) {                                      // tile row of W that belongs in row p of the stage's W part
        const int w = p / WN, r = p - w * WN, q = (r & 8) + r8;
        return w * WN + lane_channel<FN>(r >> 4, q);
    };
    uint32_t va[2][QA];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < QA; ++q) va[h][q] = (uint32_t)(pa + h * (WM / 2) + q * SA + r8) * (uint32_t)g.lda + chunk;
    const uint32_t vw0 = (uint32_t)w_row(pw0) * (uint32_t)g.ldw + chunk, vw1 = (uint32_t)w_row(pw1) * (uint32_t)g.ldw + chunk;
    const uint32_t sw0 = (uint32_t)(SW0 * g.ldw), sw1 = (uint32_t)(SW1 * g.ldw);
    static_assert(QW0 <= 2 && QW1 <= 2, "scalar offsets of the W requests");
    v4i da, dw;                                                    // request stream: descriptors of its tile's operands
    da[3] = dw[3] = 0x00020000;                                    // (32-bit data, raw)
    uint32_t koff = 0, kinc = 128, rstage = lds0;                  // byte of its K step, bytes to the next one; stage
    int rlt = lt;
    auto buffer = [](v4i& d, const void* p, uint32_t bytes) {
        const uint64_t u = (uint64_t)(uintptr_t)p;
        d[0] = (int32_t)(uint32_t)u;
        d[1] = (int32_t)((uint32_t)(u >> 32) & 0xffffu);
        d[2] = (int32_t)bytes;
    };
    auto request_tile = [&](int l) {
        if (l < count) {
            int m0, n0;
            tile_at(l, m0, n0);
            const int rows = g.M - m0 < BM ? g.M - m0 : BM;
            buffer(da, g.A + (int64_t)m0 * g.lda, (uint32_t)rows * (uint32_t)g.lda);
            buffer(dw, g.W + (int64_t)n0 * g.ldw, (uint32_t)BN * (uint32_t)g.ldw);
            kinc = 128;
        } else {                                                   // empty buffers, for good
            da[2] = dw[2] = 0;
            kinc = 0;
        }
    };
    // request q of group h (0 or 1): the A rows first
    auto request_one = [&](int h, int q) {
        const bool is_a = q < QA;
        const int k = is_a ? q : q - QA;
        const int row = is_a ? h * (WM / 2) + k * SA : k * (h == 0 ? SW0 : SW1);
        const uint32_t place = rstage + (uint32_t)((is_a ? pa : BM + (h == 0 ? pw0 : pw1)) * 128);
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds"
                     :: "s"(place), "i"(row * 128), "v"(is_a ? va[h][is_a ? k : 0] : (h == 0 ? vw0 : vw1)), "s"(is_a ? da : dw),
                        "s"(is_a || k == 0 ? koff : koff + (h == 0 ? sw0 : sw1)) : "memory", "m0", "scc");
    };
    auto request_advance = [&]() {
        koff += kinc;
        rstage = 2 * lds0 + (uint32_t)SL::STAGE - rstage;
        if (koff == kbytes) {
            koff = 0;
            rlt += g.per_xcd;
            request_tile(rlt);
        }
    };
    // Constants of a tile's columns (bias, mult, shift: 3 x BN dwords) by DMA, 64 dwords per request, dealt round the
    // wavefronts; missing arrays are filled in by hand.
    int par_n0 = -1, par_buf = 1;
    auto request_constants = [&](int n0) {
        if (n0 == par_n0) return;
        par_n0 = n0;
        par_buf ^= 1;
        constexpr int CPA = BN / 64;
        static_assert(BN % 64 == 0, "whole requests of constants");
        const uint32_t base = lds0 + (uint32_t)(SL::PAR + par_buf * 3 * BN * 4);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int32_t* src = a == 0 ? g.bias : (a == 1 ? g.mult : g.shift);
            if (a == 0 ? g.bias != nullptr : g.per_channel != 0) {
#pragma unroll
                for (int c = 0; c < CPA; ++c)
                    if ((a * CPA + c) % NW == wave) {
                        const int32_t* sb = src + n0 + c * 64;
                        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                                     :: "s"(base + (uint32_t)((a * BN + c * 64) * 4)), "v"((uint32_t)lane * 4u), "s"(sb) : "memory", "m0");
                    }
            } else {
                int32_t* p = reinterpret_cast<int32_t*>(lds + SL::PAR + par_buf * 3 * BN * 4) + a * BN;
                int32_t fill = a == 0 ? 0 : (a == 1 ? g.dy_m : g.dy_s), c0 = tid;
                asm volatile("" : "+s"(fill), "+v"(c0));           // (made here each time: no register for them in the loop)
                for (int c = c0; c < BN; c += NT) p[c] = fill;
            }
        }
    };
    constexpr auto vm = [](int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); };

    v4i acc[FN][FM];
    // operand reads: block rows are multiples of 16, so the swizzle depends on frow only; slice sl of the step
    // (the second slice is four chunks on: the address with bit 6 flipped)
    const int rd0 = frow * 128 + ((fch ^ ((frow >> 1) & 7)) << 4);
    auto operand = [&](int sl, int off) { return *reinterpret_cast<const v4i*>(lds + off + (sl ? rd0 ^ 64 : rd0)); };
    v4i at[FMH][2], ab[FMH][2], w0[FN0][2], w1[FN1][2];
    int stage = 0;                                                 // LDS offset of the step being computed
    auto read_a = [&](v4i (&d)[FMH][2], int st, int h, int q) {    // q: block q / 2, slice q % 2
        d[q >> 1][q & 1] = operand(q & 1, st + (wm0 + (h * FMH + (q >> 1)) * 16) * 128);
    };
    auto read_w0 = [&](int st, int q) { w0[q >> 1][q & 1] = operand(q & 1, st + BM * 128 + (wn0 + (q >> 1) * 16) * 128); };
    auto read_w1 = [&](int st, int q) { w1[q >> 1][q & 1] = operand(q & 1, st + BM * 128 + (wn0 + (FN0 + (q >> 1)) * 16) * 128); };

    // ---- prologue -------------------------------------------------------------------------------
    int m0, n0;
    tile_at(lt, m0, n0);
    request_constants(n0);
    request_tile(lt);
    auto request_two_steps = [&]() {
#pragma unroll 1
        for (int st = 0; st < 2; ++st) {
#pragma unroll
            for (int q = 0; q < N0; ++q) request_one(0, q);
#pragma unroll
            for (int q = 0; q < N1; ++q) request_one(1, q);
            request_advance();
        }
    };
    request_two_steps();
    if constexpr (GELU) {
        int8_t* lut = lds + SL::LUT;
        const int32_t rnd = 1 << ((g.gelu.s - 33) & 31), sh = (g.gelu.s - 32) & 31;
        for (int e = tid; e < g.gelu_lut_n; e += NT) {
            const int32_t q = g.gelu_lut_lo + e;
            lut[e] = (int8_t)(g.gelu_fast ? gelu_one_fast(q, g.gelu, rnd, sh) : gelu_one(q, g.gelu));
        }
    }
    __builtin_amdgcn_s_waitcnt(vm(N0 + N1));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // The MFMAs of one quadrant: W blocks i0 .. i0 + NI - 1 (operands xw) by A blocks j0 .. j0 + FMH - 1 (operands xa), slice by
    // slice; `between(idx)` issues what goes in front of MFMA idx (`sched_barrier` pins that order).  A tile's first step adds to zero.
    auto quadrant = [&](auto& xw, auto ni_tag, int i0, v4i (&xa)[FMH][2], int j0, auto zero_tag, auto&& between) {
        constexpr int NI = decltype(ni_tag)::value;
        constexpr bool ZERO = decltype(zero_tag)::value;
#pragma unroll
        for (int sl = 0; sl < 2; ++sl)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < FMH; ++j) {
                    between((sl * NI + i) * FMH + j);
                    __builtin_amdgcn_sched_barrier(0);
                    acc[i0 + i][j0 + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[j][sl], xw[i][sl], ZERO && sl == 0 ? v4i{0, 0, 0, 0} : acc[i0 + i][j0 + j], 0, 0, 0);
                }
        __builtin_amdgcn_sched_barrier(0);
    };
    using NI0 = std::integral_constant<int, FN0>;
    using NI1 = std::integral_constant<int, FN1>;
    constexpr int M0 = 2 * FN0 * FMH, M1 = 2 * FN1 * FMH;          // MFMAs of the two kinds of quadrant
    static_assert(2 * FN1 <= M0 && 2 * FMH <= M1 && 2 * FMH <= M0 && 2 * FN0 <= M1, "one operand read per MFMA at most");
    // One K step.  REQ 2 is the first one of a tile.  REQ 1: each half requests its group for the step after next.  REQ 2: nothing in the first half (a wavefront may
    // still be in the epilogue of the last tile, with the first operands of this step to read), both groups in the second.
    // wait: whether the next step has to be waited for.
    auto step = [&](auto req_tag, bool wait) {
        constexpr int REQ = decltype(req_tag)::value;
        using Z = std::integral_constant<bool, REQ == 2>;
        const int nst = SL::STAGE - stage;
        // request r of n over the MFMAs [0, M0 + M1) of a half step
        auto ask = [&](int h, int n, int idx) {
#pragma unroll
            for (int r = 0; r < N0 + N1; ++r)
                if (r < n && idx == (2 * r + 1) * (M0 + M1) / (2 * n)) request_one(REQ == 2 ? (r < N0 ? 0 : 1) : h, REQ == 2 && r >= N0 ? r - N0 : r);
        };
        quadrant(w0, NI0{}, 0, at, 0, Z{}, [&](int idx) {
            if (idx < 2 * FN1) read_w1(stage, idx);
            if (REQ == 1) ask(0, N0, idx);
        });
        quadrant(w1, NI1{}, FN0, at, 0, Z{}, [&](int idx) {
            if (idx < 2 * FMH) read_a(ab, stage, 1, idx);
            if (REQ == 1) ask(0, N0, M0 + idx);
        });
        if (wait) {
            // group 0 of the next step has landed when only younger requests are outstanding: group 1 of that step and (made in
            // this half) group 0 of the one after
            __builtin_amdgcn_s_waitcnt(vm(REQ == 1 ? N1 + N0 : N1));
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        quadrant(w0, NI0{}, 0, ab, FMH, Z{}, [&](int idx) {
            if (idx < 2 * FMH) read_a(at, nst, 0, idx);
            ask(1, REQ == 2 ? N0 + N1 : N1, idx);
        });
        quadrant(w1, NI1{}, FN0, ab, FMH, Z{}, [&](int idx) {
            if (idx < 2 * FN0) read_w0(nst, idx);
            ask(1, REQ == 2 ? N0 + N1 : N1, M0 + idx);
        });
        request_advance();
        if (wait) __builtin_amdgcn_s_waitcnt(vm(N0 + N1));             // the same for its group 1
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        stage = nst;
    };

    bool first = true;
    const uint32_t lut_lds = lds0 + (uint32_t)SL::LUT;
    using R1 = std::integral_constant<int, 1>;
    using R2 = std::integral_constant<int, 2>;
    for (;;) {
#pragma unroll
        for (int q = 0; q < 2 * FMH; ++q) read_a(at, stage, 0, q);
#pragma unroll
        for (int q = 0; q < 2 * FN0; ++q) read_w0(stage, q);
        // (the first two steps of a tile that follows another were waited for before that one's stores, see below)
        step(R2{}, first);
        // The constants of the next tile, into the buffer that the tile before this one left: every epilogue waits for all that has been requested.
        // (At that tile's head they stood behind the stores: 600 cycles of every wavefront.)
        const int par_own = par_buf;
        if (lt + g.per_xcd < count) {
            int next_m0, next_n0;
            tile_at(lt + g.per_xcd, next_m0, next_n0);
            request_constants(next_n0);
        }
        for (uint32_t kt = 128; kt < kbytes; kt += 128) step(R1{}, true);

        // ---- epilogue ---------------------------------------------------------------------------
        // acc[i][j][e] = C[m0 + wm0 + 16 j + 4 u + e][n0 + wn0 + lane_channel(i, r16)]
        // (the lane's own index again: what follows from it is made here and not kept in registers through the loop)
        int el = lane;
        asm volatile("" : "+v"(el));
        const int r16 = el & 15, u = el >> 4;
        const int32_t* par = reinterpret_cast<const int32_t*>(lds + SL::PAR + par_own * 3 * BN * 4);
        // (what only the epilogue needs of the arguments is fetched here: kept in scalar registers through the loop it
        // would spill them)
        typedef const __attribute__((address_space(4))) StreamArgs* kernel_args;
#if defined(__HIP_DEVICE_COMPILE__)
        kernel_args ga = (kernel_args)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(ga));
#else
        kernel_args ga = nullptr;
#endif
        const int last = ga->M - 1 - m0;
        // Output and residual are buffers that end with the last row: lanes past it load zeros and store nothing.
        const int rows = last < BM ? last : BM - 1;                // (whole rows of them before the last one's BN columns)
        // Residual: the lane's own channels, as the stores have them.
        typedef unsigned v2u __attribute__((ext_vector_type(2)));
        typedef unsigned v3u __attribute__((ext_vector_type(3)));
        typedef unsigned v4u __attribute__((ext_vector_type(4)));
        const bool has_res = !OUT_I8 && ga->R != nullptr;
        constexpr uint32_t ES = OUT_I8 ? 1 : 2;
        // Rows between lanes and memory: 16 bytes a lane, neighbouring lanes on neighbouring bytes.  (An instruction whose neighbouring lanes
        // are in different rows takes the address unit 3.3 (stores) to 4.5 times as long: 45 against 14 cycles for 1 KB to L2, 95 against
        // 20 from it.)  A unit of 16 or 32 rows goes through the wavefront's own part of LDS, whose instructions are executed in order.
        // CP: pieces of 16 bytes in a row of the wavefront's columns; PITCH: bytes of a row there, such that the four rows of an
        // access by token (16 lanes each) fall into different banks; lane l moves pieces 64 k + l of a unit, k = 0 .. MV - 1.
        int8_t* const turn = lds + SL::TURN + wave * SL::TURN_WAVE;
        struct Rows {
            int cp, pitch, unit, mv;                               // unit: rows of blocks in it
        };
        constexpr Rows RO = OUT_I8 ? (FN == 4 ? Rows{4, 80, 1, 1} : Rows{6, 112, 2, 3}) : (FN == 4 ? Rows{8, 160, 1, 2} : Rows{12, 224, 1, 3});
        constexpr Rows RR = FN == 4 ? Rows{4, 80, 1, 1} : Rows{6, 112, 2, 3};          // residual
        static_assert(GELU || (16 * RO.unit * RO.pitch <= SL::TURN_WAVE && (OUT_I8 || 16 * RR.unit * RR.pitch <= SL::TURN_WAVE)), "place to turn rows");
        static_assert(16 * RO.unit * RO.cp == 64 * RO.mv && FM % RO.unit == 0 && FM % RR.unit == 0, "whole units");
        auto moved_row = [&](const Rows& r, int k) { return (64 * k + el) / r.cp; };
        auto moved_at = [&](const Rows& r, int k) { return moved_row(r, k) * r.pitch + (64 * k + el) % r.cp * 16; };
        auto fence = []() { __builtin_amdgcn_wave_barrier(); };
        // Residual: units of rows AHEAD of their use, as they are moved.
        constexpr int AHEAD = FN == 4 ? 4 : 2;
        v4u rt[OUT_I8 ? 1 : AHEAD][RR.mv];
        const auto rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(ga->R + (int64_t)m0 * ga->ldr + n0), 0,
                                                          has_res ? (int)((uint32_t)rows * (uint32_t)ga->ldr + BN) : 0, 0x00020000);
        auto load_residual = [&](int unit) {
#pragma unroll
            for (int k = 0; k < RR.mv; ++k)
                // (the unit's rows in the lane's offset: a scalar offset is documented as no part of the buffer's range check, so rows past M would pass it)
                rt[OUT_I8 ? 0 : unit % AHEAD][k] = __builtin_amdgcn_raw_buffer_load_b128(
                    rb, (wm0 + unit * RR.unit * 16 + moved_row(RR, k)) * ga->ldr + wn0 + (64 * k + el) % RR.cp * 16, 0, 0);
        };
        // Fast form: every shift in [33, 62], every |bias| and K * 127^2 below 2^30 (|acc + bias| stays below 2^31), the residual shift in [8, 62] (see gemm_kernel.h),
        // and a GELU table.
        bool fast, fold, tall;
        {
            // (|bias| below 2^30 or bias = -2^30: the two highest bits are equal)
            int32_t lo = par[2 * BN + el], hi = lo, pb = par[el], big = pb ^ (pb << 1);
#pragma unroll
            for (int c = 64; c < BN; c += 64) {
                const int32_t ps = par[2 * BN + c + el];
                lo = lo < ps ? lo : ps;
                hi = hi > ps ? hi : ps;
                pb = par[c + el];
                big |= pb ^ (pb << 1);
            }
            fast = __builtin_amdgcn_ballot_w64(big < 0 || lo < 33 || hi > 62) == 0 && ga->res_fast && ga->k_fast && (!GELU || ga->gelu_lut_n > 0);
            fold = __builtin_amdgcn_ballot_w64(hi > 43) == 0;
            tall = __builtin_amdgcn_ballot_w64(lo < 40) == 0;
        }
        const int32_t lut_lo = ga->gelu_lut_lo, lut_hi = ga->gelu_lut_n - 1;
        const int32_t clamp_lo = -ga->out_clamp, clamp_hi = ga->out_clamp;
        const auto cb = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(ga->C) + ((int64_t)m0 * ga->ldc + n0) * ES, 0,
                                                          (int)(((uint32_t)rows * (uint32_t)ga->ldc + BN) * ES), 0x00020000);
        if (ga->path_word && m0 == 0 && n0 == 0 && wave + el == 0)
            *ga->path_word = !fast ? IBERT_EPILOGUE_STAGED : (GELU ? IBERT_EPILOGUE_DIRECT_GELU_TABLE : IBERT_EPILOGUE_DIRECT);
        if (fast) {
            if constexpr (!OUT_I8) {
#pragma unroll
                for (int unit = 0; unit < AHEAD && unit * RR.unit < FM; ++unit) load_residual(unit);
            }
            // constants of the lane's channels: c0 = bias m + 2^(s-1) (gemm_kernel.h); `low` further bits of the value are kept
            int64_t c0[FN];
            int32_t mm[FN], sh[FN];
            auto constants = [&](int low, int32_t off, bool use_off) {
#pragma unroll
                for (int i = 0; i < FN; ++i) {
                    const int c = wn0 + lane_channel<FN>(i, r16);
                    const int32_t b = par[c], s = par[2 * BN + c];
                    mm[i] = par[BN + c];
                    c0[i] = (int64_t)b * mm[i] + ((int64_t)1 << ((s - 1) & 63));
                    if (use_off) c0[i] -= (int64_t)off << (s & 63);
                    sh[i] = (s - 32 - low) & 31;
                }
            };
            auto value = [&](int i, int n) { return (int32_t)(((int64_t)acc[i][n >> 2][n & 3] * mm[i] + c0[i]) >> 32) >> sh[i]; };
            // Token n of the lane: row 16 (n / 4) + 4 u + n % 4 of the wavefront's tile.  Its results go to LDS; when a unit is complete it is read
            // back as it is moved, and stored while the next one is being made.  Before the first store this wavefront's requests have all
            // landed (HOLD units give them time, of 256x192 INT8 and GELU tiles the first of two: with everything stored behind the last value [32768,3072] x K 1024
            // INT8 101.7 us, as it is 98.3, [15311,3072] x K 768 + GELU 44.9 / 43.2, forward of Base 32 x 128 779.1 / 771.0), so that the waits of the next tile's first step, which
            // would count stores among the loads, can be left out.
            constexpr int UNITS = FM / RO.unit, HOLD = UNITS == 2 ? 1 : UNITS >= 8 && OUT_I8 ? 4 : 2;
            constexpr bool SOON = UNITS == 2;                      // its first unit is stored four tokens into the second, when it has come back from LDS
            v4u mv[UNITS][RO.mv];
            auto store = [&](int unit) {
#pragma unroll
                for (int k = 0; k < RO.mv; ++k)
                    // (the unit's rows in the lane's offset: with a scalar offset register, and then only, the compiler puts no wait state behind
                    // a store whose registers the next instruction overwrites, and on this chip stores of 16 bytes need one there too --
                    // the last quarter of the lanes stored what came after)
                    __builtin_amdgcn_raw_buffer_store_b128(mv[unit][k], cb, ((wm0 + moved_row(RO, k)) * ga->ldc + wn0) * (int)ES + (64 * k + el) % RO.cp * 16 +
                                                                                unit * RO.unit * 16 * ga->ldc * (int)ES, 0, 0);
            };
            auto put = [&](int n, uint32_t w0, uint32_t w1, uint32_t w2) {     // INT8: w0 and half of w2; INT16: w0, w1 and w2
                int8_t* const row = turn + (16 * (n / 4 % RO.unit) + 4 * u + n % 4) * RO.pitch;
                if (n % (4 * RO.unit) == 0) fence();
                if constexpr (OUT_I8) {
                    *reinterpret_cast<uint32_t*>(row + 4 * r16) = w0;
                    if (FN == 6) *reinterpret_cast<uint16_t*>(row + 64 + 2 * r16) = (uint16_t)w2;
                } else {
                    *reinterpret_cast<v2u*>(row + 8 * r16) = v2u{w0, w1};
                    if (FN == 6) *reinterpret_cast<uint32_t*>(row + 128 + 4 * r16) = w2;
                }
                if ((n + 1) % (4 * RO.unit) == 0) {
                    const int unit = n / (4 * RO.unit);
                    fence();
#pragma unroll
                    for (int k = 0; k < RO.mv; ++k) mv[unit][k] = *reinterpret_cast<const v4u*>(turn + moved_at(RO, k));
                    if (unit + 1 == HOLD) __builtin_amdgcn_s_waitcnt(vm(0));
#pragma unroll
                    for (int x = unit + 1 == HOLD ? 0 : unit - 1; x < unit; ++x)
                        if (unit + 1 >= HOLD && !SOON) store(x);
                }
                if (SOON && n == 4 * RO.unit + 3) store(0);
            };
            using T = std::true_type;
            using F = std::false_type;
            constexpr int TOKENS = 4 * FM;
            if constexpr (GELU) {
                // Table reads stay outstanding while the next values are made: a token is packed LAG tokens after its reads were
                // issued.  FOLD: the table's address is folded into the requantization constant (gemm_kernel.h)
                constexpr int LAG = 12 / FN;                       // (a wait can leave at most 15 reads outstanding)
                const int32_t lo = (int32_t)lut_lds;
                int32_t by[TOKENS][FN];
                // Tokens are stored as they are packed, four bytes a lane (and two): neighbouring lanes are on neighbouring bytes of four rows as it
                // is.  With the rows turned in LDS first the time was the same ([32768,4096] x K 1024 131.8 / 131.1 us, [4096,3072] x K 768 16.4 / 16.3),
                // and what that takes of LDS is room of the table: one of 20 thousand entries found none on 256x256 then, 140 -> 282 us.
                constexpr int HELD = HOLD * 4 * RO.unit;           // (tokens, see HOLD)
                uint32_t w4[TOKENS], w2[TOKENS];
                const int corner = (wm0 + 4 * u) * ga->ldc + wn0;
                auto store_token = [&](int n) {
                    const int at = corner + (16 * (n / 4) + n % 4) * ga->ldc;
                    __builtin_amdgcn_raw_buffer_store_b32(w4[n], cb, at + 4 * r16, 0, 0);
                    if (FN == 6) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)w2[n], cb, at + 64 + 2 * r16, 0, 0);
                };
                auto pack = [&](int n) {
                    w4[n] = pack4_perm(by[n][0], by[n][1], by[n][2], by[n][3]);
                    w2[n] = FN == 6 ? __builtin_amdgcn_perm(by[n][FN - 1], by[n][FN - 2], 0x0c0c0400u) : 0u;
                    if (n + 1 == HELD) __builtin_amdgcn_s_waitcnt(vm(0));
#pragma unroll
                    for (int x = n + 1 == HELD ? 0 : n; x <= n; ++x)
                        if (n + 1 >= HELD) store_token(x);
                };
                auto finish = [&](auto fold_tag) {
                    constexpr bool FOLD = decltype(fold_tag)::value;
                    typedef const __attribute__((address_space(3))) uint8_t* lds_bytes;
                    constants(0, lut_lo - lo, FOLD);
#pragma unroll
                    for (int n = 0; n < TOKENS; ++n) {
#pragma unroll
                        for (int i = 0; i < FN; ++i) by[n][i] = *(lds_bytes)(uintptr_t)(uint32_t)med3_i32(FOLD ? value(i, n) : value(i, n) - (lut_lo - lo), lo, lo + lut_hi);
                        if (n >= LAG) pack(n - LAG);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int n = TOKENS - LAG; n < TOKENS; ++n) pack(n);
                };
                if (fold) finish(T{}); else finish(F{});
            } else if constexpr (OUT_I8) {
                // TALL, every shift at least 40: shifted by eight less, a value keeps its fraction in the low byte of 16 bits, where
                // packing two of them saturates to [-128, 128): what is left of the clamp to +-127 is half an instruction a value.
                auto finish = [&](auto tall_tag) {
                    constexpr bool TALL = decltype(tall_tag)::value;
                    constants(TALL ? 8 : 0, 0, false);
#pragma unroll
                    for (int n = 0; n < TOKENS; ++n) {
                        int32_t o[FN];
#pragma unroll
                        for (int i = 0; i < FN; ++i) o[i] = value(i, n);
                        if constexpr (TALL) {
                            const uint32_t a = pack2_i16_above(o[0], o[1], -127 * 256), b = pack2_i16_above(o[2], o[3], -127 * 256);
                            const uint32_t c = FN == 6 ? pack2_i16_above(o[FN - 2], o[FN - 1], -127 * 256) : 0u;
                            put(n, __builtin_amdgcn_perm(b, a, 0x07050301u), 0u, __builtin_amdgcn_perm(c, c, 0x0c0c0301u));
                        } else {
#pragma unroll
                            for (int i = 0; i < FN; ++i) o[i] = med3_i32(o[i], clamp_lo, clamp_hi);
                            put(n, pack4_perm(o[0], o[1], o[2], o[3]), 0u, __builtin_amdgcn_perm((uint32_t)o[FN - 1], (uint32_t)o[FN - 2], 0x0c0c0400u));
                        }
                        if (n % 2 == 1) __builtin_amdgcn_sched_barrier(0);     // (bounds the live registers)
                    }
                };
                if (tall && clamp_hi == 127) finish(T{}); else finish(F{});
            } else {
                // SHORT: the residual's product fits 32 bits (residual_short) and the clamp is that of the type.  (No residual: zeros.)
                auto finish = [&](auto short_tag) {
                    constexpr bool SHORT = decltype(short_tag)::value;
                    const int32_t r_m = ga->res_short.m, r_rnd = ga->res_short.rnd, r_s = ga->res_short.s;
                    constants(0, 0, false);
#pragma unroll
                    for (int n0_ = 0; n0_ < TOKENS; n0_ += 4 * RR.unit) {
                        uint32_t r4[4 * RR.unit], r2[4 * RR.unit];
                        const int ru = n0_ / (4 * RR.unit);
                        fence();
#pragma unroll
                        for (int k = 0; k < RR.mv; ++k) *reinterpret_cast<v4u*>(turn + moved_at(RR, k)) = rt[ru % AHEAD][k];
                        fence();
#pragma unroll
                        for (int t = 0; t < 4 * RR.unit; ++t) {
                            const int8_t* row = turn + (16 * (t / 4) + 4 * u + t % 4) * RR.pitch;
                            r4[t] = *reinterpret_cast<const uint32_t*>(row + 4 * r16);
                            r2[t] = FN == 6 ? *reinterpret_cast<const uint16_t*>(row + 64 + 2 * r16) : 0u;
                        }
                        if ((ru + AHEAD) * RR.unit < FM) load_residual(ru + AHEAD);
#pragma unroll
                        for (int t = 0; t < 4 * RR.unit; ++t) {
                            const int n = n0_ + t;
                            int32_t o[FN];
                            uint32_t w[3] = {0u, 0u, 0u};
#pragma unroll
                            for (int i = 0; i < FN; ++i) {
                                o[i] = value(i, n);
                                const int32_t r8 = (int32_t)(int8_t)((i < 4 ? r4[t] : r2[t]) >> (8 * (i & 3)));
                                if (SHORT) o[i] += smad24(r8, r_m, r_rnd) >> r_s;
                                else o[i] = med3_i32(o[i] + (int32_t)(((int64_t)r8 * ga->res_m + ga->res_rnd) >> ga->res_s), clamp_lo, clamp_hi);
                            }
#pragma unroll
                            for (int i = 0; i < FN; i += 2)
                                w[i >> 1] = SHORT ? pack2_i16_above(o[i], o[i + 1], -32767) : __builtin_amdgcn_perm((uint32_t)o[i + 1], (uint32_t)o[i], 0x05040100u);
                            put(n, w[0], w[1], w[2]);
                            if (n % 2 == 1 || !SHORT) __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                };
                if (ga->res_short.ok && clamp_hi == 32767) finish(T{}); else finish(F{});
            }
            if constexpr (!GELU) store(UNITS - 1);
        } else {
            // Any constants: 64-bit arithmetic in a rolled loop, 16 rows of each row of wavefronts at a time through LDS, where the
            // next tile's first steps had arrived -- they are requested again afterwards.  (Unrolled over the accumulators like
            // the fast form this costs so many registers that the kernel needs scratch memory, and then its main loop takes
            // half as long again even where no scratch is touched: 25.8 k -> 39 k cycles for 8 steps.)
            constexpr int SP = BN + 4, G4 = BN / 4;
            int32_t* const st = reinterpret_cast<int32_t*>(lds);
            __builtin_amdgcn_s_waitcnt(vm(0));
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll 1
            for (int j = 0; j < FM; ++j) {
#pragma unroll
                for (int k = 0; k < FM; ++k)
                    if (k == j) {
#pragma unroll
                        for (int i = 0; i < FN; ++i)
#pragma unroll
                            for (int e = 0; e < 4; ++e) st[(wave % WR * 16 + 4 * u + e) * SP + wn0 + 16 * i + r16] = acc[i][k][e];
                    }
                __syncthreads();
#pragma unroll 1
                for (int q = wave * 64 + el; q < 16 * WR * G4; q += NT) {
                    const int r = q / G4, c = (q - r * G4) * 4, row = (r >> 4) * WM + 16 * j + (r & 15);
                    if (row > last) continue;
                    // (columns by block column: four channels are 16 apart, two pairs of the last 32 a pair and the next)
                    const int cw = c % WN, c0 = cw < 64 ? c - cw + cw / 4 : c - cw + 64 + (cw - 64) / 2;
                    v4i a4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) a4[e] = st[r * SP + c0 + (cw < 64 ? 16 * e : 16 * (e & 1) + (e >> 1))];
                    uint32_t r4 = 0;
                    if (has_res) r4 = *reinterpret_cast<const uint32_t*>(ga->R + (int64_t)(m0 + row) * ga->ldr + n0 + c);
                    int32_t o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        int64_t v = dyadic64((int32_t)((uint32_t)a4[e] + (uint32_t)par[c + e]), par[BN + c + e], par[2 * BN + c + e] & 63);
                        if (has_res) v += dyadic64((int32_t)(int8_t)(r4 >> (8 * e)), ga->res_m, ga->res_s);
                        o[e] = clamp_i64_to_i32(v, ga->out_clamp);
                        if constexpr (GELU) o[e] = gelu_one(o[e], GeluConst{ga->gelu.q_b, ga->gelu.q_c, ga->gelu.q_1, ga->gelu.q_max, ga->gelu.m, ga->gelu.s});
                    }
                    char* const cp = reinterpret_cast<char*>(ga->C) + ((int64_t)(m0 + row) * ga->ldc + n0 + c) * ES;
                    if constexpr (OUT_I8) *reinterpret_cast<uint32_t*>(cp) = pack4_i8(o[0], o[1], o[2], o[3]);
                    else *reinterpret_cast<uint2*>(cp) = uint2{__builtin_amdgcn_perm((uint32_t)o[1], (uint32_t)o[0], 0x05040100u),
                                                               __builtin_amdgcn_perm((uint32_t)o[3], (uint32_t)o[2], 0x05040100u)};
                }
                __syncthreads();
            }
            rlt = lt + g.per_xcd;
            koff = 0;
            rstage = lds0 + (uint32_t)stage;
            request_tile(rlt);
            request_two_steps();
            __builtin_amdgcn_s_waitcnt(vm(0));
            asm volatile("s_barrier" ::: "memory");
        }
        lt += g.per_xcd;
        if (lt >= count) break;
        tile_at(lt, m0, n0);
        first = false;
    }
}

// Does the kernel serve this problem (g as filled by launch_gemm)?
template <int BM, int BN, int NW>
bool stream_ok(const GemmArgs& g, bool i8)
{
    const bool c_ok = i8 ? g.c_vec16 : (g.c16 && aligned(g.C, 16) && g.ldc % 8 == 0);
    return g.nbatch == 1 && g.M >= 1 && g.N % BN == 0 && g.K % 128 == 0 && g.lda < (1 << 20) && g.ldw < (1 << 20) && g.ldc < (1 << 20) &&
           c_ok && (i8 ? !g.R : (!g.R || (g.r_vec && g.ldr < (1 << 20)))) && (int64_t)((g.M + BM - 1) / BM) * (g.N / BN) < (1 << 26);
}

// An XCD reads its share of W again for every round of tiles: shares side by side until one is at most half of its 4 MB
// L2 (each further one doubles the reads of A).  log2 of their number.
inline int stream_shares(const GemmArgs& g, int tiles_m, int tiles_n)
{
    int xs = 0;
    while (xs < 2 && tiles_n % (2 << xs) == 0 && (((int64_t)g.N * g.K) >> xs) > (2 << 20) && tiles_m >= (8 >> xs)) ++xs;
    return xs;
}

// Deals the tiles of a problem.
inline void stream_deal(StreamArgs& s, const GemmArgs& g, int bm, int bn)
{
    s.tiles_m = (g.M + bm - 1) / bm;
    const int tiles_n = g.N / bn;
    s.xs = stream_shares(g, s.tiles_m, tiles_n);
    s.gs = 3 - s.xs;
    s.bn = tiles_n >> s.xs;
    s.bn_magic = udiv_magic(s.bn);
    const int64_t run = ((int64_t)s.tiles_m * s.bn + (1 << s.gs) - 1) >> s.gs;      // the longest run of an XCD
    s.per_xcd = (int32_t)(run < 32 ? run : 32);                    // one workgroup per CU
}

template <int BM, int BN, int NW, bool GELU>
int launch_stream(GemmArgs& g, bool i8, hipStream_t stream)
{
    if (!stream_ok<BM, BN, NW>(g, i8) || (GELU && !i8)) return IBERT_ERR_NOT_IMPLEMENTED;
    StreamArgs s;
    s.A = g.A; s.W = g.W; s.bias = g.bias; s.mult = g.mult; s.shift = g.shift; s.R = g.R; s.C = g.C;
    s.M = g.M; s.nk = g.K / 128;
    s.lda = (int32_t)g.lda; s.ldw = (int32_t)g.ldw; s.ldc = (int32_t)g.ldc; s.ldr = (int32_t)g.ldr;
    stream_deal(s, g, BM, BN);
    s.per_channel = g.per_channel; s.dy_m = g.dy_m; s.dy_s = g.dy_s; s.out_clamp = g.out_clamp;
    s.res_m = g.res_m; s.res_s = g.res_s; s.res_fast = g.res_fast; s.res_rnd = g.res_rnd;
    s.res_short = g.c16 && g.out_clamp == 32767 ? residual_short(g) : ResShort{0, 0, 0, 0};
    s.k_fast = (int64_t)g.K * 16129 < (1 << 30);
    s.gelu_fast = g.gelu_fast; s.gelu_lut_lo = g.gelu_lut_lo; s.gelu_lut_n = 0; s.gelu = g.gelu;
    s.path_word = g.path_word;
    const dim3 grid(8u * (unsigned)s.per_xcd), block(64 * NW);
#define IBERT_STREAM_LAUNCH(I8_)                                                                                    \
    do {                                                                                                            \
        using SL = StreamLayout<BM, BN, NW, I8_, GELU && I8_>;                                                      \
        size_t lds_bytes = SL::LUT;                                                                                 \
        if (GELU && g.gelu_lut_n <= SL::ROOM) {                                                                     \
            s.gelu_lut_n = g.gelu_lut_n;                                                                            \
            lds_bytes += (size_t)g.gelu_lut_n;                                                                      \
        }                                                                                                           \
        auto kern = gemm_stream_kernel<BM, BN, NW, I8_, GELU && I8_>;                                               \
        static bool attr_done = false;                                                                              \
        if (!attr_done) {                                                                                           \
            IBERT_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 163840));               \
            attr_done = true;                                                                                       \
        }                                                                                                           \
        hipLaunchKernelGGL(kern, grid, block, lds_bytes, stream, s);                                                \
    } while (0)
    if constexpr (GELU) IBERT_STREAM_LAUNCH(true);
    else if (i8) IBERT_STREAM_LAUNCH(true);
    else IBERT_STREAM_LAUNCH(false);
#undef IBERT_STREAM_LAUNCH
    IBERT_LAUNCH_CHECK("gemm_stream_kernel");
    static const KernelName names[2] = {{"gemm_stream_kernel<%d, %d, %d, %s, %s>", BM, BN, NW, "false", GELU ? "true" : "false"},
                                        {"gemm_stream_kernel<%d, %d, %d, %s, %s>", BM, BN, NW, "true", GELU ? "true" : "false"}};
    g_last_kernel = names[i8 ? 1 : 0].text;
    return IBERT_OK;
}

}  // namespace ibert
