// Steps 1 to 4 of an encoder layer in one kernel: the QKV projection of one head of one sequence (INT8 MatMul, bias, per-channel requantization to
// INT8; App. C.1) and that head's attention (Fig. 1 right; Alg. 3), bit-identical to ibert_gemm_i8_requant followed by ibert_attention_i.  Q, K and V of the
// head never leave the compute unit, unless the caller wants them.
//
// Shape: head width 64, up to 256 tokens a sequence, a hidden width of whole K steps (128), parameters that the attention has a table of the exponent for.  A
// workgroup of eight or sixteen wavefronts multiplies the rows of one sequence, or of two or four short ones, by the head's 64 rows of each of W_q, W_k and W_v: a tile of 32 to
// 256 rows x 192, rows past the end of a sequence read from its last one, 16 FM x 48 a wavefront.
//   * K steps of 128 bytes go from global memory straight into a ring of STAGES stages of LDS.  A step is two phases of MFMAs, each of which reads the operands of the
//     next one and, the second, requests a later step; one barrier.  With two stages and eight wavefronts two workgroups share a compute unit (80 KB each).
//   * Sums start at the bias.  After the loop the stages make room for what the attention reads: Q, K_h and V_h as rows of 64 bytes, swizzled as attention.hip has
//     them, the table of the exponent, and the multipliers and shifts of the 192 channels.
//   * What bounds it: with two workgroups on a unit the path from L2 while they multiply (40 KB a step in 1600 to 1700 cycles for the two, 50 B/clk), then vector ALU issue.  Cycles,
//     thousands, 128 rows, K 768, one workgroup on a unit / two: first step there 3.7 / 3.7, five more 6.9 / 7.1 to 9, requantization 2.4 / 3.3, attention 4.2 / 5.0 of 20 / 24 to 30.
//     Launched apart the two kernels took those cycles, a launch (1.7 us), Q, K, V out and in, and two heads and tails.  Forwards, us: Base b32 811.6 -> 771.3, b8 s61 419.9 -> 410.7, Large
//     32 x 128 2108 -> 1938; one layer of 256 channels, 4 heads, called by itself 26.4 -> 23.3.
//   * Tried and not kept: all operands of a step read before its MFMAs (a barrier more, reads and MFMAs one after the other: 1600 cycles a step by itself, 1340 as it is); requests by
//     half of the wavefronts in front of the MFMAs and by the other half behind them (the same); wave priorities, workgroups of a unit out of step by a sleep (the same);
//     sixteen wavefronts on two sequences of 128 (equal on one round of tiles, 2 to 4 % behind on more).
#include <type_traits>

#include "attention_core.h"
#include "ibert_testing.h"

namespace ibert {

struct QkvAttentionArgs {
    AttentionArgs att;             // (first: see read_ahead; qkv, qblks and one_buffer are not used)
    const int8_t* x;               // [batch * seq, K]
    const int8_t* w;               // [3 K, K]: W_q, W_k, W_v
    const int32_t* bias;
    const int32_t* mult;
    const int32_t* shift;
    int8_t* qkv;                   // optional: Q | K | V as the MatMul by itself would store them, [batch * seq, 3 K]
    int32_t batch, nk;             // nk: K steps (K / 128)
    int32_t xs, cols, groups;      // see qkv_attention_place
    uint32_t cols_magic;           // see udiv_fix
};

constexpr int QA_COLS = 192;

// The (group of sequences, head) of a workgroup; false: there is none.  Workgroups go round the XCDs.  XCD x has the heads of share x % 2^xs, `cols` of them, and of
// the groups with these heads behind each other the (x >> xs)-th of 2^(3 - xs) runs.
__host__ __device__ __forceinline__ bool qkv_attention_place(const QkvAttentionArgs& g, unsigned block, int& group, int& h)
{
    const int x = block & 7, part = x >> g.xs, gs = 3 - g.xs, all = g.groups * g.cols;
    const int first = (int)(((int64_t)part * all) >> gs), end = (int)(((int64_t)(part + 1) * all) >> gs), at = first + (int)(block >> 3);
    group = udiv_fix(at, g.cols, g.cols_magic);
    h = (x & ((1 << g.xs) - 1)) * g.cols + at - group * g.cols;
    return at < end;
}

// NW wavefronts in NW / 4 rows of four, 16 FM x 48 each; SEQS sequences in SEG rows each.
template <int NW, int FM, int SEQS>
struct QkvLayout {
    static constexpr int ROWS = 4 * FM * NW, SEG = ROWS / SEQS, NKB = (SEG + 63) / 64, STAGE = (ROWS + QA_COLS) * 128;
    static constexpr int KEYS = ROWS - SEG + 64 * NKB;             // rows of K and V that the last sequence's key blocks end in
    static constexpr int Q = 0, K = ROWS * 64, V = K + KEYS * 64, MADE = V + KEYS * 64, TABLE = MADE + QA_COLS * 8 + 64;
};

template <int NW, int FM, int SEQS, int FORM, int STAGES>
__global__ __launch_bounds__(64 * NW, 4) void qkv_attention_kernel(QkvAttentionArgs g)
{
    using QL = QkvLayout<NW, FM, SEQS>;
    static_assert(SEQS == 1 || QL::SEG == 32 || QL::SEG % 64 == 0, "sequences of whole halves of a key block");
    constexpr int FN = 3;                                          // MFMA blocks of a wavefront: FM x FN
    constexpr int NB = (QA_COLS + QL::ROWS) / 8, NQ = (NB + NW - 1) / NW;     // 1 KB requests (8 rows of 128 bytes) of a step, and of a wavefront
    constexpr int REST = NB % NW;                                  // so many wavefronts make NQ, if not all do
    const AttentionArgs& a = g.att;
    extern __shared__ __attribute__((aligned(16))) int8_t qa_lds[];
    // every argument is in registers from here on: one trip to memory, not one at each first use
    asm volatile("" :: "s"(a.ctx), "s"(a.heads), "s"(a.seq), "s"(a.blocks), "s"(a.ld_ctx), "s"(a.s_m), "s"(a.s_s), "s"(a.c_m), "s"(a.c_s),
                 "s"(a.sm.q_b), "s"(a.sm.q_c), "s"(a.sm.q_ln2), "s"(a.sm.k), "s"(a.t.top), "s"(a.t.below), "s"(a.t.shift), "s"(a.key_lens),
                 "s"(g.x), "s"(g.w), "s"(g.bias), "s"(g.mult), "s"(g.shift), "s"(g.qkv), "s"(g.nk), "s"(g.xs), "s"(g.cols), "s"(g.groups), "s"(g.cols_magic), "s"(g.batch));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)qa_lds;
    if (__builtin_expect((int)blockIdx.x >= a.blocks, 0)) {
        read_ahead<NW, false>(lds0, wave, lane, (int)blockIdx.x - a.blocks);
        return;
    }
    int group, h;
    if (!qkv_attention_place(g, blockIdx.x, group, h)) return;
    const int b0 = group * SEQS;                                   // the first sequence
    const int L = a.seq, hidden = a.heads * ATT_DH, nk = g.nk;
    const int seqs = SEQS == 1 || g.batch - b0 < SEQS ? (SEQS == 1 ? 1 : g.batch - b0) : SEQS;

    // The thread's channel, and the lane's twelve: their constants are on their way before the tiles are.  Sums start at the bias.
    const int frow = lane & 15, fch = lane >> 4;
    const int wr = wave % (NW / 4) * 16 * FM, wc = wave / (NW / 4) * 48;      // the wavefront's first row and column of the tile
    const bool maker = tid < QA_COLS;
    int32_t c_m = 0, c_s = 63;
    if (maker) {
        const int channel = (tid >> 6) * hidden + h * ATT_DH + lane;
        c_m = g.mult[channel];
        c_s = g.shift[channel];
    }
    typedef int32_t v4i_any __attribute__((ext_vector_type(4), aligned(4)));
    v4i acc[FN][FM];
    int32_t big = 0;                                               // negative: a bias outside [-2^30, 2^30)
#pragma unroll
    for (int i = 0; i < FN; ++i) {
        const int col = wc + 16 * i;
        const v4i c = *reinterpret_cast<const v4i_any*>(g.bias + (col >> 6) * hidden + h * ATT_DH + (col & 63) + 4 * fch);
#pragma unroll
        for (int e = 0; e < 4; ++e) big |= c[e] ^ (c[e] << 1);
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = c;
    }

    // ---- requests ------------------------------------------------------------------------------
    // Blocks of 8 rows: 24 of W (the head's 64 rows of each of the three matrices), then those of x; request i of a wavefront is block NW i + wave.
    // The sequences' rows and the head's are buffers: the K step, and which of the three matrices, is the scalar offset.
    const int r8 = lane >> 3;
    const uint32_t chunk = (uint32_t)(((lane & 7) ^ (((wave & 1) << 2) | (r8 >> 1))) << 4);
    const uint32_t K = (uint32_t)nk * 128u;
    auto buffer = [](const int8_t* p, uint32_t bytes) {
        const uint64_t u = (uint64_t)(uintptr_t)p;
        return v4i{__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)u), __builtin_amdgcn_readfirstlane((int32_t)((uint32_t)(u >> 32) & 0xffffu)), (int32_t)bytes, 0x00020000};
    };
    const v4i dx = buffer(g.x + (int64_t)b0 * L * K, (uint32_t)(seqs * L) * K), dw = buffer(g.w + (int64_t)h * ATT_DH * K, (uint32_t)(2 * hidden + ATT_DH) * K);
    uint32_t vo[NQ], so[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int q = NW * i + wave;
        if (q < 24) {
            vo[i] = (uint32_t)((q & 7) * 8 + r8) * K + chunk;
            so[i] = (uint32_t)((q >> 3) * hidden) * K;
        } else {
            const int t = (q - 24) * 8 + r8;                       // row of the tile: row r of sequence s of the group
            int s = SEQS == 1 ? 0 : t / QL::SEG, r = t - s * QL::SEG;
            s = s < seqs ? s : seqs - 1;
            r = r < L ? r : L - 1;
            vo[i] = (uint32_t)(s * L + r) * K + chunk;
            so[i] = 0;
        }
    }
    auto request_one = [&](int i, int step, int st) {
        if (REST != 0 && i == NQ - 1 && wave >= REST) return;
        const bool w = NW * (i + 1) <= 24 || (NW * i < 24 && NW * i + wave < 24);
        v4i d;
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = w ? dw[e] : dx[e];
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(lds0 + (uint32_t)(st * QL::STAGE + wave * 1024 + NW * i * 1024)), "v"(vo[i]), "s"(d), "s"(so[i] + (uint32_t)step * 128u) : "memory", "m0");
    };
    auto request = [&](int step, int st) {
#pragma unroll
        for (int i = 0; i < NQ; ++i) request_one(i, step, st);
    };
    constexpr auto vm = [](int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); };
    auto landed = [&](auto younger_tag) {                          // all but the requests of so many younger steps
        constexpr int Y = decltype(younger_tag)::value;
        if (Y > 0 && REST != 0 && wave >= REST) __builtin_amdgcn_s_waitcnt(vm(Y * (NQ - 1)));
        else __builtin_amdgcn_s_waitcnt(vm(Y * NQ));
    };
#pragma unroll
    for (int st = 0; st < STAGES; ++st)
        if (st < nk) request(st, st);

    // ---- Q, K, V -------------------------------------------------------------------------------
    // A step is two phases, one for each 64 of its 128 bytes; each multiplies what the one before has read.  At the barrier between them the stage has been
    // read and the next step has landed.
    const int rd = frow * 128 + ((fch ^ ((frow >> 1) & 7)) << 4);
    v4i xf[2][FM], wf[2][FN];
    auto read_one = [&](int q, int st, int s) {
        const int8_t* const base = qa_lds + st * QL::STAGE + (s ? rd ^ 64 : rd);
        if (q < FM) xf[s][q] = *reinterpret_cast<const v4i*>(base + (QA_COLS + wr + 16 * q) * 128);
        else wf[s][q - FM] = *reinterpret_cast<const v4i*>(base + (wc + 16 * (q - FM)) * 128);
    };
    // MFMAs of one half of a step; `between(idx)` issues what goes in front of MFMA idx
    auto phase = [&](auto half_tag, auto&& between) {
        constexpr int s = decltype(half_tag)::value;
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j) {
                between(i * FM + j);
                __builtin_amdgcn_sched_barrier(0);
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[s][i], xf[s][j], acc[i][j], 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int NR = FM + FN, NM = FM * FN;                      // operand reads and MFMAs of a phase
    auto wait_for = [&](int younger) {
        if (younger <= 0) landed(std::integral_constant<int, 0>{});
        else if (younger == 1) landed(std::integral_constant<int, 1>{});
        else if (younger == 2) landed(std::integral_constant<int, 2>{});
        else landed(std::integral_constant<int, 3>{});
    };
    wait_for((nk < STAGES ? nk : STAGES) - 1);
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int q = 0; q < NR; ++q) read_one(q, 0, 0);
    int st = 0;
    for (int k = 0; k < nk; ++k) {
        const int nst = st + 1 == STAGES ? 0 : st + 1;
        phase(std::integral_constant<int, 0>{}, [&](int idx) {
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (idx == q * NM / NR) read_one(q, st, 1);
        });
        // step k + 1 has landed when only the steps behind it are outstanding: k + 2 .. k + STAGES - 1
        if (k + 1 < nk) wait_for((nk - 1 < k + STAGES - 1 ? nk - 1 : k + STAGES - 1) - (k + 1));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // (the reads behind the last step fetch stale bytes that nothing uses)
        phase(std::integral_constant<int, 1>{}, [&](int idx) {
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (idx == q * NM / NR) read_one(q, nst, 0);
            if (k + STAGES < nk) {
#pragma unroll
                for (int i = 0; i < NQ; ++i)
                    if (idx == (2 * i + 1) * NM / (2 * NQ)) request_one(i, k + STAGES, st);
            }
        });
        st = nst;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- requantization into LDS ---------------------------------------------------------------
    // A wavefront's columns are of two matrices at most; their multipliers and shifts go to LDS, and how they can be computed with as the least of both.
    // FAST (gemm_kernel.h): every shift in [33, 62], every |bias| below 2^30: |sum| is below 2^31, as K * 128^2 is below 2^30 too.  TALL: and every shift at least 40, which those of
    // these matrices mostly are.  With w = floor(sum m / 2^(s - 8)), the high half of a product shifted, the result is floor((w + 128) / 256): 16 bits of w hold all that the clamp
    // leaves, so packing two saturates, the 128 is added to both (saturating) and the high bytes are the result: 3.75 instructions a value, with a 64-bit
    // multiply-add 4.75 slots.
    enum { SLOW, FAST, TALL };
    int32_t* const par = reinterpret_cast<int32_t*>(qa_lds + QL::MADE);        // multipliers, shifts; three modes
    if (maker) {
        par[tid] = c_m;
        par[QA_COLS + tid] = c_s;
        const int mode = __builtin_amdgcn_ballot_w64(c_s < 33 || c_s > 62) != 0 ? SLOW : (__builtin_amdgcn_ballot_w64(c_s < 40) != 0 ? FAST : TALL);
        if (lane == 0) par[2 * QA_COLS + wave] = mode;
    }
    make_exp_table(a, lds0 + QL::TABLE, tid, 64 * NW);
    __syncthreads();
    const int m0 = par[2 * QA_COLS + (wc >> 6)], m1 = par[2 * QA_COLS + ((wc + 32) >> 6)];
    const int mode = __builtin_amdgcn_ballot_w64(big < 0) != 0 ? (int)SLOW : __builtin_amdgcn_readfirstlane(m0 < m1 ? m0 : m1);
    auto requantize = [&](auto&& pack) {
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const int col = wc + 16 * i, part = col >> 6, ch16 = (col >> 4) & 3;
            const v4i m = *reinterpret_cast<const v4i*>(par + col + 4 * fch), sh = *reinterpret_cast<const v4i*>(par + QA_COLS + col + 4 * fch);
            // (rows 16 j on: the swizzles depend on frow only)
            int8_t* const to = qa_lds + (part == 0 ? QL::Q : (part == 1 ? QL::K : QL::V)) + (wr + frow) * 64 + ((ch16 ^ (part == 2 ? swz_v(frow) : swz_k(frow))) << 4) + 4 * fch;
#pragma unroll
            for (int j = 0; j < FM; ++j) *reinterpret_cast<uint32_t*>(to + j * 1024) = pack(acc[i][j], m, sh);
        }
    };
    if (mode == TALL)
        requantize([](const v4i& v, const v4i& m, const v4i& sh) {
            typedef short v2s __attribute__((ext_vector_type(2)));
            int32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = __mulhi(v[e], m[e]) >> ((sh[e] - 40) & 31);
            auto two = [](int32_t x, int32_t y) {
                const v2s r = __builtin_elementwise_max(__builtin_elementwise_add_sat(__builtin_bit_cast(v2s, __builtin_amdgcn_cvt_pk_i16(x, y)), v2s{128, 128}), v2s{-127 * 256, -127 * 256});
                return __builtin_bit_cast(uint32_t, r);
            };
            return __builtin_amdgcn_perm(two(w[2], w[3]), two(w[0], w[1]), 0x07050301u);
        });
    else if (mode == FAST)
        requantize([](const v4i& v, const v4i& m, const v4i& sh) {
            int32_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = med3_const<-127, 127>((int32_t)(((int64_t)v[e] * m[e] + ((int64_t)1 << ((sh[e] - 1) & 63))) >> 32) >> ((sh[e] - 32) & 31));
            return pack4_perm(o[0], o[1], o[2], o[3]);
        });
    else
        requantize([](const v4i& v, const v4i& m, const v4i& sh) {
            int32_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = clamp_i64_to_i32(dyadic64(v[e], m[e], sh[e] & 63), 127);
            return pack4_perm(o[0], o[1], o[2], o[3]);
        });
    __syncthreads();
    if (g.qkv) {
        for (int p = tid; p < 12 * QL::ROWS; p += 64 * NW) {
            const int part = p / (4 * QL::ROWS), row = (p >> 2) % QL::ROWS, c = p & 3, s = row / QL::SEG, r = row - s * QL::SEG;
            if (s < seqs && r < L)
                *reinterpret_cast<v4i*>(g.qkv + (int64_t)((b0 + s) * L + r) * 3 * hidden + part * hidden + h * ATT_DH + 16 * c) = *reinterpret_cast<const v4i*>(
                    qa_lds + (part == 0 ? QL::Q : (part == 1 ? QL::K : QL::V)) + row * 64 + ((c ^ (part == 2 ? swz_v(row) : swz_k(row))) << 4));
        }
    }

    // ---- attention: 16 queries a wavefront ------------------------------------------------------
    const int s = 16 * wave / QL::SEG, qrow0 = 16 * wave - s * QL::SEG, b = b0 + s;
    if (16 * wave >= QL::ROWS || s >= seqs || qrow0 >= L) return;
    int keys = L;                                                  // that are not masked
    if (a.key_lens) {
        keys = a.key_lens[b];
        keys = keys < 1 ? 1 : (keys > L ? L : keys);
    }
    attention_rows<QL::NKB, FORM>(a, qa_lds + QL::Q + 16 * wave * 64, qa_lds + QL::K + s * QL::SEG * 64, qa_lds + QL::V + s * QL::SEG * 64, lds0 + QL::TABLE, lane, b,
                                  b * a.heads + h, h, qrow0, keys, (keys + 63) >> 6, []() {}, []() {});
}

// ---- launcher ----------------------------------------------------------------------------------
// log2 of the shares of heads: fewest bytes to the L2s, x to 2^xs and W to 2^(3 - xs) of them.
static int qkv_shares(int64_t tokens, int32_t heads)
{
    auto cost = [&](int xs) { return (tokens << xs) + ((int64_t)3 * ATT_DH * heads << (3 - xs)); };
    int best = 0;
    for (int xs = 1; xs <= 3; ++xs)
        if (heads % (1 << xs) == 0 && cost(xs) < cost(best)) best = xs;
    return best;
}

// Deals the heads of groups of `seqs` sequences; returns the workgroups.
static int64_t qkv_deal(QkvAttentionArgs& g, int32_t batch, int32_t seq, int32_t heads, int seqs)
{
    g.batch = batch;
    g.groups = (batch + seqs - 1) / seqs;
    g.xs = qkv_shares((int64_t)batch * seq, heads);
    g.cols = heads >> g.xs;
    g.cols_magic = udiv_magic(g.cols);
    return (((int64_t)g.groups * g.cols + (8 >> g.xs) - 1) >> (3 - g.xs)) * 8;       // (the longest run of an XCD)
}

// The tile of a problem: wavefronts, 16-row blocks of one, sequences, stages.  Measured as whole forwards of 6 layers, us a layer, W of all layers in the memory-side cache.
//   * Four stages where workgroups do not share a unit: 8 x 12 heads, L = 64 34.7 / 34.2, 11 x 12, L = 96 42.5 / 42.0, 8 x 16, L = 32 33.9 / 32.8.  Up to three
//     quarters of the units: with more the workgroups that read ahead find no place beside them, 21 x 12, L = 48 39.5 / 40.6.
//   * Sequences side by side where more than one workgroup falls on a unit, as each brings the head's W: L = 64, 128 x 12 heads 103.5 -> 97.3; L = 32,
//     43 x 12 49.8 -> 46.4 (two) and 46.7 (four), 128 x 12 72.8 -> 66.8 and 63.8.  With fewer they would leave units idle: 21 x 12, L = 64 46.1 against 49.5.
struct QkvTile {
    int nw, fm, seqs, stages;
    int rows() const { return 4 * fm * nw / seqs; }                // of a sequence
    int code() const { return 1000 * nw + 100 * fm + 10 * seqs + stages; }
};
static int g_qkv_override = -1;
static QkvTile qkv_tile(int32_t batch, int32_t seq, int32_t heads)
{
    if (g_qkv_override > 1) return QkvTile{g_qkv_override / 1000, g_qkv_override / 100 % 10, g_qkv_override / 10 % 10, g_qkv_override % 10};
    const int64_t n = (int64_t)batch * heads;
    if (seq > 192) return QkvTile{16, 4, 1, 2};
    if (seq > 128) return QkvTile{16, 3, 1, 3};
    if (seq > 64 || n <= 256) return QkvTile{8, (seq + 31) / 32, 1, n <= 192 ? 4 : 2};
    if (seq > 32) return QkvTile{8, 4, 2, 2};
    return n <= 768 ? QkvTile{8, 2, 2, 2} : QkvTile{8, 4, 4, 2};
}

// Is it faster than the MatMul and the attention one after the other?  us a layer, those / this:
//   * One workgroup multiplies a whole head, by itself on its unit for a long time where there are few: 4 x 12 heads, L = 64 31.3 / 30.7, L = 128 36.1 / 36.7; 1 x 12, L = 128
//     26.9 / 30.1; 8 x 12, L = 64 35.4 / 34.2, L = 128 41.6 / 42.1; 11 x 12, L = 128 49.7 / 47.5, 16 x 12 52.4 / 48.4, 32 x 12 68.5 / 65.7, 64 x 12 109.5 / 99.2; 16 x 16 68.6 / 64.4,
//     32 x 16 90.9 / 82.1.
//   * A head of one to three K steps takes little longer than a launch.  A layer called by itself is ahead anywhere (us, graph and launches one by one: 2 heads 1 x 128 25.3 / 23.2 and 27.5 / 22.2, 4 heads
//     25.7 / 24.3 and 28.7 / 22.7, 6 heads 27.0 / 26.5 and 28.1 / 23.2, 6 x 128 32.2 / 31.7 and 28.7 / 27.8).  In a forward of several layers the weights come from farther away, and up to eight sequences a
//     workgroup waits for them longer than the launch takes, by the rows and K steps it has: us a forward of 12 layers, 2 heads 1 x 64 213.1 / 208.0, 1 x 96 224.0 / 225.8, 1 x 128 222.5 / 227.4, 8 x 128 249.3 /
//     251.1, 9 x 128 258.2 / 258.2, 12 x 128 269.2 / 265.0; 4 heads 1 x 64 222.0 / 219.0, 1 x 65 229.6 / 234.4, 1 x 128 232.2 / 242.0, 8 x 128 306.7 / 314.3, 9 x 70 276.9 / 274.2, 10 x 128 334.8 / 330.6; 6 heads
//     1 x 32 229.2 / 228.9, 3 x 33 241.8 / 254.0, 3 x 64 266.5 / 267.7, 1 x 128 257.2 / 273.9, 4 x 128 304.4 / 313.4, 8 x 100 342.1 / 345.2, 9 x 100 358.3 / 352.7, 16 x 128 432.3 / 416.6.
//   * More tokens of a wider model: the persistent MatMul streams, while here the path from L2 bounds the loop (more bytes a product), 256 x 16, L = 128 forwards
//     of 24 layers 10.0 / 10.2 ms; 64 x 16 3.37 / 3.24.  With 768 channels 256 x 12 311.6 / 296.3.  (Between 1024 workgroups and 4096 the two are mostly equal: forwards of 8 layers, us, 72 x 16 1336 / 1320,
//     80 x 16 1373 / 1351, 96 x 16 1486 / 1473, 128 x 16 1788 / 1783, 160 x 16 2453 / 2439, but 192 x 16 2815 / 2702: the line could lie higher.)
//   * 512 workgroups have a place at once, and a few more begin anew behind them, which costs a wide head (more K steps) most: forwards of 24 layers, ms, 32 x 16, L = 128 1.99 / 1.82,
//     33 x 16 2.71 / 2.78, 39 x 16 2.79 / 2.85, 44 x 16 3.04 / 2.91, 48 x 16 3.11 / 3.00, 52 x 16 3.27 / 3.24; 12 layers of 768 43 x 12 1.106 / 1.100, 48 x 12 1.119 / 1.113.  Of 8 layers, us: 39 x 16 903 / 919,
//     41 x 16 928 / 932, 42 x 16 920 / 917, 43 x 16 979 / 943: the kernel is ahead from 688 workgroups on, 16 before the line.
//   * Rows past the end of a sequence are multiplied too: 512 x 12, L = 40 195.0 / 197.9, L = 16 113.6 / 109.6, but 1024 x 12 173.4 / 178.2; 512 x 16, L = 40 308.6 / 340.6.  Up to 512 (sequence, head) pairs, where tiles
//     of 64 rows begin, it is even: forwards of 6 layers, us, 22 x 12, L = 33 231.9 / 232.9, 24 x 12 234.7 / 232.7, 42 x 12 280.7 / 270.4; 24 layers, 17 x 16 1035 / 1043, 20 x 16 1053 / 1052, 24 x 16 1069 / 1065.  (Short
//     sequences of two or four heads beyond 512 would be ahead, 6 layers: 1000 x 2, L = 20 322 / 290, 700 x 2, L = 40 348 / 341, but 700 x 6 728 / 756.)
//   * More than 128 tokens take all of a unit, so that whole rounds of units count: 16 x 16, L = 256 95.1 / 86.1, 21 x 12 88.1 / 82.3, L = 192 69.7 / 66.0; 11 x 12, L = 150 50.9 /
//     51.0; 24 x 12, L = 192 75.3 / 79.6.  At 160 pairs, us a forward of 6 layers: 10 x 16, L = 129 375.6 / 377.4, L = 256 445.9 / 428.8; 20 x 8, L = 129 301.5 / 297.6; 40 x 4 270.3 / 273.9, L = 193 297.2 / 286.5.
// alone: a layer called by itself.
static bool qkv_faster(int32_t batch, int32_t seq, int32_t heads, bool alone)
{
    const int64_t n = (int64_t)batch * heads;
    if (n > 512 && 4 * seq < 3 * qkv_tile(batch, seq, heads).rows()) return false;
    if (seq > 128) return n >= 160 && n <= 256;
    if (heads > 12 && (n > 1024 || (seq > 64 && n > 512 && n < 704))) return false;
    return n >= (seq > 64 ? 128 : 96) || (heads <= 6 && (alone || batch > 8 || seq + 16 * heads <= 128));
}

// (Buffers of W_qkv below 2 GiB, and sums of products below 2^30, which the kernel's fast requantizations take for granted.)
constexpr int32_t QA_MAX_HIDDEN = 1 << 13;
static_assert((int64_t)QA_MAX_HIDDEN * 128 * 128 < (1 << 30) && (int64_t)3 * QA_MAX_HIDDEN * QA_MAX_HIDDEN < 0x7fffffff, "widths");

bool qkv_attention_ok(const int8_t* x, const int8_t* w, const int8_t* ctx, int32_t batch, int32_t seq, int32_t hidden, int32_t heads, const ibert_dyadic& scores_dy,
                      const ibert_softmax_params& sp, const ibert_dyadic& ctx_dy, bool alone)
{
    if (seq > 256 || hidden != heads * ATT_DH || hidden % 128 != 0 || hidden > QA_MAX_HIDDEN || (int64_t)batch * heads > (1 << 24) || !aligned(x, 16) || !aligned(w, 16) ||
        !aligned(ctx, 4))
        return false;
    if (g_qkv_override == 0 || (g_qkv_override < 0 && !qkv_faster(batch, seq, heads, alone)) || seq > qkv_tile(batch, seq, heads).rows()) return false;
    AttentionArgs a;
    return attention_args(a, nullptr, batch, seq, heads, scores_dy, sp, ctx_dy, nullptr, nullptr, false) >= 3;
}

void qkv_attention_ahead(ReadAhead& ahead, const int8_t* w, int32_t batch, int32_t seq, int32_t hidden, int32_t heads)
{
    GemmPlan p;
    p.xs = qkv_shares((int64_t)batch * seq, heads);
    p.rows = hidden >> p.xs;
    if (p.xs < 2) ahead.add(w, 3 * hidden, hidden, p);             // (each KB once, by any XCD)
    else
        for (int i = 0; i < 3; ++i) ahead.add(w + (int64_t)i * hidden * hidden, hidden, hidden, p);
}

template <int NW, int FM, int SEQS, int STAGES>
static int launch_tile(QkvAttentionArgs& g, int form, hipStream_t stream)
{
    using QL = QkvLayout<NW, FM, SEQS>;
    static_assert(STAGES * QL::STAGE <= 163840 && QL::TABLE + 4 * ATT_TABLE <= STAGES * QL::STAGE, "LDS budget");
    const int64_t blocks = qkv_deal(g, g.batch, g.att.seq, g.att.heads, SEQS);
    g.att.blocks = (int32_t)blocks;
    const dim3 grid((unsigned)(blocks + g.att.ahead_wgs)), block(64 * NW);
#define IBERT_QA_LAUNCH(F_)                                                                                       \
    do {                                                                                                          \
        auto kern = qkv_attention_kernel<NW, FM, SEQS, F_, STAGES>;                                               \
        static bool attr_done = false;                                                                            \
        if (!attr_done) {                                                                                         \
            IBERT_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                              \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, STAGES * QL::STAGE)); \
            attr_done = true;                                                                                     \
        }                                                                                                         \
        hipLaunchKernelGGL(kern, grid, block, STAGES * QL::STAGE, stream, g);                                     \
        static const KernelName name("qkv_attention_kernel<%d, %d, %d, %d, %d>", NW, FM, SEQS, F_, STAGES);       \
        g_last_kernel = name.text;                                                                                \
    } while (0)
    if (form == 3) IBERT_QA_LAUNCH(3); else IBERT_QA_LAUNCH(4);
#undef IBERT_QA_LAUNCH
    IBERT_LAUNCH_CHECK("qkv_attention_kernel");
    return IBERT_OK;
}

int launch_qkv_attention(const int8_t* x, const int8_t* w, const int32_t* bias, const int32_t* mult, const int32_t* shift, int8_t* qkv, int8_t* ctx, int32_t batch,
                         int32_t seq, int32_t hidden, int32_t heads, const ibert_dyadic& scores_dy, const ibert_softmax_params& sp, const ibert_dyadic& ctx_dy,
                         const int32_t* key_lens, const ReadAhead* ahead, hipStream_t stream)
{
    QkvAttentionArgs g;
    const int form = attention_args(g.att, ctx, batch, seq, heads, scores_dy, sp, ctx_dy, key_lens, ahead, false);
    const QkvTile t = qkv_tile(batch, seq, heads);
    if (form < 3 || seq > t.rows()) return IBERT_ERR_NOT_IMPLEMENTED;
    g.x = x; g.w = w; g.bias = bias; g.mult = mult; g.shift = shift; g.qkv = qkv;
    g.batch = batch; g.nk = hidden / 128;
    switch (t.code()) {
#define IBERT_QA_TILE(NW_, FM_, S_, ST_) case 1000 * NW_ + 100 * FM_ + 10 * S_ + ST_: return launch_tile<NW_, FM_, S_, ST_>(g, form, stream);
        IBERT_QA_TILE(8, 1, 1, 2) IBERT_QA_TILE(8, 2, 1, 2) IBERT_QA_TILE(8, 3, 1, 2) IBERT_QA_TILE(8, 4, 1, 2)
        IBERT_QA_TILE(8, 1, 1, 4) IBERT_QA_TILE(8, 2, 1, 4) IBERT_QA_TILE(8, 3, 1, 4) IBERT_QA_TILE(8, 4, 1, 4)
        IBERT_QA_TILE(8, 2, 2, 2) IBERT_QA_TILE(8, 4, 2, 2) IBERT_QA_TILE(8, 4, 4, 2)
        IBERT_QA_TILE(16, 3, 1, 3) IBERT_QA_TILE(16, 4, 1, 2)
#undef IBERT_QA_TILE
        default: return IBERT_ERR_NOT_IMPLEMENTED;
    }
}

}  // namespace ibert

extern "C" void ibert_qkv_attention_override(int32_t tile) { ibert::g_qkv_override = tile; }

extern "C" int ibert_qkv_attention_plan(int32_t batch, int32_t seq, int32_t heads, int32_t* tile, uint8_t* places, uint8_t* readers, uint8_t* ahead)
{
    using namespace ibert;
    if (!tile || !places || !readers || !ahead) return IBERT_ERR_NULL;
    if (batch < 1 || seq < 1 || seq > 256 || heads < 2 || heads % 2) return IBERT_ERR_SHAPE;
    const QkvTile t = qkv_tile(batch, seq, heads);
    *tile = t.code();
    if (g_qkv_override < 0 && !qkv_faster(batch, seq, heads, true)) return IBERT_ERR_NOT_IMPLEMENTED;
    QkvAttentionArgs g;
    g.att.heads = heads;
    const int64_t blocks = qkv_deal(g, batch, seq, heads, t.seqs);
    for (int64_t k = 0; k < blocks; ++k) {
        int group, h;
        if (!qkv_attention_place(g, (unsigned)k, group, h)) continue;
        if (group < 0 || group >= g.groups || h < 0 || h >= heads) return IBERT_ERR_SHAPE;
        for (int s = group * t.seqs; s < (group + 1) * t.seqs && s < batch; ++s) ++places[(int64_t)s * heads + h];
        for (int m = 0; m < 3; ++m) readers[m * heads + h] |= (uint8_t)(1 << (k & 7));
    }
    const int32_t hidden = heads * ATT_DH;
    const int64_t kbs = (int64_t)3 * hidden * hidden / 1024;
    const int8_t* const w = reinterpret_cast<const int8_t*>((uintptr_t)4096);      // (an aligned address; nothing is read)
    ReadAhead r;
    qkv_attention_ahead(r, w, batch, seq, hidden, heads);
    for (int i = 0; i < r.n; ++i) {
        const auto& q = r.part[i];
        for (int x = 0; x < 8; ++x) {
            const int s = ReadAhead::share(x, q.xs);
            for (int32_t k = 0; k < ReadAhead::count(s, q.kb, q.blocks, q.xs); ++k) {
                const int64_t at = (q.p - w) / 1024 + ReadAhead::at(s, k, q.kb, q.kb_magic, q.xs);
                if (at < 0 || at >= kbs) return IBERT_ERR_SHAPE;
                ++ahead[x * kbs + at];
            }
        }
    }
    return IBERT_OK;
}

extern "C" int ibert_qkv_attention_chosen(int32_t batch, int32_t seq, int32_t heads, int32_t layers, int32_t* tile)
{
    using namespace ibert;
    if (!tile) return IBERT_ERR_NULL;
    if (batch < 1 || seq < 1 || heads < 2 || heads % 2 || layers < 1) return IBERT_ERR_SHAPE;
    *tile = seq <= 256 && qkv_faster(batch, seq, heads, layers == 1) ? qkv_tile(batch, seq, heads).code() : 0;
    return IBERT_OK;
}
