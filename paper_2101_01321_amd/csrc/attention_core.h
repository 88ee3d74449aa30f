// What the attention of one wavefront is made of: 16 queries of a (batch, head) against the keys and values that stand in LDS (Alg. 3 between its
// two MatMuls; Fig. 1 right).  Shared by the kernel that reads packed QKV (attention.hip) and the one that makes its own (qkv_attention.hip).
#pragma once
#include "common.h"
#include "softmax_math.h"

namespace ibert {

typedef int v4i __attribute__((ext_vector_type(4)));

// FORM 3, 4: I-Exp over the distances top .. 0 from the row maximum, in LDS, every entry twice.  An accumulator that is `below` or more under
// the largest of its row is so far from it that I-Exp is zero, and at `below` the distance is at most `top`.
struct ExpTable {
    int32_t top, below, shift;             // shift: |33 - scores shift|
};

struct AttentionArgs {
    const int8_t* qkv;     // [batch*seq, 3*hidden]: Q | K | V, heads side by side
    int8_t* ctx;           // [batch*seq, hidden]
    int32_t heads, seq, qblks;
    int32_t blocks;        // workgroups of the attention itself; ahead_wgs further ones read ahead
    int32_t one_buffer;    // K_h and V_h share their place in LDS, see att_may_share
    uint32_t qblks_magic, heads_magic;   // floor(2^32 / d) + 1: see udiv_fix (a division by a run-time divisor is some thirty scalar instructions)
    int32_t xcd_q, xcd_r;  // workgroups per XCD and the remainder, see the kernel
    int32_t ld_qkv, ld_ctx;
    int32_t s_m, s_s;      // scores requantization
    int32_t c_m, c_s;      // context requantization
    SoftmaxConst sm;
    int32_t z_m, z_c, z_s; // FORM 1, 2: floor(d / q_ln2) = (z_c - z_m u) >> z_s for u = q_b - d
    ExpTable t;            // FORM 3, 4
    const int32_t* key_lens;   // optional [batch]: sequence b attends to its first key_lens[b] keys only
    int32_t* scores;       // FORM 0 only, optional: the INT32 scores [batch*heads, seq, seq] and
    int8_t* probs;         // the INT8 probabilities are also stored
    int32_t ahead_wgs;
    ReadAhead ahead;
};

constexpr int ATT_DH = 64, ATT_QB = 64, ATT_THREADS = 256;
constexpr int ATT_TABLE = 1536;            // entries of 4 bytes, at most

// Fills what a launch has in common (attention.hip); returns its FORM.  store: the scores or probabilities are asked for.
int attention_args(AttentionArgs& a, int8_t* ctx, int32_t batch, int32_t seq, int32_t heads, const ibert_dyadic& scores_dy, const ibert_softmax_params& sp,
                   const ibert_dyadic& ctx_dy, const int32_t* key_lens, const ReadAhead* ahead, bool store);

// LDS chunk swizzles of 64-byte rows: four rows share a 256-byte bank cycle.  K and Q: a lane group reads one chunk of 16
// consecutive rows.  V: a transposing read takes one chunk of rows 16 apart and of 16 consecutive ones.
__device__ __forceinline__ int swz_k(int row) { return (row >> 1) & 3; }
__device__ __forceinline__ int swz_v(int row) { return (row >> 2) & 3; }

// DY(x; m, s) for |x| < 2^b when b <= s <= 62 (b <= 23): x m + 2^(s-1) fits 63 bits and the result fits 32 (it is
// below 2^(b+31-s)), so the floor-division by 2^s is bits [s, s+32) of the 64-bit sum: the high dword shifted by
// s - 32 (HIGH: s >= 32), or for s < 32 a funnel shift of the two dwords.  add = 2^(s-1), or that plus a multiple of 2^s.
template <bool HIGH>
__device__ __forceinline__ int32_t dyadic_hi(int32_t x, int32_t m, int64_t add, int32_t sh)
{
    const int64_t p = (int64_t)x * m + add;
    const int32_t hi = (int32_t)(p >> 32);
    return HIGH ? hi >> ((sh - 32) & 31) : (int32_t)__builtin_amdgcn_alignbit((uint32_t)hi, (uint32_t)p, (uint32_t)(sh & 31));
}

// A copy of a uniform value that the compiler does not relate to the original.  The tests of the block loops below then stay
// scalar compares where they stand; related, they are evaluated once and carried as lane masks, which costs two vector
// instructions and a register pair for each test.
__device__ __forceinline__ int32_t opaque(int32_t v)
{
    asm volatile("" : "+s"(v));
    return v;
}

// The table of I-Exp (see ExpTable), 4 (top + 1) bytes at LDS address `tab`, by `threads` threads.
__device__ __forceinline__ void make_exp_table(const AttentionArgs& a, uint32_t tab, int tid, int threads)
{
    typedef __attribute__((address_space(3))) uint32_t* lds_u32;
    for (int t = tid; t <= a.t.top; t += threads) *(lds_u32)(uintptr_t)(tab + 4u * (uint32_t)t) = iexp_from_diff_fast((uint32_t)(a.t.top - t), a.sm) * 0x10001u;
}

// Workgroups behind the attention's own that read ahead (see ReadAhead), each for its own XCD: 1 KB a request into LDS that nobody reads.  NW:
// wavefronts of a workgroup; index: of the workgroup among these.  The kernel's first argument is its AttentionArgs.
// UNROLL: all parts of a layer whose steps run apart in one run of code, for attention over one key block.  It is over before a loop, which waits for each part's
// arguments anew, has asked for its last part, so that the launch waits for those requests.  A loop otherwise: unrolled, its 4 KB stand between the kernel's head and the attention's own
// code.  Forwards, us, loop / unrolled (a layout of the code alone may be worth 1.5 %): Large 1 x 16 560.6 / 550.9, 1 x 40 605.1 / 591.0, 1 x 64 612.8 / 599.1, 2 x 60 682.6 /
// 666.7, 4 x 64 806.3 / 794.8, Base 1 x 40 270.7 / 271.5; two key blocks and more, Large 1 x 128 677.1 / 677.2, 4 x 256 1258 / 1273, Base 1 x 128 308.5 / 309.8, 1 x 512 460.2 / 463.9.
template <int NW, bool UNROLL>
__device__ __forceinline__ void read_ahead(uint32_t lds0, int wave, int lane, int index)
{
    const int x = (int)blockIdx.x & 7, first = index >> 3;
    const uint32_t dst = lds0 + (uint32_t)wave * 1024u;
    // (the arguments are fetched here: the attention's own workgroups have no use for them)
    typedef const __attribute__((address_space(4))) AttentionArgs* kernel_args;
#if defined(__HIP_DEVICE_COMPILE__)
    kernel_args ga = (kernel_args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ga));
#else
    kernel_args ga = nullptr;
#endif
    const int wgs = ga->ahead_wgs >> 3;                            // (of an XCD)
    auto part = [&](int r) {
        const auto& q = ga->ahead.part[r];
        const int s = ReadAhead::share(x, q.xs), total = ReadAhead::count(s, q.kb, q.blocks, q.xs);
        for (int k = first * NW + wave; k < total; k += NW * wgs) {
            const int8_t* src = q.p + ReadAhead::at(s, k, q.kb, q.kb_magic, q.xs) * 1024;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(dst), "v"((uint32_t)lane * 16u), "s"(src) : "memory", "m0");
        }
    };
    if constexpr (UNROLL) {
#pragma unroll
        for (int r = 0; r < ReadAhead::APART; ++r) part(r);        // (parts that are not used have no blocks)
    } else {
        const int parts = ga->ahead.n;
#pragma unroll 1
        for (int r = 0; r < parts; ++r) part(r);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);                    // (the LDS is given back only when nothing writes to it any more)
}

// NKB: key blocks of 64.  FORM 0: any constants, and the only form that stores scores and probabilities.  FORM 1, 2: the
// 24-bit Softmax forms apply (softmax_fast_ok), the scores multiplier is positive and its shift in [32, 45] / [21, 31],
// the context shift in [23, 62].  FORM 3, 4: and a table serves (exp_table), the scores shift up to 33 / above.  There, whole blocks of masked keys are skipped (their probabilities are exactly zero:
// |scores| < 2^30, so the distance to INT32_MIN is far beyond 31 q_ln2).  The loops over key blocks are unrolled (the values
// live in registers) but each block stands behind a uniform test against the run-time block count, also where there is no
// mask: without those tests the scheduler interleaves all blocks and doubles the registers (NKB = 8: 303 instead of 150).
//
// Bound: vector ALU issue (FORM 3: busy 87 % of the cycles at L = 128, 256 x 16 heads, 70 % at L = 512, 64 x 12; LDS 50 %).
// So what a score costs is what counts.  FORM 3, 4: a table of I-Exp, made while K_h arrives.  A score is then a cap, a shift, the high half of
// a product, an address and a read of 16 bits (4 cycles for 64 lanes at random entries): w = floor(2 x), x the unrounded score, is one 32-bit
// product, where the 64-bit multiply-add of the rounded one takes two slots and its shift a third; with every entry twice the table does
// the rounding.  Each phase reads the operands of a block ahead of the one it multiplies (the tests between the blocks keep the compiler
// from it), and the cap at 127 stands behind a test of the row.  us, S = 2^-6, arithmetic exponent / this: L = 512, 64 x 12 heads 89.5 /
// 72.1, 16 x 16 33.5 / 28.3; L = 384, 64 x 12 55.2 / 43.1; L = 251, 61 x 12 28.5 / 24.0; L = 128, 256 x 16 43.4 / 40.1, 32 x 12 6.64 / 6.19,
// 1 x 12 4.02 / 4.03.  (Instructions a score at L = 512, all told: 18 -> 9.4.)
// FORM 1, 2: the requantization is monotone, so the
// row maximum is taken on the raw accumulators; with mx its requantized value, u = q_b - d = q_b - mx + score comes out
// of the same 64-bit multiply-add as the score itself (an integer added behind the rounding shift is that integer times 2^s
// added before it), so neither a subtraction nor q_b - d costs an instruction of its own: 2 (multiply-add, half rate) + shift
// + cap, then z (2), q_b - r, the polynomial, its shift, half an add and half a maximum.
//
// qs: the wavefront's 16 queries, rows of 64 bytes (swz_k); ks, vs: K_h and V_h, 64 NKB rows (swz_k, swz_v).  qrow0: the wavefront's first query in the sequence;
// nk: keys that are not masked; nkb: key blocks worked on.  keys_read() is called when all scores have been made, before_values() before V_h is read.
template <int NKB, int FORM, typename KeysRead, typename BeforeValues>
__device__ __forceinline__ void attention_rows(const AttentionArgs& a, const int8_t* qs, const int8_t* ks, int8_t* vs, uint32_t tab, int lane, int b, int bh,
                                               int h, int qrow0, int nk, int nkb, KeysRead&& keys_read, BeforeValues&& before_values)
{
    constexpr int NI = 4 * NKB;
    typedef const __attribute__((address_space(3))) uint16_t* lds_u16;
    const int frow = lane & 15, fch = lane >> 4, L = a.seq;
    // ---- scores --------------------------------------------------------------------------------
    const int qrow = qrow0 + frow;                         // the lane's query
    const v4i qf = *reinterpret_cast<const v4i*>(qs + frow * 64 + ((fch ^ swz_k(frow)) << 4));
    const int64_t s_rnd = (int64_t)1 << ((a.s_s - 1) & 63), c_rnd = (int64_t)1 << ((a.c_s - 1) & 63);
    v4i sc[NI];                                            // sc[i][r]: key 16 i + 4 fch + r
    const int n0 = opaque(nkb);
    // (the operands of a block are read while the one before it is multiplied: across the test between them the compiler does not)
    v4i kf[2][4];
    auto read_k = [&](int kb) {
#pragma unroll
        for (int i = 0; i < 4; ++i) kf[kb & 1][i] = *reinterpret_cast<const v4i*>(ks + (64 * kb + 16 * i + frow) * 64 + ((fch ^ swz_k(frow)) << 4));
    };
    read_k(0);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        if (kb >= n0) continue;
        if (kb + 1 < NKB) read_k(kb + 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[4 * kb + i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf[kb & 1][i], qf, v4i{0, 0, 0, 0}, 0, 0, 0);
    }
    keys_read();
    if constexpr (FORM == 0) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if (kb >= n0) continue;
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int key = 16 * i + 4 * fch + r;
                    sc[i][r] = clamp_i64_to_i32(dyadic64(sc[i][r], a.s_m, a.s_s), 2147483647);
                    if (a.scores && qrow < L && key < L) a.scores[((int64_t)bh * L + qrow) * L + key] = sc[i][r];
                }
        }
    }
    // masked keys, and rows past the end of the sequence (only a block that the end cuts has any; FORM 0: every block may)
    const int n1 = opaque(nkb);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
        if (kb < n1 && nk < 64 * (kb + 1)) {
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) sc[i][r] = 16 * i + 4 * fch + r < nk ? sc[i][r] : INT32_MIN;
        }

    // ---- softmax over the keys of the lane's query (four lanes share a query) ------------------
    const auto larger = [](int32_t x, int32_t y) { return x > y ? x : y; };
    int32_t mx = INT32_MIN, mx1 = INT32_MIN;               // two chains, two values a step
    const int n2 = opaque(nkb);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        if (kb >= n2) continue;
#pragma unroll
        for (int i = 4 * kb; i < 4 * kb + 4; ++i) {
            mx = larger(larger(mx, sc[i][0]), sc[i][1]);
            mx1 = larger(larger(mx1, sc[i][2]), sc[i][3]);
        }
    }
    mx = larger(mx, mx1);
    mx = combine_rows32(combine_rows16(mx, larger), larger);
    uint32_t sum = 0;
    if constexpr (FORM == 0) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if (kb >= n2) continue;
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // (a masked key may keep a share of a row at the bottom of the INT32 range; a row past the end none)
                    const uint32_t e = iexp_from_diff((uint32_t)mx - (uint32_t)sc[i][r], a.sm);
                    sc[i][r] = 16 * i + 4 * fch + r < L ? (int32_t)e : 0;
                    sum += (uint32_t)sc[i][r];
                }
        }
    } else if constexpr (FORM >= 3) {
        // w = floor(2 acc m / 2^s), so that DY(acc) = floor((w + 1) / 2).  With 2 R = (w(mx) + 1) & ~1 the distance is d = R - DY(acc) for
        // w + 1 - 2 R = -2 d and -2 d + 1: the two places of entry d, of which the table holds d = top first.
        // (opaque, and so is the addend of the address: it is one shift-and-add then, and not three instructions)
        const auto twice = [&](int32_t acc) {
            int32_t w = FORM == 3 ? __mulhi(acc << (a.t.shift & 31), a.s_m) : __mulhi(acc, a.s_m) >> (a.t.shift & 31);
            asm("" : "+v"(w));
            return w;
        };
        const int32_t lowest = mx - a.t.below;             // (masked keys, INT32_MIN, come to lie there too)
        uint32_t row_t = tab + 2u * (uint32_t)(2 * a.t.top + 1 - ((twice(mx) + 1) & ~1));
        asm("" : "+v"(row_t));
        const int nx = opaque(nkb);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if (kb >= nx) continue;
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sc[i][r] = *(lds_u16)(uintptr_t)(((uint32_t)twice(sc[i][r] > lowest ? sc[i][r] : lowest) << 1) + row_t);
                    if (r == 3) __builtin_amdgcn_sched_barrier(0);
                }
        }
        const int ns = opaque(nkb);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if (kb >= ns) continue;
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i) {
                sum += (uint32_t)sc[i][0] + (uint32_t)sc[i][1];
                sum += (uint32_t)sc[i][2] + (uint32_t)sc[i][3];
            }
        }
    } else {
        const int64_t mxq = ((int64_t)mx * a.s_m + s_rnd) >> a.s_s;                  // the row maximum, |.| < 2^30
        const int64_t row_c = s_rnd + (((int64_t)a.sm.q_b - mxq) << a.s_s);          // |.| < 2^59
        const int32_t u_lo = (int32_t)a.sm.q_b - (int32_t)a.sm.d_cap;
        const int nx = opaque(nkb);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if (kb >= nx) continue;
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t u = dyadic_hi<FORM == 1>(sc[i][r], a.s_m, row_c, a.s_s);
                    sc[i][r] = u > u_lo ? u : u_lo;
                }
            if (nk < 64 * (kb + 1)) {
#pragma unroll
                for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sc[i][r] = 16 * i + 4 * fch + r < nk ? sc[i][r] : u_lo;
            }
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t u = sc[i][r];
                    const uint32_t z = (uint32_t)smad24(u, a.z_m, a.z_c) >> a.z_s;             // floor(d / q_ln2) <= 31
                    const uint32_t v = umad24(z, a.sm.q_ln2, (uint32_t)u);                    // q_b - r, in (0, q_b]
                    sc[i][r] = (int32_t)(umad24(v, v, a.sm.q_c) >> z);                        // I-Poly, Alg. 1
                }
                sum += (uint32_t)sc[i][0] + (uint32_t)sc[i][1];
                sum += (uint32_t)sc[i][2] + (uint32_t)sc[i][3];
            }
        }
    }
    const auto add = [](int32_t x, int32_t y) { return (int32_t)((uint32_t)x + (uint32_t)y); };
    sum = (uint32_t)combine_rows32(combine_rows16((int32_t)sum, add), add);
    const uint32_t Fz = 0x80000000u / sum;                 // sum >= q_b^2 + q_c >= 1 (the maximum itself)

    // may a probability round to 128?  (Only one next to certainty; the row maximum is the largest, and its exponent is the same in every row.)
    const bool cap = FORM != 0 && __builtin_amdgcn_ballot_w64((umad24(umad24(a.sm.q_b, a.sm.q_b, a.sm.q_c), Fz, 1u << 23) >> 31) != 0) != 0;
    v4i pf[NKB];                                           // probabilities as MFMA operands, one per key block
    const int n3 = opaque(nkb);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        if (kb >= n3) continue;
        if constexpr (FORM == 0) {
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i) {
                uint32_t o[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    o[r] = normalise((uint32_t)sc[i][r], Fz, a.sm.k);
                    o[r] = o[r] > 127u ? 127u : o[r];
                    const int key = 16 * i + 4 * fch + r;
                    if (a.probs && qrow < L && key < L) a.probs[((int64_t)bh * L + qrow) * L + key] = (int8_t)o[r];
                }
                pf[kb][i & 3] = (int32_t)(o[0] | (o[1] << 8) | (o[2] << 16) | (o[3] << 24));
            }
        } else {
            // e < 2^24 and Fz <= 2^23 (sum >= q_b^2 + q_c >= 2^8), so the 24-bit multiply is exact.  For k = 7 (a byte
            // boundary: bits 24 to 31) the value is the top byte, 0 .. 128, and four of them are packed by permutes; 128
            // becomes the cap 127 by subtracting bit 7 from each byte.  A smaller k shifts first (and cannot reach 128).
#pragma unroll
            for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) sc[i][r] = (int32_t)umad24((uint32_t)sc[i][r], Fz, 1u << (30 - a.sm.k));
            if (a.sm.k != 7) {
                asm volatile("");                          // (a branch: as selects this would cost every value two instructions)
#pragma unroll
                for (int i = 4 * kb; i < 4 * kb + 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sc[i][r] = (int32_t)((uint32_t)sc[i][r] >> (7 - a.sm.k));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const v4i& o = sc[4 * kb + i];
                const uint32_t lo = __builtin_amdgcn_perm((uint32_t)o[1], (uint32_t)o[0], 0x0c0c0703u), hi = __builtin_amdgcn_perm((uint32_t)o[3], (uint32_t)o[2], 0x0c0c0703u);
                pf[kb][i] = (int32_t)__builtin_amdgcn_perm(hi, lo, 0x05040100u);
            }
        }
        if (cap) {
#pragma unroll
            for (int i = 0; i < 4; ++i) pf[kb][i] -= (int32_t)(((uint32_t)pf[kb][i] >> 7) & 0x01010101u);
        }
    }

    // ---- context -------------------------------------------------------------------------------
    // Operand of the transposed V for channels 16 cb .. +15: lane (frow, fch) needs channel 16 cb + frow of the keys
    // 64 kb + 16 i + 4 fch + r, i and r = 0 .. 3, in this order.  ds_read_b64_tr_b8: in each group of 16 lanes the pair of
    // lanes 2j, 2j + 1 points at the two 8-byte halves of 16 channels of a row j, and lane x receives channel x of the rows
    // j = 0 .. 7; so the group's rows are the keys i = 0, 1 (i = 2, 3 in the second read), r = 0 .. 3.
    before_values();
    typedef int v2i __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) v2i* lds_v2i;
    const int vrow = 16 * (frow >> 3) + 4 * fch + ((frow >> 1) & 3);
    int8_t* out = a.ctx + (int64_t)(b * L + qrow) * a.ld_ctx + h * ATT_DH + 4 * fch;
    v4i acc[4] = {};
    const int nc = opaque(nkb);
    v2i vf[2][4][2];
    auto read_v = [&](int kb) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            int8_t* const p = vs + vrow * 64 + ((cb ^ swz_v(vrow)) << 4) + 8 * (frow & 1) + kb * 4096;
            vf[kb & 1][cb][0] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)p);
            vf[kb & 1][cb][1] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(p + 2048));
        }
    };
    read_v(0);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        if (kb >= nc) continue;
        if (kb + 1 < NKB) read_v(kb + 1);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const v2i lo = vf[kb & 1][cb][0], hi = vf[kb & 1][cb][1];
            acc[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(v4i{lo.x, lo.y, hi.x, hi.y}, pf[kb], acc[cb], 0, 0, 0);
        }
    }
    auto store = [&](auto requantized) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const uint32_t pk = pack4_perm(requantized(acc[cb][0]), requantized(acc[cb][1]), requantized(acc[cb][2]), requantized(acc[cb][3]));
            if (qrow < L) *reinterpret_cast<uint32_t*>(out + 16 * cb) = pk;
        }
    };
    if (FORM == 0) store([&](int32_t v) { return clamp_i64_to_i32(dyadic64(v, a.c_m, a.c_s), 127); });
    else if (a.c_s >= 32) store([&](int32_t v) { return med3_const<-127, 127>(dyadic_hi<true>(v, a.c_m, c_rnd, a.c_s)); });
    else store([&](int32_t v) { return med3_const<-127, 127>(dyadic_hi<false>(v, a.c_m, c_rnd, a.c_s)); });
}

}  // namespace ibert
