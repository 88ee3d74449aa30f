// Self-attention core of one encoder layer in one kernel: scores = DY(Q_h K_h^T), integer Softmax over the
// keys (Alg. 3; Eq. 11-14), context = clamp(DY(P V_h)) -- steps 2, 3 and 4 of the layer (Fig. 1 right;
// Sec. 4.1), bit-identical to running them one after the other.  The INT32 scores and the INT8
// probabilities never leave the CU.
//
// Shape: head width 64, any sequence length up to 512 (a whole score row, L/4 values per lane, stays in registers; the
// integer exponent cannot be rescaled exactly, so the row maximum must be known before the first exponent is taken).
// One workgroup of four wavefronts owns 64 queries of one (batch, head); a wavefront owns 16.  The kernel is instantiated
// per number of 64-key blocks; rows past the end of the sequence are read from its last row, their keys are masked and
// their queries not stored.
//   * From 6 or 7 key blocks on K_h and V_h may take turns in one LDS buffer (see att_may_share).
//   * Everything goes from global memory straight into LDS (global_load_lds, 1 KB = 16 rows of 64 bytes per request), in
//     row-major order with the 16-byte chunks of a row swizzled by the row: the wavefront's queries, K_h and V_h.
//   * K_h rows are MFMA operands as they stand (one 16-byte read per lane).  V_h is needed transposed: ds_read_b64_tr_b8 hands
//     a lane 8 keys of one channel, from rows that the lanes of a 16-lane group choose freely (see `context` below).
//   * Scores: one MFMA (16x16x64) per wavefront and 16 keys; lane l then holds, for query l%16, the keys
//     {16 i + 4 (l/16) + r}.  Row maximum and row sum finish with two cross-lane steps over the four lanes
//     that share a query.
//   * The probabilities are packed four to a dword as they are produced; the four dwords i = 4kb..4kb+3 are
//     exactly the lane's MFMA operand for key block kb under the key order above, so P never moves.
//   * Context: requantized and stored as 4 bytes per lane.
//   * Padded sequences: the keys from key_lens[b] on take the logit INT32_MIN before the row maximum is taken (the
//     paper does not treat padding; this is the integer form of adding minus infinity to a masked logit).
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

// May K_h and V_h take turns in one LDS buffer?  From 7 key blocks on (61 and 69 KB with two buffers) only two workgroups fit a
// compute unit, two wavefronts a SIMD, which do not hide the chains of the exponent from each other; with one buffer three do.
// V_h is then requested when all scores have been made and arrives during the Softmax.  us, L = 512: 64 x 12 heads 108.3 -> 92.3,
// 8 x 12 16.3 -> 15.3; L = 448, 72 x 12 97.8 -> 81.9; FORM 0, L = 448: 64 x 12 229.4 -> 184.4, 11 x 7 39.6 -> 33.1.  (Six blocks and
// fewer: three workgroups fit, no change; six with a table of the exponent beside them: two, and one buffer is ahead, L = 384: 64 x 12 heads 51.8
// -> 42.9, 8 x 12 11.6 -> 10.2.)  Not FORM 0 with 8 blocks: it needs 171 vector registers, more than three wavefronts of a
// SIMD have, so V_h would only come later (L = 512: 64 x 12 heads 296.6, with one buffer 298.5; 60 x 16 at L = 500 372.0, 374.2).
// Not where every workgroup has its place with two buffers: V_h had better come early then (1 x 12 heads at L = 512: 7.8, with
// one buffer 8.1).
constexpr bool att_may_share(int nkb, int form) { return nkb == 7 || (nkb == 8 && form != 0) || (nkb == 6 && form >= 3); }
constexpr int ATT_SHARE_WGS = 512;

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
template <int NKB, int FORM>
__global__ __launch_bounds__(ATT_THREADS) void attention_kernel(AttentionArgs a)
{
    constexpr int NI = 4 * NKB;
    const bool one = att_may_share(NKB, FORM) && a.one_buffer;
    extern __shared__ __attribute__((aligned(16))) int8_t att_lds[];
    int8_t* const qs = att_lds;                                               // queries [64][64]
    int8_t* const ks = qs + ATT_QB * ATT_DH;                                  // K_h [64 NKB][64]
    int8_t* const vs = one ? ks : ks + 64 * NKB * ATT_DH;                     // V_h [64 NKB][64]
    const uint32_t tab = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)att_lds + (uint32_t)((1 + (one ? 1 : 2) * NKB) * 64 * ATT_DH);
    typedef __attribute__((address_space(3))) uint32_t* lds_u32;
    typedef const __attribute__((address_space(3))) uint16_t* lds_u16;

    // every argument is in registers from here on: one trip to memory, not one at each first use
    asm volatile("" :: "s"(a.qkv), "s"(a.ctx), "s"(a.heads), "s"(a.seq), "s"(a.qblks), "s"(a.blocks), "s"(a.one_buffer), "s"(a.qblks_magic), "s"(a.heads_magic),
                 "s"(a.xcd_q), "s"(a.xcd_r), "s"(a.ld_qkv), "s"(a.ld_ctx), "s"(a.s_m), "s"(a.s_s), "s"(a.c_m), "s"(a.c_s),
                 "s"(a.sm.q_b), "s"(a.sm.q_c), "s"(a.sm.q_ln2), "s"(a.sm.k), "s"(a.z_m), "s"(a.z_c), "s"(a.z_s), "s"(a.t.top), "s"(a.t.below), "s"(a.t.shift),
                 "s"(a.key_lens));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= a.blocks) {
        // Workgroups that read ahead (see ReadAhead), each for its own XCD: 1 KB a request into LDS that nobody reads.  They come last,
        // one for every unit: the attention's own are on their way by then, and a unit that has some runs these beside them.
        const int x = (int)blockIdx.x & 7, first = ((int)blockIdx.x - a.blocks) >> 3;
        const uint32_t dst = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)att_lds + (uint32_t)wave * 1024u;
        // (its arguments are fetched here: the attention's own workgroups have no use for them)
        typedef const __attribute__((address_space(4))) AttentionArgs* kernel_args;
#if defined(__HIP_DEVICE_COMPILE__)
        kernel_args ga = (kernel_args)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(ga));
#else
        kernel_args ga = nullptr;
#endif
        const int wgs = ga->ahead_wgs >> 3;                // of an XCD
#pragma unroll
        for (int r = 0; r < ReadAhead::MOST; ++r) {
            const auto& q = ga->ahead.part[r];
            const int s = ReadAhead::share(x, q.xs), total = ReadAhead::count(s, q.kb, q.blocks, q.xs);
            for (int k = first * 4 + wave; k < total; k += 4 * wgs) {
                const int8_t* src = q.p + ReadAhead::at(s, k, q.kb, q.kb_magic, q.xs) * 1024;
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                             :: "s"(dst), "v"((uint32_t)lane * 16u), "s"(src) : "memory", "m0");
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);                // (the LDS is given back only when nothing writes to it any more)
        return;
    }
    // Workgroups are dealt round-robin to the 8 XCDs.  The query blocks of a head read the same K and V,
    // and neighbouring heads share 128-byte lines of the packed QKV rows: give each XCD a contiguous run of
    // (batch, head, query block) -- xcd_q of them, one more for the first xcd_r XCDs -- so that those re-reads hit its own L2.
    const int xcd = blockIdx.x & 7;
    const int bid = xcd * a.xcd_q + (xcd < a.xcd_r ? xcd : a.xcd_r) + (int)(blockIdx.x >> 3);
    const int bh = udiv_fix(bid, a.qblks, a.qblks_magic);
    const int qblk = bid - bh * a.qblks;                   // which 64 of the queries
    const int b = udiv_fix(bh, a.heads, a.heads_magic), h = bh - b * a.heads;
    const int L = a.seq, hidden = a.heads * ATT_DH;
    const int8_t* base = a.qkv + (int64_t)b * L * a.ld_qkv + h * ATT_DH;
    int nk = L;                                            // keys that are not masked
    if (a.key_lens) {
        nk = a.key_lens[b];
        nk = nk < 1 ? 1 : (nk > L ? L : nk);
    }
    const int nkb = ((FORM == 0 ? L : nk) + 63) >> 6;      // key blocks worked on

    // ---- global -> LDS -------------------------------------------------------------------------
    const int frow = lane & 15, fch = lane >> 4;
    const int qrow0 = qblk * ATT_QB + wave * 16;           // the wavefront's first query
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)att_lds + (uint32_t)wave * 1024u;
    const int r16 = lane >> 2;
    auto request = [&](const int8_t* src, int row0, uint32_t chunk, uint32_t dst) {
        int row = row0 + r16;
        row = row < L ? row : L - 1;
        const uint32_t voff = (uint32_t)row * (uint32_t)a.ld_qkv + chunk;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(dst), "v"(voff), "s"(src) : "memory", "m0");
    };
    auto request_v = [&](int n) {
        const uint32_t cv = (uint32_t)(((lane & 3) ^ swz_v(r16)) << 4);
#pragma unroll
        for (int p = 0; p < NKB; ++p)
            if (p < n) request(base + 2 * hidden, 64 * p + 16 * wave, cv, lds0 + (uint32_t)(ATT_QB * ATT_DH + ((one ? 0 : NKB) + p) * 4096));
    };
    {
        // lane l of a request brings, for row l / 4 of its 16, the chunk that the swizzle puts at byte 16 l
        const uint32_t ck = (uint32_t)(((lane & 3) ^ swz_k(r16)) << 4);
        request(base, qrow0, ck, lds0);
        const int n = opaque(nkb);
#pragma unroll
        for (int p = 0; p < NKB; ++p)
            if (p < n) request(base + hidden, 64 * p + 16 * wave, ck, lds0 + (uint32_t)(ATT_QB * ATT_DH + p * 4096));
        if (!one) request_v(n);
        if constexpr (FORM >= 3) {                         // while they arrive
            for (int t = tid; t <= a.t.top; t += ATT_THREADS) *(lds_u32)(uintptr_t)(tab + 4u * (uint32_t)t) = iexp_from_diff_fast((uint32_t)(a.t.top - t), a.sm) * 0x10001u;
        }
        // the queries and K have landed (V may still be on its way: it is not needed before the context)
        if (!one && n == NKB) __builtin_amdgcn_s_waitcnt(0x0f70 | NKB);
        else __builtin_amdgcn_s_waitcnt(0x0f70);
        if (FORM >= 3) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_barrier" ::: "memory");
    }

    // ---- scores --------------------------------------------------------------------------------
    const int qrow = qrow0 + frow;                         // the lane's query
    const v4i qf = *reinterpret_cast<const v4i*>(qs + (16 * wave + frow) * 64 + ((fch ^ swz_k(frow)) << 4));
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
    if (one) {                                             // K has been read by every wavefront: V may take its place
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        request_v(opaque(nkb));
    }
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
    __builtin_amdgcn_s_waitcnt(0x0f70);
    asm volatile("s_barrier" ::: "memory");                // V has landed for every wavefront
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

// Is the one-kernel form available for this shape and these pointers?
bool attention_fused_ok(const int8_t* qkv, const int8_t* ctx, int32_t seq, int32_t hidden, int32_t heads)
{
    return seq >= 1 && seq <= 512 && heads >= 1 && hidden == heads * ATT_DH && hidden < (1 << 20) && aligned(qkv, 16) && aligned(ctx, 4);
}

// The lengths for which the one-kernel form was always used: callers may pass no scratch for them, and the workspace
// regions scores and probs are documented as untouched.
bool attention_whole_blocks(int32_t seq) { return seq % 128 == 0 && seq <= 512; }

constexpr int ATT_TABLE = 1536;            // entries of 4 bytes
static constexpr size_t att_lds_bytes(int nkb, bool one_buffer) { return (size_t)(ATT_QB + (one_buffer ? 1 : 2) * 64 * nkb) * ATT_DH; }

// The table of I-Exp, if one serves: exponents of at most 16 bits and a scores shift for which the index is a 32-bit product (accumulators
// are at most 2^20).  At S = 2^-6 it has some 620 entries and pays throughout; at 2^-7 some 1430, on which one workgroup a compute unit or
// fewer gain nothing (us, arithmetic / table: 1 x 12 heads, L = 128 3.98 / 4.11; 8 x 12, L = 61 3.62 / 3.69; 64 x 12, L = 512 86.7 / 73.9).
static bool exp_table(const ibert_softmax_params& sp, int32_t m, int32_t s, int64_t blocks, ExpTable* t)
{
    const int64_t most = (int64_t)sp.q_b * sp.q_b + sp.q_c;
    if (most >= 65536 || m <= 0 || s < 23 || s > 45) return false;
    int bits = 0;
    while (most >> bits) ++bits;
    const int64_t zero = (int64_t)bits * sp.q_ln2;                 // I-Exp is zero from this distance on
    const int64_t below = (((zero + 1) << s) + m - 1) / m;         // an accumulator so far under the maximum is at least `zero` away ...
    const int64_t top = ((below * m) >> s) + 1;                    // ... and at most so much
    if (top >= (blocks > 256 ? ATT_TABLE : ATT_TABLE / 2) || below >= (1 << 30)) return false;
    if (s <= 33 && (((int64_t)1 << 20) + below) << (33 - s) >= ((int64_t)1 << 31)) return false;
    t->top = (int32_t)top; t->below = (int32_t)below; t->shift = s <= 33 ? 33 - s : s - 33;
    return true;
}

// FORM of a launch that stores neither scores nor probabilities (see the kernel): accumulators are at most 64*128^2 = 2^20 (scores) and
// 512*127*128 < 2^23 (context).
static int attention_form(const ibert_softmax_params& sp, const ibert_dyadic& scores, const ibert_dyadic& ctx, int64_t blocks, ExpTable* t)
{
    if (!softmax_fast_ok(sp) || scores.m <= 0 || scores.s < 21 || scores.s > 45 || ctx.s < 23 || ctx.s > 62) return 0;
    if (exp_table(sp, scores.m, scores.s, blocks, t)) return scores.s <= 33 ? 3 : 4;
    return scores.s >= 32 ? 1 : 2;
}

template <int NKB>
static int launch_attention_l(const AttentionArgs& a, int64_t blocks, int form, hipStream_t stream)
{
    const size_t lds_bytes = att_lds_bytes(NKB, att_may_share(NKB, form) && a.one_buffer) + (form >= 3 ? 4 * (size_t)(a.t.top + 1) : 0);
    const dim3 grid((unsigned)(blocks + a.ahead_wgs)), block(ATT_THREADS);
#define IBERT_ATT_LAUNCH(F_)                                                                                      \
    do {                                                                                                          \
        auto kern = attention_kernel<NKB, F_>;                                                                    \
        static bool attr_done = false;                                                                            \
        if (!attr_done && lds_bytes > 65536) {                                                                    \
            IBERT_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                              \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)att_lds_bytes(NKB, false) + 4 * ATT_TABLE)); \
            attr_done = true;                                                                                     \
        }                                                                                                         \
        hipLaunchKernelGGL(kern, grid, block, lds_bytes, stream, a);                                              \
    } while (0)
    switch (form) {
        case 0: IBERT_ATT_LAUNCH(0); break;
        case 1: IBERT_ATT_LAUNCH(1); break;
        case 2: IBERT_ATT_LAUNCH(2); break;
        case 3: IBERT_ATT_LAUNCH(3); break;
        default: IBERT_ATT_LAUNCH(4); break;
    }
#undef IBERT_ATT_LAUNCH
    return IBERT_OK;
}

int launch_attention(const int8_t* qkv, int8_t* ctx, int32_t batch, int32_t seq, int32_t hidden, int32_t heads,
                     ibert_dyadic scores_dy, const ibert_softmax_params& sp, ibert_dyadic ctx_dy, hipStream_t stream,
                     const int32_t* key_lens, int32_t* scores, int8_t* probs, const ReadAhead* ahead)
{
    if (!attention_fused_ok(qkv, ctx, seq, hidden, heads)) return IBERT_ERR_NOT_IMPLEMENTED;
    AttentionArgs a;
    a.qblks = (seq + ATT_QB - 1) / ATT_QB;
    const int64_t blocks = (int64_t)batch * heads * a.qblks;
    if (blocks == 0) return IBERT_OK;
    if (blocks > 0x7fffffffLL - 256) return IBERT_ERR_SHAPE;
    a.blocks = (int32_t)blocks;
    a.one_buffer = blocks > ATT_SHARE_WGS;                         // (where the kernel may at all)
    a.ahead_wgs = ahead ? 256 : 0;
    a.ahead = ahead ? *ahead : ReadAhead{};
    a.qkv = qkv; a.ctx = ctx; a.heads = heads; a.seq = seq;
    a.qblks_magic = udiv_magic(a.qblks); a.heads_magic = udiv_magic(heads);
    a.xcd_q = (int32_t)(blocks / 8); a.xcd_r = (int32_t)(blocks % 8);
    a.ld_qkv = 3 * hidden; a.ld_ctx = hidden;
    a.s_m = scores_dy.m; a.s_s = scores_dy.s; a.c_m = ctx_dy.m; a.c_s = ctx_dy.s;
    a.sm = softmax_const(sp);
    // z = floor(d / q_ln2) = (d M) >> z_s with M = floor(2^z_s / q_ln2) + 1 (exact for d <= 31 q_ln2 while
    // 31 q_ln2^2 < 2^z_s); z_s = 26 keeps M inside 23 bits for the smallest q_ln2
    a.z_s = sp.q_ln2 >= 17 ? 27 : 26;
    const uint32_t M = (1u << a.z_s) / (uint32_t)(sp.q_ln2 > 0 ? sp.q_ln2 : 1) + 1u;
    a.z_m = -(int32_t)M;
    a.z_c = (int32_t)(M * (uint32_t)sp.q_b);
    a.key_lens = key_lens;
    a.scores = scores; a.probs = probs;
    a.t = ExpTable{0, 0, 0};
    const int form = scores || probs ? 0 : attention_form(sp, scores_dy, ctx_dy, blocks, &a.t);
    int rc;
    switch ((seq + 63) / 64) {
        case 1: rc = launch_attention_l<1>(a, blocks, form, stream); break;
        case 2: rc = launch_attention_l<2>(a, blocks, form, stream); break;
        case 3: rc = launch_attention_l<3>(a, blocks, form, stream); break;
        case 4: rc = launch_attention_l<4>(a, blocks, form, stream); break;
        case 5: rc = launch_attention_l<5>(a, blocks, form, stream); break;
        case 6: rc = launch_attention_l<6>(a, blocks, form, stream); break;
        case 7: rc = launch_attention_l<7>(a, blocks, form, stream); break;
        default: rc = launch_attention_l<8>(a, blocks, form, stream); break;
    }
    if (rc) return rc;
    IBERT_LAUNCH_CHECK("attention_kernel");
    g_last_kernel = "attention_kernel";
    return IBERT_OK;
}

template <int NKB, int FORM>
static int attention_occupancy(int32_t* two, int32_t* one)
{
    const void* kern = reinterpret_cast<const void*>(attention_kernel<NKB, FORM>);
    const size_t table = FORM >= 3 ? 4 * ATT_TABLE : 0;
    IBERT_HIP_CHECK(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)att_lds_bytes(NKB, false) + 4 * ATT_TABLE));
    IBERT_HIP_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(two, kern, ATT_THREADS, att_lds_bytes(NKB, false) + table));
    IBERT_HIP_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(one, kern, ATT_THREADS, att_lds_bytes(NKB, true) + table));
    return IBERT_OK;
}

}  // namespace ibert

extern "C" int ibert_attention_form(const ibert_dyadic* scores_dy, const ibert_softmax_params* softmax, const ibert_dyadic* ctx_dy, int64_t workgroups, int32_t* form)
{
    if (!scores_dy || !softmax || !ctx_dy || !form) return IBERT_ERR_NULL;
    ibert::ExpTable t;
    *form = ibert::attention_form(*softmax, *scores_dy, *ctx_dy, workgroups, &t);
    return IBERT_OK;
}

extern "C" int ibert_attention_buffers(int32_t seq, int32_t form, int64_t workgroups, int32_t* shared, int32_t* fit_two, int32_t* fit_one)
{
    using namespace ibert;
    if (!shared || !fit_two || !fit_one) return IBERT_ERR_NULL;
    if (form < 0 || form > 4 || seq < (form >= 3 ? 321 : 385) || seq > 512) return IBERT_ERR_SHAPE;
    const int nkb = (seq + 63) / 64;
    *shared = att_may_share(nkb, form) && workgroups > ATT_SHARE_WGS;
    switch (10 * nkb + form) {
        case 63: return attention_occupancy<6, 3>(fit_two, fit_one);
        case 64: return attention_occupancy<6, 4>(fit_two, fit_one);
        case 70: return attention_occupancy<7, 0>(fit_two, fit_one);
        case 71: return attention_occupancy<7, 1>(fit_two, fit_one);
        case 72: return attention_occupancy<7, 2>(fit_two, fit_one);
        case 73: return attention_occupancy<7, 3>(fit_two, fit_one);
        case 74: return attention_occupancy<7, 4>(fit_two, fit_one);
        case 80: return attention_occupancy<8, 0>(fit_two, fit_one);
        case 81: return attention_occupancy<8, 1>(fit_two, fit_one);
        case 82: return attention_occupancy<8, 2>(fit_two, fit_one);
        case 83: return attention_occupancy<8, 3>(fit_two, fit_one);
        default: return attention_occupancy<8, 4>(fit_two, fit_one);
    }
}
