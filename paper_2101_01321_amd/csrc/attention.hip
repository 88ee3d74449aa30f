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
#include "attention_core.h"

namespace ibert {

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

// See attention_rows.
template <int NKB, int FORM>
__global__ __launch_bounds__(ATT_THREADS) void attention_kernel(AttentionArgs a)
{
    const bool one = att_may_share(NKB, FORM) && a.one_buffer;
    extern __shared__ __attribute__((aligned(16))) int8_t att_lds[];
    int8_t* const qs = att_lds;                                               // queries [64][64]
    int8_t* const ks = qs + ATT_QB * ATT_DH;                                  // K_h [64 NKB][64]
    int8_t* const vs = one ? ks : ks + 64 * NKB * ATT_DH;                     // V_h [64 NKB][64]
    const uint32_t tab = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)att_lds + (uint32_t)((1 + (one ? 1 : 2) * NKB) * 64 * ATT_DH);

    // every argument is in registers from here on: one trip to memory, not one at each first use
    asm volatile("" :: "s"(a.qkv), "s"(a.ctx), "s"(a.heads), "s"(a.seq), "s"(a.qblks), "s"(a.blocks), "s"(a.one_buffer), "s"(a.qblks_magic), "s"(a.heads_magic),
                 "s"(a.xcd_q), "s"(a.xcd_r), "s"(a.ld_qkv), "s"(a.ld_ctx), "s"(a.s_m), "s"(a.s_s), "s"(a.c_m), "s"(a.c_s),
                 "s"(a.sm.q_b), "s"(a.sm.q_c), "s"(a.sm.q_ln2), "s"(a.sm.k), "s"(a.z_m), "s"(a.z_c), "s"(a.z_s), "s"(a.t.top), "s"(a.t.below), "s"(a.t.shift),
                 "s"(a.key_lens));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= a.blocks) {
        // (last, one for every unit: the attention's own are on their way by then, and a unit that has some runs these beside them)
        read_ahead<ATT_THREADS / 64, NKB == 1>((uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)att_lds, wave, lane, (int)blockIdx.x - a.blocks);
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
            make_exp_table(a, tab, tid, ATT_THREADS);
        }
        // the queries and K have landed (V may still be on its way: it is not needed before the context)
        if (!one && n == NKB) __builtin_amdgcn_s_waitcnt(0x0f70 | NKB);
        else __builtin_amdgcn_s_waitcnt(0x0f70);
        if (FORM >= 3) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_barrier" ::: "memory");
    }

    attention_rows<NKB, FORM>(
        a, qs + 16 * wave * 64, ks, vs, tab, lane, b, bh, h, qrow0, nk, nkb,
        [&]() {
            if (one) {                                     // K has been read by every wavefront: V may take its place
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                request_v(opaque(nkb));
            }
        },
        []() {                                             // V has landed for every wavefront
            __builtin_amdgcn_s_waitcnt(0x0f70);
            asm volatile("s_barrier" ::: "memory");
        });
}

// Is the one-kernel form available for this shape and these pointers?
bool attention_fused_ok(const int8_t* qkv, const int8_t* ctx, int32_t seq, int32_t hidden, int32_t heads)
{
    return seq >= 1 && seq <= 512 && heads >= 1 && hidden == heads * ATT_DH && hidden < (1 << 20) && aligned(qkv, 16) && aligned(ctx, 4);
}

// The lengths for which the one-kernel form was always used: callers may pass no scratch for them, and the workspace
// regions scores and probs are documented as untouched.
bool attention_whole_blocks(int32_t seq) { return seq % 128 == 0 && seq <= 512; }

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

int attention_args(AttentionArgs& a, int8_t* ctx, int32_t batch, int32_t seq, int32_t heads, const ibert_dyadic& scores_dy, const ibert_softmax_params& sp,
                   const ibert_dyadic& ctx_dy, const int32_t* key_lens, const ReadAhead* ahead, bool store)
{
    a.qblks = (seq + ATT_QB - 1) / ATT_QB;
    const int64_t blocks = (int64_t)batch * heads * a.qblks;
    a.blocks = (int32_t)blocks;
    a.one_buffer = blocks > ATT_SHARE_WGS;                         // (where the kernel may at all)
    a.ahead_wgs = ahead ? 256 : 0;
    a.ahead = ahead ? *ahead : ReadAhead{};
    a.qkv = nullptr; a.ctx = ctx; a.heads = heads; a.seq = seq;
    a.qblks_magic = udiv_magic(a.qblks); a.heads_magic = udiv_magic(heads);
    a.xcd_q = (int32_t)(blocks / 8); a.xcd_r = (int32_t)(blocks % 8);
    a.ld_qkv = 3 * heads * ATT_DH; a.ld_ctx = heads * ATT_DH;
    a.s_m = scores_dy.m; a.s_s = scores_dy.s; a.c_m = ctx_dy.m; a.c_s = ctx_dy.s;
    a.sm = softmax_const(sp);
    // z = floor(d / q_ln2) = (d M) >> z_s with M = floor(2^z_s / q_ln2) + 1 (exact for d <= 31 q_ln2 while
    // 31 q_ln2^2 < 2^z_s); z_s = 26 keeps M inside 23 bits for the smallest q_ln2
    a.z_s = sp.q_ln2 >= 17 ? 27 : 26;
    const uint32_t M = (1u << a.z_s) / (uint32_t)(sp.q_ln2 > 0 ? sp.q_ln2 : 1) + 1u;
    a.z_m = -(int32_t)M;
    a.z_c = (int32_t)(M * (uint32_t)sp.q_b);
    a.key_lens = key_lens;
    a.scores = nullptr; a.probs = nullptr;
    a.t = ExpTable{0, 0, 0};
    return store ? 0 : attention_form(sp, scores_dy, ctx_dy, blocks, &a.t);
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
    const int64_t blocks = (int64_t)batch * heads * ((seq + ATT_QB - 1) / ATT_QB);
    if (blocks == 0) return IBERT_OK;
    if (blocks > 0x7fffffffLL - 256) return IBERT_ERR_SHAPE;
    const int form = attention_args(a, ctx, batch, seq, heads, scores_dy, sp, ctx_dy, key_lens, ahead, scores || probs);
    a.qkv = qkv; a.scores = scores; a.probs = probs;
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
