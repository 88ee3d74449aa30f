// INT8 MatMul for few tokens: a launch that lasts as long as its own latencies.  Arithmetic and epilogue are those of
// gemm_kernel.h; what differs is how the work is laid out.
//
//   * With a hundred rows a tile per compute unit is small and its K long: the tile configurations of gemm_kernel.h walk K in
//     order, a barrier and a trip to memory per step.  Here up to eight wavefronts share the K steps of a tile, each requests
//     all of its steps (as many as LDS holds) at once, straight into LDS, and computes them without a barrier; the partial
//     sums meet in LDS at the end.
//   * Requests are rows of 128 bytes (eight rows a request).  Loading the operands straight into registers in MFMA order
//     instead -- 16 rows of 64 bytes -- saves LDS but ran at 27 bytes per ns and compute unit: every quarter of such a load
//     touches 16 cache lines.
//   * The arguments are fetched from memory at once: fetched where each is first used, behind branches, they cost a third of
//     the kernel (the same kernel with K 768: 5.1 against 3.9 us, [128,2304]).
//   * Measured, us, W cold, against the 32x32 and 64x64 ring tiles (a kernel that does nothing takes 1.7 in the same chain):
//     128 rows: [2304] x K 768 5.4 -> 3.9, [768] x K 768 4.2 -> 2.9, [3072] x K 768 + GELU 5.6 -> 4.2, [768] x K 3072 7.1 -> 4.6;
//     488 rows: [768] x K 768 5.6 -> 3.7, [768] x K 3072 9.0 -> 6.2; 1024 rows: [1024] x K 4096 13.1 -> 12.1,
//     [768] x K 3072 10.7 -> 8.7; [128] x K 128 3.5 -> 2.3.  What is left of [128,3072] x K 768: 1.7 launch, 1.0 W from beyond L2.
#pragma once
#include "gemm_kernel.h"
#include "gemm_stream.h"

namespace ibert {

struct FewArgs {
    const int8_t* A;
    const int8_t* W;
    int32_t M, nk;                 // nk: K steps (K / 128)
    int32_t lda, ldw;
    int32_t tiles_m, tiles_n;
    int32_t xs, rm;                // log2 of the XCDs side by side; tile rows of an XCD's share
    uint32_t rm_magic;             // see udiv_fix
    int32_t nwl, stages;           // log2 of the wavefronts of a workgroup; K steps each of them has in flight
    int32_t ldc, ldr, out_clamp;
    const int32_t* bias;
    const int32_t* mult;
    const int32_t* shift;
    const int8_t* R;
    void* C;
    int32_t res_m, res_s;
    int64_t res_rnd;
    int32_t fast, c16;             // fast: K * 127^2 < 2^30 and the residual's shift is in [8, 62], or there is none
    int32_t gelu_fast;
    GeluConst gelu;
};

// The tile of a workgroup, which need not exist (see few_grid).  Workgroups go round the XCDs.  2^xs of them share the tile columns,
// 2^(3 - xs) the tile rows, so that each reads only its part of W (and of A).
__host__ __device__ __forceinline__ void few_tile(const FewArgs& g, unsigned block, int& tm, int& tn)
{
    const int xcd = block & 7, j0 = block >> 3;
    const int q = udiv_fix(j0, g.rm, g.rm_magic);
    tm = (xcd >> g.xs) * g.rm + (j0 - q * g.rm);
    tn = (q << g.xs) + (xcd & ((1 << g.xs) - 1));
}

// Tile of 16 HM rows x 16 HN columns.
template <int HM, int HN, bool OUT_I8, bool GELU>
__global__ __launch_bounds__(512) void gemm_few_kernel(FewArgs g)
{
    constexpr int TM = 16 * HM, TN = 16 * HN, UPR = 4 * HN;        // UPR: 16-byte units of a row of partial sums
    constexpr int NT = TM * UPR;                                   // threads of the epilogue, four values each
    constexpr int STAGE = (TM + TN) * 128, NL = (TM + TN) / 8;     // bytes and requests of a K step
    constexpr int EP = (NT + 511) / 512;                           // groups of four values a thread finishes
    static_assert(TM * TN * 4 <= STAGE, "a wavefront's sums fit where its first stage was");
    extern __shared__ __align__(16) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    few_tile(g, blockIdx.x, tm, tn);
    const int m0 = tm * TM, n0 = tn * TN;
    const int nw = 1 << g.nwl, nk = g.nk, stages = g.stages;
    // every argument is in registers from here on (one trip to memory, not one at each first use)
    asm volatile("" :: "s"(g.A), "s"(g.W), "s"(g.M), "s"(g.bias), "s"(g.mult), "s"(g.shift), "s"(g.R), "s"(g.C), "s"(g.ldc), "s"(g.ldr), "s"(g.out_clamp),
                 "s"(g.res_m), "s"(g.res_s), "s"(g.res_rnd), "s"(g.fast), "s"(g.c16));
    if (tn >= g.tiles_n || tm >= g.tiles_m) return;

    // Each wavefront has a ring of stages of its own in LDS, so that nothing but the sum at the end needs a barrier.
    const int8_t* const A = g.A + (int64_t)m0 * g.lda;
    const int8_t* const W = g.W + (int64_t)n0 * g.ldw;
    const int lr8 = lane >> 3, lp = lane & 7, r = lane & 15;
    int8_t* const home = lds + wave * stages * STAGE;
    const uint32_t home0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t*)lds + (uint32_t)(wave * stages * STAGE);
    // 1 KB blocks of eight rows: the lane's row and (swizzled) chunk
    const uint32_t ch0 = (uint32_t)((lp ^ (lr8 >> 1)) << 4), ch1 = ch0 ^ 64u;
    uint32_t va[2 * HM];
#pragma unroll
    for (int i = 0; i < 2 * HM; ++i) va[i] = (uint32_t)min(8 * i + lr8, g.M - 1 - m0) * (uint32_t)g.lda + ((i & 1) ? ch1 : ch0);
    const uint32_t vw = (uint32_t)lr8 * (uint32_t)g.ldw, vw0 = vw + ch0, vw1 = vw + ch1;
    auto request = [&](int step, int st) {
        const int64_t k = (int64_t)step * 128;
#pragma unroll
        for (int b = 0; b < NL; ++b) {
            const bool is_w = b < 2 * HN;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(home0 + (uint32_t)(st * STAGE + b * 1024)),
                            "v"(is_w ? ((b & 1) ? vw1 : vw0) : va[is_w ? 0 : b - 2 * HN]),
                            "s"(is_w ? W + k + (int64_t)(8 * b) * g.ldw : A + k) : "memory", "m0");
        }
    };
    for (int i = 0; i < stages; ++i)
        if (wave + (i << g.nwl) < nk) request(wave + (i << g.nwl), i);

    // what the epilogue needs, behind the first requests
    int em[EP], en[EP];
    bool ends[EP];
    v4i b4[EP], m4[EP], s4[EP];
    uint32_t res4[EP];
#pragma unroll
    for (int p = 0; p < EP; ++p) {
        const int t = tid + 512 * p;
        em[p] = t / UPR;
        en[p] = n0 + 4 * (t - em[p] * UPR);
        ends[p] = t < NT && m0 + em[p] < g.M;
        b4[p] = m4[p] = s4[p] = v4i{0, 0, 0, 0};
        res4[p] = 0;
        if (ends[p]) {
            b4[p] = *reinterpret_cast<const v4i*>(g.bias + en[p]);
            m4[p] = *reinterpret_cast<const v4i*>(g.mult + en[p]);
            s4[p] = *reinterpret_cast<const v4i*>(g.shift + en[p]);
            if (!OUT_I8 && g.R) res4[p] = *reinterpret_cast<const uint32_t*>(g.R + (int64_t)(m0 + em[p]) * g.ldr + en[p]);
        }
    }

    constexpr auto vm = [](int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); };
    static_assert(3 * NL < 64, "outstanding requests");
    v4i acc[HN][HM];
#pragma unroll
    for (int i = 0; i < HN; ++i)
#pragma unroll
        for (int j = 0; j < HM; ++j) acc[i][j] = v4i{0, 0, 0, 0};
    auto slot = [](int m, int c) { return (m * UPR + (c ^ (UPR >= 8 ? m & 7 : (m >> 1) & 3))) * 16; };
    int st = 0;
    for (int step = wave; step < nk; step += nw) {
        // steps requested after this one (the constants' loads are younger still: waiting for them too does no harm)
        int younger = 0;
        if (stages > 1) {
            const int left = (nk - 1 - step) >> g.nwl;
            younger = left < stages - 1 ? left : stages - 1;
        }
        if (younger == 0) __builtin_amdgcn_s_waitcnt(vm(0));
        else if (younger == 1) __builtin_amdgcn_s_waitcnt(vm(NL));
        else if (younger == 2) __builtin_amdgcn_s_waitcnt(vm(2 * NL));
        else __builtin_amdgcn_s_waitcnt(vm(3 * NL));
        asm volatile("" ::: "memory");
        v4i wb[2][HN], xa[2][HM];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int8_t* base = home + st * STAGE + r * 128 + (((h * 4 + (lane >> 4)) ^ swz<8>(r)) << 4);
#pragma unroll
            for (int n = 0; n < HN; ++n) wb[h][n] = *reinterpret_cast<const v4i*>(base + n * 2048);
#pragma unroll
            for (int m = 0; m < HM; ++m) xa[h][m] = *reinterpret_cast<const v4i*>(base + TN * 128 + m * 2048);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int n = 0; n < HN; ++n)
#pragma unroll
                for (int m = 0; m < HM; ++m)
                    acc[n][m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wb[h][n], xa[h][m], acc[n][m], 0, 0, 0);
        const int next = step + (stages << g.nwl);
        if (next < nk) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the stage has been read
            request(next, st);
        }
        st = st + 1 == stages ? 0 : st + 1;
    }
    if (wave < nk) {                                               // this wavefront's sums, where its first stage was
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < HN; ++i)
#pragma unroll
            for (int j = 0; j < HM; ++j) *reinterpret_cast<v4i*>(home + slot(16 * j + r, 4 * i + (lane >> 4))) = acc[i][j];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < EP; ++p) {
        if (!ends[p]) continue;
        v4i sum = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < 8; ++w)
            if (w < nw && w < nk) sum += *reinterpret_cast<const v4i*>(lds + w * stages * STAGE + slot(em[p], (en[p] - n0) >> 2));

        int32_t o[4];
        bool fast = g.fast != 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int32_t ab = b4[p][e] < 0 ? -b4[p][e] : b4[p][e];
            fast = fast && s4[p][e] >= 33 && s4[p][e] <= 62 && ab >= 0 && ab < (1 << 30);
        }
        if (__builtin_amdgcn_ballot_w64(!fast) == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t x = (int64_t)(sum[e] + b4[p][e]) * m4[p][e] + ((int64_t)1 << ((s4[p][e] - 1) & 63));
                int32_t v = (int32_t)(x >> 32) >> ((s4[p][e] - 32) & 31);
                if (!OUT_I8 && g.R) v += (int32_t)(((int64_t)(int8_t)(res4[p] >> (8 * e)) * g.res_m + g.res_rnd) >> g.res_s);
                o[e] = med3_i32(v, -g.out_clamp, g.out_clamp);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int64_t v = dyadic64(sum[e] + b4[p][e], m4[p][e], s4[p][e]);
                if (!OUT_I8 && g.R) v += dyadic64((int8_t)(res4[p] >> (8 * e)), g.res_m, g.res_s);
                o[e] = clamp_i64_to_i32(v, g.out_clamp);
            }
        }
        if constexpr (GELU) {
            const int32_t rnd = 1 << ((g.gelu.s - 33) & 31), sh = (g.gelu.s - 32) & 31;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = g.gelu_fast ? gelu_one_fast(o[e], g.gelu, rnd, sh) : gelu_one(o[e], g.gelu);
        }
        const int64_t off = (int64_t)(m0 + em[p]) * g.ldc + en[p];
        if (OUT_I8) *reinterpret_cast<uint32_t*>(static_cast<int8_t*>(g.C) + off) = pack4_i8(o[0], o[1], o[2], o[3]);
        else if (g.c16) *reinterpret_cast<uint2*>(static_cast<int16_t*>(g.C) + off) =
            uint2{((uint32_t)o[0] & 0xffffu) | ((uint32_t)o[1] << 16), ((uint32_t)o[2] & 0xffffu) | ((uint32_t)o[3] << 16)};
        else *reinterpret_cast<v4i*>(static_cast<int32_t*>(g.C) + off) = v4i{o[0], o[1], o[2], o[3]};
    }
}

// Whole tile columns, K steps and vectors only; INT8 outputs without a residual.
inline bool few_ok(const GemmArgs& g, int bn, bool i8)
{
    return g.nbatch == 1 && g.M >= 1 && g.N % bn == 0 && g.K % 128 == 0 && g.lda < (1 << 23) && g.ldw < (1 << 23) &&
           g.ldc < (1 << 23) && g.ldr < (1 << 23) && g.bias && g.per_channel && aligned(g.bias, 16) && aligned(g.mult, 16) &&
           aligned(g.shift, 16) && g.c_vec && (!g.R || (!i8 && g.r_vec));
}

// How the tiles are dealt to the XCDs: the split whose largest share is smallest, of those the one with most columns.
struct FewGrid {
    int32_t xs, rm;
    int64_t per_xcd;
};
inline FewGrid few_grid(int32_t tiles_m, int32_t tiles_n)
{
    FewGrid best{0, 0, INT64_MAX};
    for (int xs = 3; xs >= 0; --xs) {
        const int32_t rm = (tiles_m + (8 >> xs) - 1) >> (3 - xs);
        const int64_t per = (int64_t)rm * ((tiles_n + (1 << xs) - 1) >> xs);
        if (per < best.per_xcd) best = FewGrid{xs, rm, per};
    }
    return best;
}

// Deals the tiles of a problem; returns the workgroups.
inline int64_t few_deal(FewArgs& f, const GemmArgs& g, int bm, int bn)
{
    f.tiles_m = (g.M + bm - 1) / bm;
    f.tiles_n = g.N / bn;
    const FewGrid fg = few_grid(f.tiles_m, f.tiles_n);
    f.xs = fg.xs; f.rm = fg.rm;
    f.rm_magic = udiv_magic(f.rm);
    return 8 * fg.per_xcd;
}

// Wavefronts, stages and LDS bytes of a workgroup.
struct FewShape {
    int32_t nwl, stages;
    size_t lds;
};
inline FewShape few_shape(int bm, int bn, int32_t nk)
{
    const size_t stage = (size_t)(bm + bn) * 128;
    FewShape s;
    s.nwl = nk <= 4 && bm * bn <= 1024 ? 2 : 3;
    s.stages = (nk + (1 << s.nwl) - 1) >> s.nwl;
    while (s.stages > 1 && (s.stages > 4 || (s.stages << s.nwl) * stage > 163840)) --s.stages;
    s.lds = (s.stages << s.nwl) * stage;
    return s;
}

template <int HM, int HN, bool GELU>
int launch_few(const GemmArgs& g, bool i8, hipStream_t stream)
{
    if (!few_ok(g, 16 * HN, i8) || (GELU && !i8)) return IBERT_ERR_NOT_IMPLEMENTED;
    FewArgs f;
    f.A = g.A; f.W = g.W; f.bias = g.bias; f.mult = g.mult; f.shift = g.shift; f.R = g.R; f.C = g.C;
    f.M = g.M; f.nk = g.K / 128;
    f.lda = (int32_t)g.lda; f.ldw = (int32_t)g.ldw; f.ldc = (int32_t)g.ldc; f.ldr = (int32_t)g.ldr;
    const int64_t blocks = few_deal(f, g, 16 * HM, 16 * HN);
    f.out_clamp = g.out_clamp;
    f.res_m = g.res_m; f.res_s = g.res_s; f.res_rnd = g.res_rnd;
    f.fast = g.res_fast && (int64_t)g.K * 16129 < (1 << 30);
    f.c16 = g.c16;
    f.gelu_fast = g.gelu_fast; f.gelu = g.gelu;
    if (blocks > 0x7fffffffLL) return IBERT_ERR_NOT_IMPLEMENTED;         // (larger tiles make fewer of them)
    const FewShape fs = few_shape(16 * HM, 16 * HN, f.nk);
    f.nwl = fs.nwl; f.stages = fs.stages;
#define IBERT_FEW_LAUNCH(I8_)                                                                                       \
    do {                                                                                                            \
        auto kern = gemm_few_kernel<HM, HN, I8_, GELU && I8_>;                                                      \
        static bool attr_done = false;                                                                              \
        if (!attr_done) {                                                                                           \
            IBERT_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 163840));               \
            attr_done = true;                                                                                       \
        }                                                                                                           \
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64u << fs.nwl), fs.lds, stream, f);                          \
    } while (0)
    if constexpr (GELU) IBERT_FEW_LAUNCH(true);
    else if (i8) IBERT_FEW_LAUNCH(true);
    else IBERT_FEW_LAUNCH(false);
#undef IBERT_FEW_LAUNCH
    IBERT_LAUNCH_CHECK("gemm_few_kernel");
    static const KernelName names[2] = {{"gemm_few_kernel<%d, %d, %s, %s>", HM, HN, "false", GELU ? "true" : "false"},
                                        {"gemm_few_kernel<%d, %d, %s, %s>", HM, HN, "true", GELU ? "true" : "false"}};
    g_last_kernel = names[i8 ? 1 : 0].text;
    return IBERT_OK;
}

}  // namespace ibert
