// INT8 x INT8 -> INT32 MatMul with bias, dyadic requantization, optional residual and clamp (Sec. 1 third contribution,
// App. C.1): argument checks, the choice of a tile configuration, the generic kernel for unaligned operands, and the
// C entry points.  The MFMA kernel is in gemm_kernel.h; its tile configurations are compiled in gemm_inst_*.hip.
#include <algorithm>

#include "gemm_few.h"
#include "gemm_stream.h"

namespace ibert {

#define IBERT_GEMM_INSTANCE(...) extern template int launch_mfma<__VA_ARGS__>(GemmArgs&, bool, hipStream_t);
#include "gemm_instances_b.inc"
#include "gemm_instances_c.inc"
#include "gemm_instances_d.inc"
#include "gemm_instances_e.inc"
#include "gemm_instances_f.inc"
#undef IBERT_GEMM_INSTANCE
extern template int launch_few<1, 1, false>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<1, 1, true>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<1, 2, false>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<1, 2, true>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<2, 2, false>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<2, 2, true>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<2, 4, false>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<2, 4, true>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<2, 6, false>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<2, 6, true>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<4, 4, false>(const GemmArgs&, bool, hipStream_t);
extern template int launch_few<4, 4, true>(const GemmArgs&, bool, hipStream_t);
extern template int launch_stream<256, 256, 8, false>(GemmArgs&, bool, hipStream_t);
extern template int launch_stream<256, 256, 8, true>(GemmArgs&, bool, hipStream_t);
extern template int launch_stream<256, 192, 8, false>(GemmArgs&, bool, hipStream_t);
extern template int launch_stream<256, 192, 8, true>(GemmArgs&, bool, hipStream_t);

// ---------------------------------------------------------------------------------------------
// Generic kernel: one output element per lane (lanes run along n), any layout and alignment.
// ---------------------------------------------------------------------------------------------
template <bool TRANS_W, bool OUT_I8>
__global__ __launch_bounds__(GEMM_THREADS) void gemm_generic_kernel(GemmArgs g)
{
    const int64_t per = (int64_t)g.M * g.N;
    const int64_t idx = (int64_t)blockIdx.x * GEMM_THREADS + threadIdx.x;
    if (idx >= per * g.nbatch) return;
    const int z = (int)(idx / per);
    const int64_t e = idx - (int64_t)z * per;
    const int i = (int)(e / g.N), n = (int)(e - (int64_t)i * g.N);
    const int zo = z / g.batch_inner, zi = z - zo * g.batch_inner;
    const int8_t* a = g.A + zo * g.sA_o + zi * g.sA_i + (int64_t)i * g.lda;
    const int8_t* w = g.W + zo * g.sW_o + zi * g.sW_i;
    int32_t acc = 0;
    if (TRANS_W) {
        w += n;
        for (int k = 0; k < g.K; ++k) acc += (int32_t)a[k] * (int32_t)w[(int64_t)k * g.ldw];
    } else {
        w += (int64_t)n * g.ldw;
        for (int k = 0; k < g.K; ++k) acc += (int32_t)a[k] * (int32_t)w[k];
    }
    if (g.bias) acc += g.bias[n];
    const int32_t m = g.per_channel ? g.mult[n] : g.dy_m;
    const int32_t s = g.per_channel ? g.shift[n] : g.dy_s;
    int32_t res = 0;
    if (g.R) res = g.R[zo * g.sR_o + zi * g.sR_i + (int64_t)i * g.ldr + n];
    const int32_t o = finish(acc, m, s, g.R != nullptr, res, g);
    const int64_t off = zo * g.sC_o + zi * g.sC_i + (int64_t)i * g.ldc + n;
    if (OUT_I8) reinterpret_cast<int8_t*>(g.C)[off] = (int8_t)o;
    else if (g.c16) reinterpret_cast<int16_t*>(g.C)[off] = (int16_t)o;
    else reinterpret_cast<int32_t*>(g.C)[off] = o;
}

// ---------------------------------------------------------------------------------------------
int check_gemm(const ibert_gemm_desc& d, const void* A, const void* W, const void* mult, const void* shift,
               const void* residual, const void* C)
{
    (void)residual;
    if (d.M < 0 || d.N < 0 || d.K < 0 || d.batch_outer < 0 || d.batch_inner < 0) return IBERT_ERR_SHAPE;
    if (d.K > (1 << 17)) return IBERT_ERR_SHAPE;
    if (d.out_dtype != IBERT_I8 && d.out_dtype != IBERT_I32 && d.out_dtype != IBERT_I16) return IBERT_ERR_PARAM_RANGE;
    if (d.out_clamp < 0 || (d.out_dtype == IBERT_I8 && d.out_clamp > 127)) return IBERT_ERR_PARAM_RANGE;
    if (d.out_dtype == IBERT_I16 && d.out_clamp > 32767) return IBERT_ERR_PARAM_RANGE;
    if (d.trans_w != 0 && d.trans_w != 1) return IBERT_ERR_PARAM_RANGE;
    if (!d.per_channel && !dyadic_ok(d.requant)) return IBERT_ERR_PARAM_RANGE;
    if (residual && !dyadic_ok(d.residual_dy)) return IBERT_ERR_PARAM_RANGE;
    const int64_t nb = (int64_t)d.batch_outer * d.batch_inner;
    if (nb == 0 || d.M == 0 || d.N == 0) return IBERT_OK;
    if (nb > 0x7fffffffLL) return IBERT_ERR_SHAPE;
    if (d.lda < d.K || d.ldc < d.N || (residual && d.ldr < d.N)) return IBERT_ERR_SHAPE;
    if (d.ldw < (d.trans_w ? d.N : d.K)) return IBERT_ERR_SHAPE;
    if (!C) return IBERT_ERR_NULL;
    if (d.K > 0 && (!A || !W)) return IBERT_ERR_NULL;
    if (d.per_channel && (!mult || !shift)) return IBERT_ERR_NULL;
    return IBERT_OK;
}

// Tile configurations of the MFMA kernel.
struct GemmConfig {
    int bm, bn;
    bool direct;          // direct-to-LDS loader (N in whole tiles, K in whole steps) or register ring
};
// (0, 1, 5, 6, 8, 10, 11, 12, 16 and 20 were kernels that the rule below never takes any more, as another one with the same
//  tile is faster for every problem; their numbers stand for that one, and so they do with GELU where it carries GELU.)
static const GemmConfig kConfigs[] = {      // index = configuration number of ibert_gemm_config_override
    {256, 192, true},       // = 13
    {128, 128, true},       // = 7
    {128, 128, false},
    {64, 64, false},
    {64, 128, false},
    {128, 96, true},        // = 9
    {256, 192, true},       // = 13
    {128, 128, true},
    {256, 256, true},       // = 23
    {128, 96, true},
    {256, 128, true},       // = 14
    {128, 96, true},        // = 21
    {128, 128, true},       // = 22
    {256, 192, true},       // eight wavefronts
    {256, 128, true},       // eight wavefronts
    {32, 32, false},
    {256, 256, true},       // = 23
    {64, 96, true},
    {64, 96, true},
    {64, 128, true},
    {128, 96, true},        // = 21
    {128, 96, true},        // eight wavefronts in four rows of two and four that only request tiles
    {128, 128, true},       // the same
    {256, 256, true},       // persistent (gemm_stream.h)
    {256, 192, true},       // persistent
    {16, 16, true},         // K split over the wavefronts (gemm_few.h)
    {16, 32, true},
    {32, 32, true},
    {32, 64, true},
    {32, 96, true},
    {64, 64, true},
};
constexpr int kNumConfigs = sizeof(kConfigs) / sizeof(kConfigs[0]);
static int g_config_override = -1;
static bool g_xcd_blocks = true;
bool xcd_blocks_enabled() { return g_xcd_blocks; }
static uint32_t* g_path_word = nullptr;

// GELU with its requantization, on the host (the arithmetic of gelu_one in 64 bits; the preconditions keep every
// value inside 32).  Used only to find where the function saturates.
static int32_t gelu_host(int64_t q, const ibert_gelu_params& p)
{
    q = q < -p.q_max ? -p.q_max : (q > p.q_max ? p.q_max : q);
    int64_t u = q < 0 ? -q : q;
    u = u > -(int64_t)p.q_b ? -(int64_t)p.q_b : u;
    const int64_t v = u + p.q_b, poly = v * v + p.q_c;
    const int64_t erf = q < 0 ? -poly : (q == 0 ? 0 : poly);
    const int64_t t = q * (erf + p.q_1);
    const int sh = p.out.s;
    const __int128 prod = (__int128)t * p.out.m + (sh > 0 ? ((__int128)1 << (sh - 1)) : 0);
    const int64_t y = (int64_t)(prod >> sh);
    return (int32_t)(y < -127 ? -127 : (y > 127 ? 127 : y));
}

// The interval [lo, lo + n) outside of which GELU-with-requantization is constant on [-q_max, q_max]: at and below
// q_b the polynomial argument is clipped, erf = -q_c, and with q_1 = q_c (c = 1 in Eq. 8-9) the product is zero;
// at and above -q_b the product is linear in q, so the clamped output is monotone and constant from its first
// saturated value on.  n = 0 when the parameters do not have that shape.
static void gelu_table_range(const ibert_gelu_params& p, int32_t* lo, int32_t* n)
{
    *lo = 0; *n = 0;
    if (p.q_1 != p.q_c || p.q_b >= 0 || p.q_max < -(int64_t)p.q_b) return;
    const int32_t top = gelu_host(p.q_max, p);
    int64_t a = -(int64_t)p.q_b, b = p.q_max;                     // first q in [a, b] with the value of q_max
    while (a < b) {
        const int64_t mid = a + (b - a) / 2;
        if (gelu_host(mid, p) == top) b = mid; else a = mid + 1;
    }
    const int64_t count = a - p.q_b + 1;
    if (count > (1 << 17)) return;
    *lo = p.q_b;
    *n = (int32_t)count;
}

// The direct-to-LDS loader handles whole tile columns and K steps (any number of rows), with row offsets that fit its
// 32-bit lane offsets.
static bool dma_ok(const ibert_gemm_desc& d, int bn)
{
    return d.N % bn == 0 && d.K % 128 == 0 && d.lda < (1 << 23) && d.ldw < (1 << 23);
}
static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// (0 <= n < 2^31: a 32-bit division)
static uint32_t blocks_of(int32_t n, int b) { return ((uint32_t)n + (uint32_t)b - 1u) / (uint32_t)b; }

// Tile choice for K % 128 == 0.  What a configuration takes is linear in the K steps and in the tiles that the fullest
// compute unit gets: with k = K / 128, n = ceil(tiles / 256) and, for tiles of which `share` fit a compute unit side by
// side, r = ceil(n / share),
//   t = first[0] + first[1] k + (n - 1) (more[0] + more[1] k) + (r - 1) (again[0] + again[1] k)        nanoseconds,
// where first[] holds launch, pipeline fill and the epilogue nobody hides, more[] one more tile on the same unit, and
// again[] the extra cost of a tile that has to wait for a place (0 where share is 1).  (Tiles of gemm_few.h: n from its own
// dealing of tiles to XCDs, and a share that depends on K.)  The coefficients are least-squares fits to 640 problems timed
// on MI355X (K 128 to 8192, N 128 to 4096, 1 to 32768 rows, W changing from call to call), for 16-bit outputs with a
// residual (32-bit ones use them too), INT8 outputs and GELU outputs; the fits were within 4 to 13 % (r.m.s.).  On 135 problems that
// no fit has seen (N 192 to 4096, K 128 to 4096, 400 to 32768 rows) the choice by the present table takes 1.2 (16-bit with residual), 1.2 (INT8) and
// 2.0 % (GELU) longer on average than the best of all configurations, at worst 19 % ([1024,3072] x K 1024 + GELU 10.4 against 8.8 us).
// Thresholds on tile counts, which the table replaced, took 16 % longer on average.
// Some lines they could not draw: [4096,1024] x K 4096 to 4096 rows more, 52 -> 40 us at 8192 rows; 2741 rows of [768] x K 3072
// 25.1 -> 14.5 us (the last tile row is ragged); a second round of large tiles that would be nearly empty, [5120,1024] x K 1024
// 19.7 -> 13.3 us.
// (Later came the persistent tiles, fitted to 240 problems with the INT8 256x192 tile as the yardstick, and GELU on the tiles with
// loaders, to 13 of up to 2741 rows.  Lane-transposed stores had made GELU on the other direct-to-LDS tiles up to 20 % faster than
// their estimates, so that the tiles with loaders were taken where these are ahead, us: [5248,3968] x K 2304 83.0 / 69.5, [4009,768] x
// K 128 5.9 / 5.4.  128x128, 128x96 and 256x128 with GELU are least-squares fits to 335 problems since; one more tile of 128x128 with
// loaders costs what these show, and 256x192 starts as it does at K 128.
// The persistent tiles were fitted again when their rows went through LDS to the lanes that store them, to 255 problems of 1200 to 32768 rows
// (85 a kind): what is left of a residual's cost there was not in the estimates, and 256x192 with one workgroup a tile was taken in
// place of the persistent one, us: [32768,768] x K 3072 81.4 / 75.8, K 768 38.5 / 30.4, [15311,768] x K 768 19.1 / 16.0.  On these problems the
// choice takes 1.0, 0.4 and 0.6 % longer than the best (residual, INT8, GELU; before 2.7, 0.4, 0.6).
// On the tiles with loaders the wavefronts that only multiply have nothing to do until the first tiles arrive and build the GELU table
// then: [488,3072] x K 768 8.4 -> 7.5 us, [1024,4096] x K 1024 12.0 -> 9.4, which are one tile for at most every unit; 64x96 and 64x128
// tiles with GELU were slower than these wherever they were tried.)
struct TileCost {
    int config, share;                      // share 0: gemm_few.h
    struct { int first[2], more[2], again[2]; } kind[3];
};
static const TileCost kTileCost[] = {
    //        16/32-bit output                        INT8 output                             INT8 output of GELU (all 0: none)
    {25, 0, {{2406, 71, 56, 48, 581, 25}, {2372, 87, 116, 37, 320, 41}, {2664, 85, 83, 47, 480, 44}}},              // 16x16, K split
    {26, 0, {{2463, 92, 33, 69, 1126, 10}, {2376, 109, 88, 58, 766, 27}, {2665, 107, 51, 70, 1077, 18}}},           // 16x32, K split
    {27, 0, {{2631, 104, 34, 120, 1206, 0}, {2502, 125, 144, 86, 1002, 17}, {2749, 131, 150, 92, 1299, 1}}},        // 32x32, K split
    {28, 0, {{2876, 148, 1793, 151, 0, 0}, {2698, 175, 1546, 142, 0, 0}, {2997, 172, 1869, 126, 0, 0}}},            // 32x64, K split
    {29, 0, {{3691, 191, 2714, 219, 0, 0}, {3347, 212, 2371, 190, 0, 0}, {3723, 220, 3034, 166, 0, 0}}},            // 32x96, K split
    {30, 0, {{3905, 198, 3034, 266, 0, 0}, {3439, 230, 2564, 224, 0, 0}, {3956, 232, 3184, 229, 0, 0}}},            // 64x64, K split
    {15, 5, {{3500, 159, 581, 77, 0, 0}, {3500, 169, 497, 75, 0, 0}, {3673, 170, 549, 69, 0, 0}}},                  // 32x32, ring
    {3, 3, {{4609, 277, 1390, 160, 0, 34}, {4205, 304, 914, 147, 0, 75}, {4819, 285, 1060, 137, 749, 68}}},         // 64x64, ring
    {2, 2, {{7472, 628, 4126, 395, 0, 310}, {6288, 662, 2788, 409, 0, 256}, {0, 0, 0, 0, 0, 0}}},                   // 128x128, ring
    {17, 2, {{4020, 347, 1212, 163, 1459, 70}, {3501, 377, 823, 116, 1047, 203}, {0, 0, 0, 0, 0, 0}}},              // 64x96, three stages
    {18, 3, {{3525, 511, 1447, 72, 682, 329}, {3070, 557, 758, 56, 683, 435}, {0, 0, 0, 0, 0, 0}}},                 // 64x96
    {21, 1, {{5825, 320, 4836, 333, 0, 0}, {4587, 353, 3465, 353, 0, 0}, {5450, 353, 4050, 353, 0, 0}}},            // 128x96, with loaders
    {19, 3, {{3722, 557, 1848, 109, 0, 409}, {3329, 618, 916, 82, 254, 483}, {0, 0, 0, 0, 0, 0}}},                  // 64x128
    {22, 1, {{6537, 376, 5539, 420, 0, 0}, {4967, 408, 3662, 420, 0, 0}, {5700, 408, 4450, 560, 0, 0}}},            // 128x128, with loaders
    {7, 2, {{5451, 645, 5215, 637, 0, 0}, {3978, 690, 2886, 617, 0, 0}, {5042, 844, 3592, 633, 0, 0}}},             // 128x128
    {9, 2, {{4894, 572, 2930, 70, 1293, 436}, {3579, 626, 1375, 102, 650, 459}, {4535, 744, 1142, 158, 1331, 462}}}, // 128x96
    {14, 1, {{7647, 840, 9487, 865, 0, 0}, {5131, 882, 4119, 883, 0, 0}, {6091, 1091, 5468, 922, 0, 0}}},            // 256x128
    {13, 1, {{10461, 862, 13760, 999, 0, 0}, {6109, 963, 5826, 1068, 0, 0}, {8700, 952, 8517, 1062, 0, 0}}},        // 256x192
    {24, 1, {{9286, 837, 6519, 1144, 0, 0}, {5910, 966, 3317, 1064, 0, 0}, {8250, 967, 4273, 1092, 0, 0}}},        // 256x192, persistent
    {23, 1, {{10445, 1055, 6535, 1343, 0, 0}, {7013, 1177, 4045, 1278, 0, 0}, {9023, 1117, 4908, 1261, 0, 0}}},      // 256x256, persistent
};

static int choose_config(const ibert_gemm_desc& d, const GemmArgs& g, int64_t nb, bool gelu)
{
    if (g_config_override >= 0 && g_config_override < kNumConfigs) return g_config_override;
    const bool i8 = d.out_dtype == IBERT_I8;
    auto tiles = [&](int bm, int bn) -> int64_t { return (int64_t)blocks_of(d.M, bm) * blocks_of(d.N, bn) * nb; };
    const bool wide = d.N % 96 == 0 || d.N % 128 == 0;                  // some direct-to-LDS tile divides N
    // (GELU stays in a kernel of its own, behind a MatMul whose result the caller finds in its scratch, where K is short
    //  and no direct-to-LDS tile fits)
    if (d.K % 128 == 0 && (d.K >= 512 || wide)) {
        int best = -1;
        int64_t best_t = 0;
        for (const TileCost& c : kTileCost) {
            const GemmConfig& f = kConfigs[c.config];
            const auto& w = c.kind[gelu ? 2 : (i8 ? 1 : 0)];
            if (w.first[0] == 0 || (f.direct && !dma_ok(d, f.bn))) continue;
            if (c.config == 23 && !stream_ok<256, 256, 8>(g, i8)) continue;
            if (c.config == 24 && !stream_ok<256, 192, 8>(g, i8)) continue;
            // Without a table the persistent tiles compute GELU in their 64-bit epilogue, the others in the direct one, and are ahead, us: no table
            // (an input scale of 2^-9) [32768,4096] x K 1024 356 / 262, [4096,3072] x K 768 36.3 / 21.4; no room for it (more than 26
            // thousand entries beside 256x256, 44 beside 256x192: output scales above 3 at an input scale of 2^-6) [32768,4096] x K 1024 354 / 331.
            if (gelu && (c.config == 23 || c.config == 24) &&
                (g.gelu_lut_n == 0 || g.gelu_lut_n > (c.config == 23 ? StreamLayout<256, 256, 8, true, true>::ROOM : StreamLayout<256, 192, 8, true, true>::ROOM))) continue;
            const int64_t k = d.K / 128;
            const int64_t one = w.first[0] + w.first[1] * k;            // (the other terms only add to it)
            if (best >= 0 && one >= best_t) continue;
            // GELU on a single K step and at most one 256x192 tile for every unit: the persistent kernel has nothing to stream.
            // It took 0.5 to 4.3 % longer at each of 24 such problems of 192 to 256 tiles (us, W changing from call to call, persistent / not:
            // [4096,3072] 11.3 / 10.8, [8192,1536] 11.3 / 10.9, [16072,768] 11.05 / 10.9).  With two steps it is ahead more often than not,
            // with more nearly always (K 768 17.0 / 17.2).  INT8 without GELU has no such line: [4096,3072] at K 128 to 512 2 to 5 %
            // longer on one card, equal within 2 % on another, the other problems 15 % shorter to 6 % longer.
            if (c.config == 24 && gelu && k == 1 && tiles(256, 192) <= 256) continue;
            int64_t n, share = c.share;
            if (share == 0) {
                if (!few_ok(g, f.bn, i8)) continue;
                const FewShape s = few_shape(f.bm, f.bn, (int32_t)k);
                n = ceil_div(few_grid((int32_t)ceil_div(d.M, f.bm), d.N / f.bn).per_xcd, 32);
                share = std::min<int64_t>(163840 / (int64_t)s.lds, 32 >> s.nwl);
            } else {
                n = ceil_div(tiles(f.bm, f.bn), 256);
            }
            const int64_t r = ceil_div(n, share);
            const int64_t t = one + (n - 1) * (w.more[0] + w.more[1] * k) +
                              (r - 1) * (w.again[0] + w.again[1] * k);
            if (best < 0 || t < best_t) { best = c.config; best_t = t; }
        }
        return best;
    }
    // The register-ring loader, which takes any K that is a multiple of 16: 128x128 tiles with a 64-wide K step while that
    // gives every CU something to do, below that 64x64 tiles.
    if (tiles(128, 128) >= 384) return 2;
    // (a handful of sequences: 32x32 tiles put four times as many compute units on a long K than 64x64 do;
    //  [128,768] x K 3072: 10.5 -> 7.0 us, K 768: 5.6 -> 4.5 us)
    if (d.K >= 512) return tiles(64, 64) <= 96 ? 15 : 3;
    return 4;
}

// The arguments of a problem, all but what the kernel's launcher and the GELU epilogue fill in.
static GemmArgs gemm_args(const ibert_gemm_desc& d, const int8_t* A, const int8_t* W, const int32_t* bias,
                          const int32_t* mult, const int32_t* shift, const int8_t* residual, void* C)
{
    const bool i8 = d.out_dtype == IBERT_I8;
    GemmArgs g;
    g.A = A; g.W = W; g.bias = bias; g.mult = mult; g.shift = shift; g.R = residual; g.C = C;
    g.M = d.M; g.N = d.N; g.K = d.K;
    g.batch_inner = d.batch_inner; g.nbatch = (int32_t)((int64_t)d.batch_outer * d.batch_inner);
    g.tiles_m = g.tiles_n = 0;
    g.xcd_chunk = 0;
    g.xcd_xn = g.xcd_xs = g.xcd_bm = g.xcd_bn = 0;
    g.lda = d.lda; g.ldw = d.ldw; g.ldc = d.ldc; g.ldr = d.ldr;
    g.sA_o = d.strideA_outer; g.sA_i = d.strideA_inner;
    g.sW_o = d.strideW_outer; g.sW_i = d.strideW_inner;
    g.sC_o = d.strideC_outer; g.sC_i = d.strideC_inner;
    g.sR_o = d.strideR_outer; g.sR_i = d.strideR_inner;
    g.per_channel = d.per_channel ? 1 : 0;
    g.dy_m = d.requant.m; g.dy_s = d.requant.s;
    g.out_clamp = d.out_clamp;
    g.res_m = d.residual_dy.m; g.res_s = d.residual_dy.s;
    g.res_fast = (!residual || (d.residual_dy.s >= 8 && d.residual_dy.s <= 62)) ? 1 : 0;
    g.res_rnd = (residual && d.residual_dy.s >= 1 && d.residual_dy.s <= 62) ? ((int64_t)1 << (d.residual_dy.s - 1)) : 0;
    g.c16 = d.out_dtype == IBERT_I16 ? 1 : 0;
    g.path_word = g_path_word;
    g.gelu_fast = 0;
    g.gelu = GeluConst{0, 0, 0, 0, 0, 0};
    g.gelu_lut_lo = g.gelu_lut_n = 0;
    g.c_vec = aligned(C, i8 ? 4 : (g.c16 ? 8 : 16)) && d.ldc % 4 == 0 && d.strideC_outer % 4 == 0 && d.strideC_inner % 4 == 0;
    g.c_vec16 = i8 && aligned(C, 16) && d.ldc % 16 == 0 && d.strideC_outer % 16 == 0 && d.strideC_inner % 16 == 0;
    g.r_vec = residual && aligned(residual, 16) && d.ldr % 16 == 0 && d.strideR_outer % 16 == 0 && d.strideR_inner % 16 == 0;
    return g;
}

// With the GELU epilogue.
static void gelu_args(GemmArgs& g, const ibert_gelu_params& p)
{
    g.gelu = GeluConst{p.q_b, p.q_c, p.q_1, p.q_max, p.out.m, p.out.s};
    g.gelu_fast = gelu_fast_ok(p) ? 1 : 0;
    gelu_table_range(p, &g.gelu_lut_lo, &g.gelu_lut_n);
}

// Rows whose 16-byte chunks are aligned, W as [N,K].
static bool rows_aligned(const ibert_gemm_desc& d, const int8_t* A, const int8_t* W)
{
    return d.trans_w == 0 && d.K > 0 && aligned(A, 16) && aligned(W, 16) && d.lda % 16 == 0 && d.ldw % 16 == 0 &&
           d.strideA_outer % 16 == 0 && d.strideA_inner % 16 == 0 && d.strideW_outer % 16 == 0 && d.strideW_inner % 16 == 0;
}

GemmPlan plan_gemm(const ibert_gemm_desc& d, const int8_t* A, const int8_t* W, const int32_t* bias, const int32_t* mult,
                   const int32_t* shift, const int8_t* residual, const void* C, const ibert_gelu_params* gelu)
{
    GemmPlan p;
    if (d.batch_outer != 1 || d.batch_inner != 1 || d.M < 1 || d.N < 1 || d.ldw != d.K || d.K % 128 != 0 || !rows_aligned(d, A, W)) return p;
    GemmArgs g = gemm_args(d, A, W, bias, mult, shift, residual, const_cast<void*>(C));
    if (gelu) gelu_args(g, *gelu);
    const int cfg = choose_config(d, g, 1, gelu != nullptr);
    const GemmConfig& f = kConfigs[cfg];
    if (d.N % f.bn != 0) return p;
    if (cfg >= 25) {
        FewArgs a;
        few_deal(a, g, f.bm, f.bn);
        p.xs = a.xs;
        p.rows = f.bn;
    } else if (cfg == 23 || cfg == 24) {
        StreamArgs a;
        stream_deal(a, g, f.bm, f.bn);
        p.xs = a.xs;
        p.rows = d.N >> p.xs;
    } else {
        dim3 grid;
        if (!mfma_deal(g, f.bm, f.bn, grid)) return p;
        // (not in blocks: one tile for every XCD, side by side, or any tile of W anywhere)
        p.xs = g.xcd_xn >= 1 ? g.xcd_xs : (g.tiles_m == 1 && g.tiles_n == 8 ? 3 : 0);
        p.rows = d.N >> p.xs;
    }
    return p;
}

// For tests, see ibert_testing.h.
static int weight_plan(const ibert_gemm_desc& d, const ibert_gelu_params* gelu, int32_t out[3], uint8_t* readers, uint8_t* ahead)
{
    alignas(16) static const int32_t any[4] = {};                  // (an aligned address; nothing is read)
    int8_t* const p = reinterpret_cast<int8_t*>(const_cast<int32_t*>(any));
    const int8_t* const residual = d.out_dtype == IBERT_I8 ? nullptr : p;
    const GemmPlan plan = plan_gemm(d, p, p, any, any, any, residual, p, gelu);
    if (plan.rows < 1) return IBERT_ERR_NOT_IMPLEMENTED;
    GemmArgs g = gemm_args(d, p, p, any, any, any, residual, p);
    if (gelu) gelu_args(g, *gelu);
    const int cfg = choose_config(d, g, 1, gelu != nullptr);
    const GemmConfig& f = kConfigs[cfg];
    out[0] = cfg; out[1] = plan.rows; out[2] = plan.xs;
    auto reads = [&](int xcd, int tm, int tn) {
        if ((int64_t)tm * f.bm < d.M)
            for (int n = tn * f.bn; n < (tn + 1) * f.bn && n < d.N; ++n) readers[n] |= (uint8_t)(1 << xcd);
    };
    int z, tm, tn;
    if (cfg >= 25) {
        FewArgs a;
        const int64_t blocks = few_deal(a, g, f.bm, f.bn);
        for (unsigned b = 0; b < blocks; ++b) {
            few_tile(a, b, tm, tn);
            reads(b & 7, tm, tn);
        }
    } else if (cfg == 23 || cfg == 24) {
        StreamArgs a;
        stream_deal(a, g, f.bm, f.bn);
        for (int x = 0; x < 8; ++x) {
            const StreamRun run = stream_run(a, x);
            for (int l = 0; l < run.count; ++l) {
                stream_tile(a, run, l, tm, tn);
                reads(x, tm, tn);
            }
        }
    } else {
        dim3 grid;
        if (!mfma_deal(g, f.bm, f.bn, grid)) return IBERT_ERR_SHAPE;
        for (unsigned by = 0; by < grid.y; ++by)
            for (unsigned bx = 0; bx < grid.x; ++bx) {
                mfma_tile(g, bx, by, z, tm, tn);
                reads((int)((by * grid.x + bx) & 7), tm, tn);
            }
    }
    ReadAhead r;
    r.add(p, d.N, d.K, plan);
    const int64_t kbs = (int64_t)d.N * d.K / 1024;
    for (int i = 0; i < r.n; ++i) {
        const auto& q = r.part[i];
        for (int x = 0; x < 8; ++x) {
            const int s = ReadAhead::share(x, q.xs);
            for (int32_t k = 0; k < ReadAhead::count(s, q.kb, q.blocks, q.xs); ++k) {
                const int64_t at = ReadAhead::at(s, k, q.kb, q.kb_magic, q.xs);
                if (at < 0 || at >= kbs) return IBERT_ERR_SHAPE;
                ++ahead[x * kbs + at];
            }
        }
    }
    return IBERT_OK;
}

// gelu != nullptr asks for the GELU epilogue (INT8 output, no residual; out_clamp must be gelu->q_max): a tile
// that does not carry it, and a problem that the tile does not serve, return IBERT_ERR_NOT_IMPLEMENTED without launching.
int launch_gemm(const ibert_gemm_desc& d, const int8_t* A, const int8_t* W, const int32_t* bias,
                const int32_t* mult, const int32_t* shift, const int8_t* residual, void* C, hipStream_t stream,
                const ibert_gelu_params* gelu)
{
    const int64_t nb = (int64_t)d.batch_outer * d.batch_inner;
    if (nb == 0 || d.M == 0 || d.N == 0) return IBERT_OK;
    GemmArgs g = gemm_args(d, A, W, bias, mult, shift, residual, C);
    const bool i8 = d.out_dtype == IBERT_I8;
    if (gelu) {
        if (!i8 || residual || d.out_clamp != gelu->q_max) return IBERT_ERR_NOT_IMPLEMENTED;
        gelu_args(g, *gelu);
    }
    const bool fast = rows_aligned(d, A, W);
    if (gelu && !(fast && d.K % 16 == 0)) return IBERT_ERR_NOT_IMPLEMENTED;
    if (fast) {
        if (d.K % 16 != 0) return launch_tail(g, i8, stream);       // bytewise K tail
        const int cfg = choose_config(d, g, nb, gelu != nullptr);
        if (gelu) {
            switch (cfg) {
                case 3: return launch_mfma<64, 64, 128, 3, false, false, true>(g, i8, stream);
                case 15: return launch_mfma<32, 32, 128, 4, false, false, true>(g, i8, stream);
                case 1: case 7: if (dma_ok(d, 128)) return launch_mfma<128, 128, 128, 2, false, true, true>(g, i8, stream); break;
                case 5: case 9: if (dma_ok(d, 96)) return launch_mfma<128, 96, 128, 2, false, true, true>(g, i8, stream); break;
                case 0: case 6: case 13: if (dma_ok(d, 192)) return launch_mfma<256, 192, 128, 2, false, true, true, 8>(g, i8, stream); break;
                case 10: case 14: if (dma_ok(d, 128)) return launch_mfma<256, 128, 128, 2, false, true, true, 8>(g, i8, stream); break;
                case 11: case 20: case 21: if (dma_ok(d, 96)) return launch_mfma<128, 96, 128, 3, false, true, true, 8, 4>(g, i8, stream); break;
                case 12: case 22: if (dma_ok(d, 128)) return launch_mfma<128, 128, 128, 3, false, true, true, 8, 4>(g, i8, stream); break;
                case 8: case 16: case 23: return launch_stream<256, 256, 8, true>(g, i8, stream);
                case 24: return launch_stream<256, 192, 8, true>(g, i8, stream);
                case 25: return launch_few<1, 1, true>(g, i8, stream);
                case 26: return launch_few<1, 2, true>(g, i8, stream);
                case 27: return launch_few<2, 2, true>(g, i8, stream);
                case 28: return launch_few<2, 4, true>(g, i8, stream);
                case 29: return launch_few<2, 6, true>(g, i8, stream);
                case 30: return launch_few<4, 4, true>(g, i8, stream);
                default: break;
            }
            return IBERT_ERR_NOT_IMPLEMENTED;
        }
        int rc = IBERT_ERR_NOT_IMPLEMENTED;                         // (a problem that the kernel does not serve)
        switch (cfg) {
            case 2: return launch_mfma<128, 128, 64, 2>(g, i8, stream);
            case 3: return launch_mfma<64, 64, 128, 3>(g, i8, stream);
            case 4: return launch_mfma<64, 128, 64, 3>(g, i8, stream);
            case 1: case 7: if (dma_ok(d, 128)) return launch_mfma<128, 128, 128, 2, false, true>(g, i8, stream); break;
            case 5: case 9: if (dma_ok(d, 96)) return launch_mfma<128, 96, 128, 2, false, true>(g, i8, stream); break;
            case 0: case 6: case 13: if (dma_ok(d, 192)) return launch_mfma<256, 192, 128, 2, false, true, false, 8>(g, i8, stream); break;
            case 10: case 14: if (dma_ok(d, 128)) return launch_mfma<256, 128, 128, 2, false, true, false, 8>(g, i8, stream); break;
            case 15: return launch_mfma<32, 32, 128, 4>(g, i8, stream);
            case 17: if (dma_ok(d, 96)) return launch_mfma<64, 96, 128, 3, false, true>(g, i8, stream); break;
            case 18: if (dma_ok(d, 96)) return launch_mfma<64, 96, 128, 2, false, true>(g, i8, stream); break;
            case 19: if (dma_ok(d, 128)) return launch_mfma<64, 128, 128, 2, false, true>(g, i8, stream); break;
            case 11: case 20: case 21: if (dma_ok(d, 96)) return launch_mfma<128, 96, 128, 3, false, true, false, 8, 4>(g, i8, stream); break;
            case 12: case 22: if (dma_ok(d, 128)) return launch_mfma<128, 128, 128, 3, false, true, false, 8, 4>(g, i8, stream); break;
            case 8: case 16: case 23: rc = launch_stream<256, 256, 8, false>(g, i8, stream); break;
            case 24: rc = launch_stream<256, 192, 8, false>(g, i8, stream); break;
            case 25: rc = launch_few<1, 1, false>(g, i8, stream); break;
            case 26: rc = launch_few<1, 2, false>(g, i8, stream); break;
            case 27: rc = launch_few<2, 2, false>(g, i8, stream); break;
            case 28: rc = launch_few<2, 4, false>(g, i8, stream); break;
            case 29: rc = launch_few<2, 6, false>(g, i8, stream); break;
            case 30: rc = launch_few<4, 4, false>(g, i8, stream); break;
            default: break;
        }
        return rc != IBERT_ERR_NOT_IMPLEMENTED ? rc : launch_mfma<128, 128, 64, 2>(g, i8, stream);
    }
    const bool fast_tw = d.trans_w == 1 && d.K > 0 && d.K % 16 == 0 && d.N >= 4 && d.N % 4 == 0 && aligned(A, 16) &&
                         aligned(W, 4) && d.lda % 16 == 0 && d.ldw % 4 == 0 && d.strideA_outer % 16 == 0 &&
                         d.strideA_inner % 16 == 0 && d.strideW_outer % 4 == 0 && d.strideW_inner % 4 == 0;
    if (fast_tw) {
        if (d.N <= 64) return launch_mfma<128, 64, 64, 2, true>(g, i8, stream);
        return launch_mfma<128, 128, 64, 2, true>(g, i8, stream);
    }
    const int64_t total = (int64_t)d.M * d.N * nb;
    const int64_t blocks = (total + GEMM_THREADS - 1) / GEMM_THREADS;
    if (blocks > 0x7fffffffLL) return IBERT_ERR_SHAPE;
    if (d.trans_w) {
        if (i8) hipLaunchKernelGGL((gemm_generic_kernel<true, true>), dim3((unsigned)blocks), dim3(GEMM_THREADS), 0, stream, g);
        else hipLaunchKernelGGL((gemm_generic_kernel<true, false>), dim3((unsigned)blocks), dim3(GEMM_THREADS), 0, stream, g);
    } else {
        if (i8) hipLaunchKernelGGL((gemm_generic_kernel<false, true>), dim3((unsigned)blocks), dim3(GEMM_THREADS), 0, stream, g);
        else hipLaunchKernelGGL((gemm_generic_kernel<false, false>), dim3((unsigned)blocks), dim3(GEMM_THREADS), 0, stream, g);
    }
    IBERT_LAUNCH_CHECK("gemm_generic_kernel");
    g_last_kernel = "gemm_generic_kernel";
    return IBERT_OK;
}

// Are dense outputs and scratch asked for, whether or not this problem still goes through them?  Which problems need them
// was once decided by the tiles that carried the epilogue then, and callers were told by a refusal; kernels that have taken
// over more problems since must not turn a call that is refused on one size into one that works on the next.
static bool gelu_asks_for_scratch(const ibert_gemm_desc& d, int64_t nb)
{
    auto whole = [&](int bm, int bn) -> int64_t {
        return d.M % bm == 0 && d.N % bn == 0 && d.K % 128 == 0 ? (int64_t)(d.M / bm) * (d.N / bn) * nb : 0;
    };
    if (whole(256, 192) >= 224) return false;
    if (whole(128, 96) >= 256) return whole(128, 96) == 256 && d.K >= 2048;
    if (whole(256, 128) >= 448) return false;
    if (whole(128, 128) >= 128) return whole(128, 128) <= 256 && d.K >= 2048;
    return ceil_div(d.M, 128) * ceil_div(d.N, 128) * nb >= 384 || d.K < 512;
}

// MatMul + GELU.  One kernel where K is a multiple of 128 and either K >= 512 or 96 or 128 divides N (choose_config);
// otherwise the MatMul writes its INT32 result (clamped to +-q_max) to `scratch` and the element-wise GELU kernel follows,
// which needs dense outputs.
int launch_gemm_gelu(const ibert_gemm_desc& d0, const int8_t* A, const int8_t* W, const int32_t* bias,
                     const int32_t* mult, const int32_t* shift, const ibert_gelu_params& gelu, int8_t* C,
                     int32_t* scratch, hipStream_t stream)
{
    ibert_gemm_desc d = d0;
    d.out_dtype = IBERT_I8;
    d.out_clamp = gelu.q_max;
    const int64_t nb = (int64_t)d.batch_outer * d.batch_inner;
    if (nb == 0 || d.M == 0 || d.N == 0) return IBERT_OK;
    const bool dense = d.ldc == d.N && (d.batch_inner == 1 || d.strideC_inner == (int64_t)d.M * d.N) &&
                       (d.batch_outer == 1 || d.strideC_outer == (int64_t)d.batch_inner * d.M * d.N);
    const int refused = !dense ? IBERT_ERR_NOT_IMPLEMENTED : (!scratch ? IBERT_ERR_WORKSPACE : IBERT_OK);
    if (refused && g_config_override < 0 && gelu_asks_for_scratch(d, nb)) return refused;
    int rc = launch_gemm(d, A, W, bias, mult, shift, nullptr, C, stream, &gelu);
    if (rc != IBERT_ERR_NOT_IMPLEMENTED) return rc;
    if (refused) return refused;
    d.out_dtype = IBERT_I32;
    rc = launch_gemm(d, A, W, bias, mult, shift, nullptr, scratch, stream);
    if (rc) return rc;
    return launch_gelu(scratch, C, nb * d.M * d.N, gelu, stream);
}

}  // namespace ibert


extern "C" int ibert_gemm_config_override(int32_t config)
{
    ibert::g_config_override = config;
    return ibert::kNumConfigs;
}


extern "C" const char* ibert_last_kernel(void) { return ibert::g_last_kernel; }

extern "C" int ibert_gemm_weight_plan(const ibert_gemm_desc* desc, int32_t gelu, int32_t plan[3], uint8_t* readers, uint8_t* ahead)
{
    if (!desc || !plan || !readers || !ahead) return IBERT_ERR_NULL;
    ibert_gelu_params usual;
    const int rc = ibert_gelu_params_from_scale(1.0 / 64, 8.0 / 127, &usual);
    return rc ? rc : ibert::weight_plan(*desc, gelu ? &usual : nullptr, plan, readers, ahead);
}

extern "C" int ibert_gemm_gelu_weight_plan(const ibert_gemm_desc* desc, const ibert_gelu_params* gelu, int32_t plan[3], uint8_t* readers, uint8_t* ahead)
{
    if (!desc || !gelu || !plan || !readers || !ahead) return IBERT_ERR_NULL;
    const int rc = ibert::check_gelu(*gelu);
    return rc ? rc : ibert::weight_plan(*desc, gelu, plan, readers, ahead);
}

extern "C" void ibert_gemm_xcd_blocks(int32_t on) { ibert::g_xcd_blocks = on != 0; }

extern "C" void ibert_gemm_epilogue_record(uint32_t* device_word) { ibert::g_path_word = device_word; }

extern "C" int ibert_gemm_i8_requant(const ibert_gemm_desc* desc, const int8_t* A, const int8_t* W,
                                     const int32_t* bias, const int32_t* mult, const int32_t* shift,
                                     const int8_t* residual, void* C, void* stream)
{
    if (!desc) return IBERT_ERR_NULL;
    const int rc = ibert::check_gemm(*desc, A, W, mult, shift, residual, C);
    if (rc) return rc;
    return ibert::launch_gemm(*desc, A, W, bias, mult, shift, residual, C, (hipStream_t)stream);
}

extern "C" int ibert_gemm_i8_gelu(const ibert_gemm_desc* desc, const int8_t* A, const int8_t* W, const int32_t* bias,
                                  const int32_t* mult, const int32_t* shift, const ibert_gelu_params* gelu,
                                  int8_t* C, int32_t* scratch, void* stream)
{
    if (!desc || !gelu) return IBERT_ERR_NULL;
    int rc = ibert::check_gelu(*gelu);
    if (rc) return rc;
    ibert_gemm_desc d = *desc;
    d.out_dtype = IBERT_I32;                       // range checks of the MatMul part: an INT32 result clamped to q_max
    d.out_clamp = gelu->q_max;
    rc = ibert::check_gemm(d, A, W, mult, shift, nullptr, C);
    if (rc) return rc;
    return ibert::launch_gemm_gelu(*desc, A, W, bias, mult, shift, *gelu, C, scratch, (hipStream_t)stream);
}
