// Shared declarations of the libibert sources: error plumbing, device-side integer helpers,
// internal launcher prototypes.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdio>

#include "ibert.h"

namespace ibert {

// Records the text of a failed HIP call for ibert_last_hip_error().
int hip_failed(hipError_t e, const char* what);

#define IBERT_HIP_CHECK(expr)                                         \
    do {                                                              \
        hipError_t _e = (expr);                                       \
        if (_e != hipSuccess) return ::ibert::hip_failed(_e, #expr);  \
    } while (0)

// Launch check: kernels are enqueued asynchronously, so only launch-time errors show up here.
#define IBERT_LAUNCH_CHECK(name)                                        \
    do {                                                                \
        hipError_t _e = hipGetLastError();                              \
        if (_e != hipSuccess) return ::ibert::hip_failed(_e, name);     \
    } while (0)

inline bool dyadic_ok(const ibert_dyadic& d) { return d.s >= 0 && d.s <= 62; }
inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// ---- device helpers -------------------------------------------------------------------------
// Requantization: round-half-up of x*m/2^s, exact in 64 bits (|x|,|m| < 2^31, s <= 62).
__device__ __forceinline__ int64_t dyadic64(int32_t x, int32_t m, int32_t s)
{
    int64_t p = (int64_t)x * (int64_t)m;
    if (s > 0) p = (p + ((int64_t)1 << (s - 1))) >> s;
    return p;
}

__device__ __forceinline__ int32_t clamp_i64_to_i32(int64_t v, int32_t lim)
{
    const int64_t l = lim;
    v = v < -l ? -l : v;
    v = v > l ? l : v;
    return (int32_t)v;
}

__device__ __forceinline__ int32_t clamp_i32(int32_t v, int32_t lo, int32_t hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

// Packs four values already inside [-128,127] into one little-endian dword.
__device__ __forceinline__ uint32_t pack4_i8(int32_t a, int32_t b, int32_t c, int32_t d)
{
    return (uint32_t)(a & 0xff) | ((uint32_t)(b & 0xff) << 8) | ((uint32_t)(c & 0xff) << 16) |
           ((uint32_t)(d & 0xff) << 24);
}

// clamp(v, lo, hi) for lo <= hi in one instruction (constant bounds: the compiler finds it by itself).
template <int LO, int HI>
__device__ __forceinline__ int32_t med3_const(int32_t v)
{
    v = v < LO ? LO : v;
    return v > HI ? HI : v;
}
__device__ __forceinline__ int32_t med3_i32(int32_t v, int32_t lo, int32_t hi)
{
    int32_t r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
    return r;
}

// Full-rate 24-bit multiplies (low 32 bits of the product of the operands' low 24 bits) and multiply-adds.  The LLVM
// intrinsics are declared by name: an add of their result is selected as one v_mad_*24 (from the C expression the compiler
// tends to pick a 64-bit multiply-add), and, unlike inline assembly, the scheduler can move them -- behind an asm block it
// also has to put an s_nop in front of the next reader of the result (softmax row: a fifth of the instructions).
__device__ uint32_t llvm_mul_u24(uint32_t a, uint32_t b) __asm("llvm.amdgcn.mul.u24.i32");
__device__ int32_t llvm_mul_i24(int32_t a, int32_t b) __asm("llvm.amdgcn.mul.i24.i32");
__device__ __forceinline__ uint32_t umul24(uint32_t a, uint32_t b) { return llvm_mul_u24(a, b); }
__device__ __forceinline__ int32_t smul24(int32_t a, int32_t b) { return llvm_mul_i24(a, b); }
__device__ __forceinline__ uint32_t umad24(uint32_t a, uint32_t b, uint32_t c) { return llvm_mul_u24(a, b) + c; }
__device__ __forceinline__ int32_t smad24(int32_t a, int32_t b, int32_t c)
{
    return (int32_t)((uint32_t)llvm_mul_i24(a, b) + (uint32_t)c);
}

// Four values already inside [-128,127] -> one dword, three byte permutes.
__device__ __forceinline__ uint32_t pack4_perm(int32_t a, int32_t b, int32_t c, int32_t d)
{
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);   // a.b0, b.b0, 0, 0
    const uint32_t hi = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// Cross-lane moves inside a row of 16 lanes (DPP): butterfly partners for all-reduce.
//   0xB1 quad_perm(1,0,3,2)  0x4E quad_perm(2,3,0,1)  0x141 row_half_mirror  0x140 row_mirror
template <int CTRL>
__device__ __forceinline__ int32_t dpp_mov(int32_t v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}

// op of a value and its partner 16 or 32 lanes away, in every lane: swapping rows of lanes between two copies of a register
// leaves the two operands in two registers, without the trip through LDS that a lane permute takes.
template <typename Op>
__device__ __forceinline__ int32_t combine_rows16(int32_t v, Op op)
{
    const auto t = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    return op((int32_t)t[0], (int32_t)t[1]);
}
template <typename Op>
__device__ __forceinline__ int32_t combine_rows32(int32_t v, Op op)
{
    const auto t = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return op((int32_t)t[0], (int32_t)t[1]);
}

// All-reduce over groups of LPR consecutive lanes (LPR = 16, 32 or 64; groups are aligned).
template <int LPR, typename Op>
__device__ __forceinline__ int32_t group_allreduce(int32_t v, Op op)
{
    v = op(v, dpp_mov<0xB1>(v));
    v = op(v, dpp_mov<0x4E>(v));
    v = op(v, dpp_mov<0x141>(v));
    v = op(v, dpp_mov<0x140>(v));
    if (LPR > 16) v = combine_rows16(v, op);
    if (LPR > 32) v = combine_rows32(v, op);
    return v;
}

// floor(n / d) for 0 <= n < 2^31 with magic = floor(2^32 / d) + 1 (0 for d == 1): the estimate is the quotient or one more.
__host__ __device__ __forceinline__ int32_t udiv_fix(int32_t n, int32_t d, uint32_t magic)
{
    if (magic == 0) return n;
#if defined(__HIP_DEVICE_COMPILE__)
    const int32_t q = (int32_t)__umulhi((uint32_t)n, magic);
#else
    const int32_t q = (int32_t)(((uint64_t)(uint32_t)n * magic) >> 32);
#endif
    return n - q * d < 0 ? q - 1 : q;
}
inline uint32_t udiv_magic(int32_t d) { return d == 1 ? 0u : (uint32_t)(((uint64_t)1 << 32) / (uint32_t)d) + 1u; }

// Name of the kernel family chosen by the most recent launch_* call (for the optional profile).
extern const char* g_last_kernel;

// A kernel's name as a profiler shows it, for static objects: made once, also where several threads launch first together.
struct KernelName {
    char text[96];
    template <typename... A>
    KernelName(const char* format, A... a) { std::snprintf(text, sizeof text, format, a...); }
};

// How the XCDs will share the weights of a MatMul (gemm.hip: plan_gemm): XCD x works on the row blocks (j << xs) + x % 2^xs,
// j = 0, 1 ..., of `rows` rows each (rows 0: no such plan).
struct GemmPlan {
    int32_t rows = 0, xs = 0;
};
// Weights that the kernels after a launch will read and that it may bring into the L2 of the XCD that reads them: clean lines stay
// in an XCD's L2 from one kernel to the next (2 MB an XCD read again by the next kernel: 2.5 us, from HBM 5.0).
// Not a matrix larger than the L2s of the eight XCDs together: it has left them before it is used, and the launch waits for it.  Forward,
// us, 24 (12 from FFN 32768 on) layers of hidden 1024, without W_1 and W_2 / with them, 128 tokens and 4096: FFN 16384 (16 MB each)
// 1057 / 1023, 4677 / 4488; 32768 (32 MB) 676 / 698, 4000 / 3800; 65536 (64 MB) 1080 / 1232, 7540 / 7650.
struct ReadAhead {
    static constexpr int MOST = 6, APART = 4;            // matrices; of a layer whose steps run apart: W_o, W_1, W_2 and the next layer's W_qkv
    static constexpr int64_t MOST_BYTES = 32 << 20;      // of a matrix
    struct Part {
        const int8_t* p;
        int32_t kb, blocks, xs;        // KB of a row block; row blocks; see GemmPlan
        uint32_t kb_magic;             // see udiv_fix
    } part[MOST];
    int n = 0;
    void add(const int8_t* w, int64_t N, int64_t K, const GemmPlan& plan)
    {
        if (n == MOST || plan.rows < 1 || !aligned(w, 16) || N * K > MOST_BYTES) return;      // (the plan may be of another layer's weights)
        // Where half of the XCDs or more read the same rows, so many copies would cost more than they bring: each KB once then, by any
        // XCD, which brings it as near as the memory-side cache and one L2.  us, Base b32 (W_o and W_2 go to all XCDs): 909 without,
        // 903 with eight copies, 852 with one; Base b1 (an eighth for each): 327 without, 336 by any XCD, 316 by the one that reads.
        const bool own = plan.xs >= 2;
        const int32_t kb = own ? (int32_t)(plan.rows * K / 1024) : 1;
        part[n++] = Part{w, kb, (int32_t)(N * K / 1024 / kb), own ? plan.xs : 3, udiv_magic(kb)};
    }
    ReadAhead()
    {
        for (Part& q : part) q = Part{nullptr, 1, 0, 0, 0};
    }
    // The share of a part that XCD x reads, its KB, and the k-th of them, counted from the part's first.
    static __host__ __device__ __forceinline__ int32_t share(int x, int32_t xs) { return x & ((1 << xs) - 1); }
    static __host__ __device__ __forceinline__ int32_t count(int s, int32_t kb, int32_t blocks, int32_t xs)
    {
        return ((blocks - s + (1 << xs) - 1) >> xs) * kb;
    }
    static __host__ __device__ __forceinline__ int64_t at(int s, int32_t k, int32_t kb, uint32_t kb_magic, int32_t xs)
    {
        const int j = udiv_fix(k, kb, kb_magic);
        return (int64_t)((j << xs) + s) * kb + (k - j * kb);
    }
};

// ---- internal launchers (validated arguments) -----------------------------------------------
int launch_gemm(const ibert_gemm_desc& d, const int8_t* A, const int8_t* W, const int32_t* bias,
                const int32_t* mult, const int32_t* shift, const int8_t* residual, void* C,
                hipStream_t stream, const ibert_gelu_params* gelu = nullptr);
// How launch_gemm will share W (gelu: with the GELU epilogue, whose table decides on the tile too).
GemmPlan plan_gemm(const ibert_gemm_desc& d, const int8_t* A, const int8_t* W, const int32_t* bias, const int32_t* mult,
                   const int32_t* shift, const int8_t* residual, const void* C, const ibert_gelu_params* gelu);
int launch_gemm_gelu(const ibert_gemm_desc& d, const int8_t* A, const int8_t* W, const int32_t* bias,
                     const int32_t* mult, const int32_t* shift, const ibert_gelu_params& gelu, int8_t* C,
                     int32_t* scratch, hipStream_t stream);
bool attention_fused_ok(const int8_t* qkv, const int8_t* ctx, int32_t seq, int32_t hidden, int32_t heads);
bool attention_whole_blocks(int32_t seq);
// scores, probs (optional): where the one-kernel form also stores those two tensors
int launch_attention(const int8_t* qkv, int8_t* ctx, int32_t batch, int32_t seq, int32_t hidden, int32_t heads,
                     ibert_dyadic scores_dy, const ibert_softmax_params& sp, ibert_dyadic ctx_dy, hipStream_t stream,
                     const int32_t* key_lens = nullptr, int32_t* scores = nullptr, int8_t* probs = nullptr,
                     const ReadAhead* ahead = nullptr);
// Steps 1 to 4 as one kernel (qkv_attention.hip): is there one for this problem, and is it the faster way?  alone: for a layer called by itself.
bool qkv_attention_ok(const int8_t* x, const int8_t* w, const int8_t* ctx, int32_t batch, int32_t seq, int32_t hidden, int32_t heads, const ibert_dyadic& scores_dy,
                      const ibert_softmax_params& sp, const ibert_dyadic& ctx_dy, bool alone);
int launch_qkv_attention(const int8_t* x, const int8_t* w, const int32_t* bias, const int32_t* mult, const int32_t* shift, int8_t* qkv, int8_t* ctx, int32_t batch,
                         int32_t seq, int32_t hidden, int32_t heads, const ibert_dyadic& scores_dy, const ibert_softmax_params& sp, const ibert_dyadic& ctx_dy,
                         const int32_t* key_lens, const ReadAhead* ahead, hipStream_t stream);
// Its W_qkv among what is read ahead.
void qkv_attention_ahead(ReadAhead& ahead, const int8_t* w, int32_t batch, int32_t seq, int32_t hidden, int32_t heads);
// key_lens (device, optional): row r keeps its first key_lens[r / rows_per_len] columns
int launch_softmax(const int32_t* x, void* y, int64_t rows, int32_t cols, int64_t ldx, int64_t ldy,
                   const ibert_softmax_params& p, hipStream_t stream, const int32_t* key_lens = nullptr,
                   int64_t rows_per_len = 0);
int launch_gelu(const int32_t* x, int8_t* y, int64_t n, const ibert_gelu_params& p, hipStream_t stream);
int launch_hgelu(const int32_t* x, int8_t* y, int64_t n, const ibert_hgelu_params& p, hipStream_t stream);
int launch_layernorm(const int32_t* x, int8_t* y, int64_t rows, int32_t C, int64_t ldx, int64_t ldy,
                     const int32_t* gamma_q, const int32_t* beta_q, int32_t shift, hipStream_t stream);
int launch_layernorm16(const int16_t* x, int8_t* y, int64_t rows, int32_t C, int64_t ldx, int64_t ldy,
                       const int32_t* gamma_q, const int32_t* beta_q, int32_t shift, hipStream_t stream);
int launch_embedding(const int32_t* ids, const int8_t* tok, const int8_t* pos, int64_t tokens, int32_t seq, int32_t C,
                     int32_t vocab, ibert_dyadic tok_dy, ibert_dyadic pos_dy, const int32_t* gamma_q,
                     const int32_t* beta_q, int32_t shift, int8_t* y, int64_t ldy, hipStream_t stream);

// Parameter validation shared by the public entry points and the layer.
int check_gemm(const ibert_gemm_desc& d, const void* A, const void* W, const void* mult,
               const void* shift, const void* residual, const void* C);
int check_softmax(const ibert_softmax_params& p, int32_t cols);
int check_gelu(const ibert_gelu_params& p);
int check_hgelu(const ibert_hgelu_params& p);
int check_layernorm(int32_t C, int32_t shift);

}  // namespace ibert
