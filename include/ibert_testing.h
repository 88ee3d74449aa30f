/*
 * libibert -- hooks for tests and tuning runs.  Not part of the method and not needed by a user of the library:
 * nothing here changes a result.
 */
#ifndef IBERT_TESTING_H
#define IBERT_TESTING_H

#include <stdint.h>

#include "ibert.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Force tile configuration `config` (0 .. count-1) of the MFMA MatMul kernel for every later MatMul launch of this
 * process that takes the 16-byte aligned path; a negative value restores the built-in choice.  Returns the number of
 * configurations.  Process-wide and not thread-safe: for single-threaded tests that walk the kernel's instantiations
 * (Sec. 4.1's MatMuls are the same arithmetic under every tiling). */
int ibert_gemm_config_override(int32_t config);

/* Switch for A/B measurements: with `on` = 0 the MFMA MatMul gives each XCD a linear run of tiles instead of a near-square
 * block of the tile grid (the default, which fetches fewer operand bytes over the fabric).  Process-wide.  The persistent and
 * the few-token kernels deal their tiles to the XCDs in ways of their own, which it does not change. */
void ibert_gemm_xcd_blocks(int32_t on);

/* Name and tile parameters of the kernel that this process launched last, as a profiler shows them ("" before the first launch).
 * Not thread-safe. */
const char* ibert_last_kernel(void);

/* While `device_word` (device uint32, owned by the caller) is non-NULL, every launch of the MFMA MatMul and of its persistent
 * form has its first workgroup store there which form of the epilogue it ran -- the choice depends on the per-channel shifts
 * and biases, which only the device sees.  The few-token kernel (ibert_last_kernel() tells) chooses the arithmetic for every
 * wavefront and stores nothing: the test for it alone made the forward of one sequence 0.8 % slower.  NULL switches the record
 * off.  Process-wide, not thread-safe. */
enum {
    IBERT_EPILOGUE_STAGED = 1,            /* through LDS, general 64-bit requantization, arithmetic GELU          */
    IBERT_EPILOGUE_DIRECT = 2,            /* register-direct (all shifts in [33, 62], |bias| < 2^30)              */
    IBERT_EPILOGUE_DIRECT_GELU_TABLE = 3, /* register-direct, GELU read from the workgroup's table in LDS         */
    IBERT_EPILOGUE_EDGE = 4               /* a tile on the edge of the output, or unaligned output rows           */
};
void ibert_gemm_epilogue_record(uint32_t* device_word);

/* The form in which the one-kernel attention computes with these parameters in a launch of `workgroups` (batch x heads x ceil(seq / 64)) that
 * stores neither scores nor probabilities: 0 any constants, 1 and 2 faster ones (scores' shift at least 32, and below), 3 and 4 those with a
 * table of the exponent (scores' shift up to 33, and above).  Host only. */
int ibert_attention_form(const ibert_dyadic* scores_dy, const ibert_softmax_params* softmax, const ibert_dyadic* ctx_dy, int64_t workgroups, int32_t* form);

/* How the one-kernel attention (Alg. 3 between its two MatMuls) holds K_h and V_h for 385 <= seq <= 512 (forms 3 and 4 from 321 on): *shared = 1 where a launch of
 * `workgroups` (batch x heads x ceil(seq / 64)) has them take turns in one LDS buffer, 0 where each has its own; *fit_two, *fit_one =
 * workgroups that a compute unit holds at once with two buffers and with one.  form: see ibert_attention_form (3 and 4:
 * fit_* with the largest table).  Asks the device. */
int ibert_attention_buffers(int32_t seq, int32_t form, int64_t workgroups, int32_t* shared, int32_t* fit_two, int32_t* fit_one);

/* How ibert_layernorm_i16 takes `rows` aligned rows: *rows_of_wavefront = 1 or 4 rows to a wavefront of layernorm_many_kernel, 0 where it is
 * layernorm_rows_kernel.  (The name that ibert_last_kernel() gives is the same for 1 and 4.)  Host only. */
int ibert_layernorm_i16_plan(int64_t rows, int32_t C, int32_t shift, int32_t* rows_of_wavefront);

/* Steps 1 to 4 of a layer as one kernel: 0 never; a tile (1000 wavefronts + 100 MFMA rows of one + 10 sequences + stages, one of those ibert_qkv_attention_plan names)
 * wherever its rows hold a sequence and the parameters allow it; negative where it is the faster way (the default).  Process-wide, not thread-safe. */
void ibert_qkv_attention_override(int32_t tile);

/* How that kernel deals a layer of heads of 64: *tile as above; IBERT_ERR_NOT_IMPLEMENTED where the choice is to run the steps apart.  places[batch * heads] (zeroed): how often a
 * (sequence, head) is worked on.  readers[3 * heads] (zeroed): bit x is set where XCD x multiplies the head's rows of W_q, W_k, W_v.  ahead[x * 3 H H / 1024 + i] (zeroed): how
 * often XCD x reads the i-th KB of W_qkv ahead when an encoder plans for it (H = 64 heads).  The choice is that for a layer called by itself.  Host only. */
int ibert_qkv_attention_plan(int32_t batch, int32_t seq, int32_t heads, int32_t* tile, uint8_t* places, uint8_t* readers, uint8_t* ahead);

/* The tile that a call of `layers` layers takes where the parameters allow that kernel, 0 where it runs the steps apart; no override.  Host only. */
int ibert_qkv_attention_chosen(int32_t batch, int32_t seq, int32_t heads, int32_t layers, int32_t* tile);

/* What the XCDs read of W [N, K] (dense rows, K a multiple of 128, N * K of 1024) when this MatMul runs with all operands aligned, and
 * what each reads ahead when an encoder plans for it.  plan: the tile configuration chosen, then rows and xs: XCD x is to have the row
 * blocks (j << xs) + x % 2^xs of `rows` rows each.  readers[n] (N bytes, zeroed by the caller): bit x is set where a workgroup on XCD x
 * multiplies row n, by the kernel's own dealing of tiles.  ahead[x * N K / 1024 + i] (8 N K / 1024 bytes, zeroed): how often XCD x reads
 * the i-th KB ahead, by the attention kernel's own arithmetic (nothing of a W above 32 MB).  gelu: with the GELU epilogue,
 * at an input scale of 2^-6 and an output scale of 8 / 127.  IBERT_ERR_NOT_IMPLEMENTED: nothing is planned for such operands; IBERT_ERR_SHAPE: a read past the end of W.  Host only. */
int ibert_gemm_weight_plan(const ibert_gemm_desc* desc, int32_t gelu, int32_t plan[3], uint8_t* readers, uint8_t* ahead);

/* The same with the GELU epilogue at these parameters, whose table some tiles have no room for. */
int ibert_gemm_gelu_weight_plan(const ibert_gemm_desc* desc, const ibert_gelu_params* gelu, int32_t plan[3], uint8_t* readers, uint8_t* ahead);

#ifdef __cplusplus
}
#endif
#endif /* IBERT_TESTING_H */
