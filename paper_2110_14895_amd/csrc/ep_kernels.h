// Launchers of the stage's HIP kernels (gfx950).  Every launcher enqueues on the
// given stream, allocates nothing and returns the launch status.  Shapes are
// validated by the caller (ep_stage.hip); the launchers re-check the
// divisibility assumptions their kernels make and refuse otherwise.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// GEMM epilogues: C = A . W^T + bias, then ...
enum EpEpilogue {
    EPI_BIAS = 0,       // store (bf16 on the bf16 path, fp32 on the fp32 path)
    EPI_BIAS_GELU = 1,  // exact erf GELU, store
    EPI_BIAS_RESID = 2, // add the fp32 residual, store fp32 (out may alias resid)
    EPI_BIAS_F32 = 3,   // store fp32 (short-M bf16 kernel only: the classifier's logits)
    EPI_PARTIAL = 4     // no bias: the bare fp32 sum over one range of K (ep_bf16_gemm_partial only)
};

// ---- fp32 path -------------------------------------------------------------
// row r of x starts at x + r * ldx
hipError_t ep_f32_layernorm(const float *x, int64_t ldx, const float *g, const float *b, float eps, float *y,
                            int64_t rows, int D, hipStream_t s);
hipError_t ep_f32_gemm(const float *A, const float *W, const float *bias, const float *resid,
                       float *C, int64_t M, int N, int K, int epi, hipStream_t s);
// C = LN(x) . W^T + bias (EPI_BIAS or EPI_BIAS_GELU) in one launch, where that pays and K <= 384
bool ep_f32_ln_gemm_supported(const float *x, const float *W, int64_t M, int N, int K);
hipError_t ep_f32_ln_gemm(const float *x, const float *g, const float *b, float eps, const float *W, const float *bias,
                          float *C, int64_t M, int N, int K, int epi, hipStream_t s);
// what becomes of the two (x and W on 16 bytes, K % 4 == 0, K <= 384) on `cus` compute units, for tests: 0 two launches, 1 and 2
// tiles of 16 and of 32, 3 rows kept in registers
extern "C" int32_t ep_query_f32_ln_route(int64_t M, int32_t N, int32_t K, int32_t cus);
hipError_t ep_f32_attention(const float *qkv, float *o, int B, int T, int D, int H, hipStream_t s);

// ---- bf16 path -------------------------------------------------------------
// x fp32 (row r at x + r * ldx, on 16 bytes, ldx < 2^31) -> y bf16 [rows, D], fp32 statistics
hipError_t ep_bf16_layernorm(const float *x, int64_t ldx, const float *g, const float *b, float eps,
                             uint16_t *y, int64_t rows, int D, hipStream_t s);
// The same after a dense layer whose K was cut into ranges (ep_bf16_gemm_partial): first
// x[r, :] = ((part[0] + part[1] + ... + part[splits-1]) + bias) + x[r, :] in place, in that order, then as above.
// part is [splits, rows, D] fp32; splits 2, 4 or 8.
hipError_t ep_bf16_layernorm_sum(float *x, const float *part, int splits, const float *bias, const float *g,
                                 const float *b, float eps, uint16_t *y, int64_t rows, int D, hipStream_t s);
// The same for the first layer of a stage that takes bf16: x = in, widened, then as above.
hipError_t ep_bf16_layernorm_widen(const uint16_t *in, float *x, const float *g, const float *b, float eps, uint16_t *y,
                                   int64_t rows, int D, hipStream_t s);
// Only the sum: out = ((part[0] + ... + part[splits-1]) + bias) + resid, n = rows * D elements, D % 4 == 0, as fp32
// (then out may alias resid) or rounded to bf16.
hipError_t ep_f32_residual_sum(const float *resid, const float *part, int splits, const float *bias, void *out,
                               bool out_bf16, int64_t rows, int D, hipStream_t s);
hipError_t ep_f32_to_bf16(const float *in, uint16_t *out, int64_t n, hipStream_t s);
// W bf16 [N, K] row by row -> p, the same bytes in the fragment order of ep_gemm_bf16_tile.h, in which every dense layer
// below but the classifier takes its weights; N % 16 == 0, K % 32 == 0
hipError_t ep_bf16_pack_weights(const uint16_t *w, uint16_t *p, int N, int K, hipStream_t s);
// A bf16 [M, K], W bf16 [N, K] in fragment order; out bf16 (EPI_BIAS, EPI_BIAS_GELU) or fp32 (EPI_BIAS_RESID).
// K % 64 == 0, N % 16 == 0; from N = 2^20 on EPI_BIAS_RESID only.
// one_order: every output is one sum over K in order, whatever M is; otherwise a persistent launch may deal its last rows
// in narrow tiles, which add up eight sums (ep_bf16_gemm_narrow_rows tells how many rows).
// after_main: if non-null, recorded on s right after the launch (it covers the rows
// ep_bf16_gemm_main_rows reports: all of them).
hipError_t ep_bf16_gemm(const uint16_t *A, const uint16_t *W, const float *bias,
                        const float *resid, void *C, int64_t M, int N, int K, int epi, bool one_order,
                        hipEvent_t after_main, hipStream_t s);
int64_t ep_bf16_gemm_narrow_rows(int64_t M, int N, int K, int epi);
int64_t ep_bf16_gemm_main_rows(int64_t M, int N, int K);
// whether its steps of K wait where the weights come from memory: tiles of up to 128 rows, whose weights are a microsecond ahead, and
// those of 192 and 256 columns, two steps; not the persistent kernel nor the higher tiles of 128 columns.  splits: the K ranges it is cut into
// RANGES: it is, and waits; PERSISTENT, HIGH: it does not; LARGE: tiles of 192 and 256 columns
enum EpWeightWait { EP_WAITS_PERSISTENT, EP_WAITS_HIGH, EP_WAITS, EP_WAITS_RANGES, EP_WAITS_LARGE };
EpWeightWait ep_bf16_gemm_weight_wait(int64_t M, int N, int K, int epi, int splits, bool one_order);
// device memory that later launches read and a launch may bring nearer (it is not written, and nothing is kept); no bytes: none
struct EpTouch { const void *p; uint32_t bytes; };
// qkv bf16 [B*T, 3D] -> o bf16 [B*T, D]; d_head 64 or 80, T <= 4096 (K and V stream through LDS in chunks)
hipError_t ep_bf16_attention(const uint16_t *qkv, uint16_t *o, int B, int T, int D, int H, EpTouch touch,
                             hipStream_t s);
// whether a launch over these has a wave to spare that touches
bool ep_bf16_attention_touches(int64_t pairs, int T);
bool ep_bf16_attention_supported(int T, int d_head);
// How attention deals the queries of `pairs` (image, head) pairs on `cus` compute units: tiles of qw queries, ng groups
// of tiles to a pair; for tests
extern "C" void ep_query_attention_plan(int64_t pairs, int32_t T, int32_t cus, int32_t *qw, int32_t *ng);

// deterministic fill used by the profiler (values in [-1, 1])
hipError_t ep_fill_pattern(float *x, int64_t n, hipStream_t s);

// the one-tile-per-workgroup kernel with K cut into `splits` ranges: part[r] = A[:, range r] . W[:, range r]^T, fp32 [splits, M, N];
// K % (64 * splits) == 0
hipError_t ep_bf16_gemm_partial(const uint16_t *A, const uint16_t *W, float *part, int64_t M, int N, int K,
                                int splits, hipStream_t s);
// ep_bf16_gemm_partial over many rows (a group of micro-batches) and the sum of its ranges, bias and residual in one launch, the same
// bits: the height of its tiles, 0 where two launches are the faster way
extern "C" int32_t ep_query_ranges_height(int64_t M, int32_t N, int32_t K, int32_t splits);
hipError_t ep_bf16_gemm_ranges(const uint16_t *A, const uint16_t *W, const float *bias, const float *resid, float *C, int64_t M, int N,
                               int K, int splits, hipStream_t s);
// how many ranges the dispatcher wants for a dense layer with fp32 output (1: ep_bf16_gemm as it is); the sums of the
// ranges never take more than EP_RANGE_SUM_BYTES, and layers of more than EP_RANGE_SUM_ROWS rows are not cut
constexpr int64_t EP_RANGE_SUM_BYTES = 32 << 20, EP_RANGE_SUM_ROWS = 1 << 15;
int ep_bf16_gemm_splits(int64_t M, int N, int K);
// What the dispatcher does with a dense layer on the current device (256 compute units where there is none); for
// tests.  epi EPI_PARTIAL: a second MLP layer, cut or not; otherwise uncut with that epilogue.  Rows [m_main, M) of a
// persistent launch are the narrow tiles in front of its walk.
struct EpDensePlan { int32_t splits, persistent, bm, bn, per_cu; int64_t m_main; };      // per_cu: workgroups to a unit
extern "C" void ep_query_dense_plan(int64_t M, int32_t N, int32_t K, int32_t epi, EpDensePlan *out);
// the same with one_order, never cut
extern "C" void ep_query_dense_plan_one_order(int64_t M, int32_t N, int32_t K, int32_t epi, EpDensePlan *out);

// LayerNorm of x and the dense layer behind it (bias, or bias and GELU) in one launch, where that pays (ep_gemm_bf16_rows.hip):
// the bits of ep_bf16_layernorm and ep_bf16_gemm.  touched: the weights have been brought into the memory-side cache, which at 1024 wide
// decides for a first MLP layer (with GELU) on some counts of rows
bool ep_bf16_ln_gemm_supported(int64_t M, int N, int K, int epi, bool touched);
extern "C" int32_t ep_query_ln_gemm_touched_mlp(int64_t M, int32_t N, int32_t K);      // for tests: with GELU, touched
// rows of a panel and the column groups that share one, on `cus` compute units; 0: two launches.  For tests
extern "C" int32_t ep_query_ln_gemm_plan(int64_t M, int32_t N, int32_t K, int32_t epi, int32_t cus, int32_t *groups);
hipError_t ep_bf16_ln_gemm(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                           int64_t M, int N, int K, int epi, bool touched, hipEvent_t after_main, hipStream_t s);

// persistent kernel for large problems (ep_gemm_bf16_persist.hip): 256 x BN tiles, BN = tile_bn
// (256 or 320).  The tile walk covers rows
// [0, m_rows); with fuse_tail the same launch also computes rows [m_rows, M) as 64 x 32 tiles.
bool ep_bf16_gemm_persistent_supported(int64_t M, int N, int K);
// resident workgroups of a launch on the current device: one per compute unit (256 if the device cannot be asked)
int ep_bf16_gemm_persistent_workgroups();
// rows (64, 32 or 16) of the narrow tiles that `wgs` workgroups deal rows past the tile walk in
int ep_bf16_gemm_tail_tile_rows(int tail_rows, int N, int wgs);
hipError_t ep_bf16_gemm_persistent(const uint16_t *A, const uint16_t *W, const float *bias,
                                   const float *resid, void *C, int64_t M, int64_t m_rows, int N,
                                   int K, int epi, int tile_bn, bool fuse_tail, hipStream_t s);

// Shader clock (MHz) and duration of workgroup 0 of the most recent persistent launch that has finished on the
// current device (hipErrorNotReady if none has); copies four counters from the device, so it synchronises.
hipError_t ep_bf16_gemm_persistent_clock(double *shader_mhz, double *seconds);

// dense layers of small and middling batches (ep_gemm_bf16_stream.hip) with the dispatcher's bm x bn tiles, bn <= 128
hipError_t ep_bf16_gemm_stream(int bm, int bn, const uint16_t *A, const uint16_t *W, const float *bias, const float *resid,
                               void *C, int64_t M, int N, int K, int splits, int epi, hipStream_t s);
// bias and residual, K in `splits` ranges as ep_bf16_gemm_partial and its reader add them up
hipError_t ep_bf16_gemm_stream_ranges(int bm, const uint16_t *A, const uint16_t *W, const float *bias, const float *resid, float *C,
                                      int64_t M, int N, int K, int splits, hipStream_t s);

// short-M kernel (ep_gemm_bf16_skinny.hip): 64 x 32 tiles, K dealt to the 8 waves of a workgroup
bool ep_bf16_gemm_skinny_supported(int64_t M, int N, int K);
// packed: W in fragment order (EPI_BIAS_RESID), otherwise row by row (EPI_BIAS_F32)
hipError_t ep_bf16_gemm_skinny(const uint16_t *A, const uint16_t *W, bool packed, const float *bias,
                               const float *resid, void *C, int64_t M, int N, int K, int epi,
                               hipStream_t s);
