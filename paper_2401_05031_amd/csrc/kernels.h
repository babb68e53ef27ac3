// Host-side launchers of the gfx950 kernels.  Internal to the library: the public surface is the
// C ABI in include/otas.h.  dtype is an otas_dtype value; every pointer is a device pointer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace otas {

enum Epilogue { EPI_NONE = 0, EPI_GELU = 1, EPI_RESIDUAL = 2, EPI_PARTIAL = 3 /* internal: raw float sums */ };

// Sets hipFuncAttributeMaxDynamicSharedMemorySize once per (kernel, device); thread-safe.
hipError_t set_max_dynamic_lds(const void* kernel, int bytes);

// One wave busy for `ticks` wall-clock periods (hipDeviceAttributeWallClockRate); sink: one int.
hipError_t launch_spin(int64_t ticks, int32_t* sink, hipStream_t s);
// One wave sampling the shader clock against the wall clock; ticks: device [samples]; shader clocks per sample: kClockProbeClocks.
constexpr int kClockProbeClocks = 4 * 127 * 64;
hipError_t launch_clock_probe(uint32_t* ticks, int32_t samples, hipStream_t s);
hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
hipError_t launch_copy_i32(const int32_t* src, int32_t* dst, int64_t n, hipStream_t s);

// Plans of up to kArgInts entries travel in a kernel's arguments: such a launcher reads the host array `plan` and never
// d_plan; larger ones must have been copied to d_plan.  HIP promises a kernel 4 KB of arguments; the implicit ones that
// the compiler adds to kernels that ask for gridDim or blockDim (256 bytes) count as well, so kernels that take a plan ask
// for neither.  A test reads what every built kernel takes.
constexpr int kArgInts = 960;
constexpr size_t kKernelArgBytes = 4096;
inline bool plan_in_args(size_t count) { return count <= (size_t)kArgInts; }

// plan: tok_off [B+1] | prm_beg [B] | prm_cnt [B] | out_off [B+1]; query q takes rows prm_beg[q] .. + prm_cnt[q] - 1 of
// the prompt tensor.
hipError_t launch_prepend(int dtype, const void* tokens, const void* prompts, void* out, const int32_t* plan,
                          size_t count, const int32_t* d_plan, int B, int max_n_out, int D, int n_lead, hipStream_t s);

// Prompting module in front of a layer l >= 1 on the float residual stream: overwrite the P prompt
// rows of every query in place (grow = false, x_new == x_old) or insert P rows at n_lead while
// copying into another buffer (grow = true).  prompts: this layer's rows, model dtype.  max_rows:
// the largest number of rows one query writes (P, or its new length).
hipError_t launch_deep_prompt(int dtype, const float* x_old, float* x_new, const void* prompts,
                              const int32_t* d_old_off, const int32_t* d_new_off, const int32_t* d_prm_off, int B,
                              int max_rows, int D, int n_lead, bool grow, hipStream_t s);

// Model ends.  patchify: images [B, C, Hi, Wi] -> patch matrix [B N, C p p] (patches row by row,
// flattened channel-major).  embed_finish: tokens [B, n_lead + N, D] = [cls | proj rows] + pos.
// task_heads: logits[q, :K_task] = W_task LN_final(x[off[q]]) + b_task; plan: off [B] | task [B] | pad to an even count |
// a HeadRef per task.
struct HeadRef { const void* w; const void* b; int32_t K; int32_t pad; };   // 24 bytes, 8-byte aligned
hipError_t launch_patchify(int dtype, const void* img, void* out, int B, int C, int Hi, int Wi, int p, hipStream_t s);
hipError_t launch_embed_finish(int dtype, const void* proj, const void* cls, const void* pos, void* tokens, int B,
                               int N, int D, int n_lead, hipStream_t s);
hipError_t launch_task_heads(int dtype, const float* x, const int32_t* plan, size_t count, const int32_t* d_plan,
                             const void* g, const void* b, int B, int D, float eps, float* logits, int k_max,
                             hipStream_t s);

// What the first LayerNorm of a pass does beside its rows, in extra workgroups: it expands the pass's plan from the
// queries' numbers (v: length [B] | r or P [B], by value: the pass needs no copy to the device) and sets up to two
// integer arrays to 1.  The extra workgroups (one per layer) finish under the rows' own time: the LayerNorm of one ViT-B
// query reads 3.9 us without and 4.4 with them, where the copy (3.9 us) and the fill (4.8 us) were launches of their own.
//   kind START_MERGE: plan = off[l][B+1], l = 0 .. L | r_eff[l][B] | trace_off[l][B], l < L (lengths by the merging rule)
//   kind START_DEEP:  plan = off[l][B+1], l < L, of lengths n + l grow P | prompt offsets [B+1]
enum StartKind { START_MERGE = 0, START_DEEP = 1 };
constexpr int kStartQueries = kArgInts / 2;   // a plan of more queries is built on the host and copied
struct StartJob {
  int32_t* plan;
  int32_t kind, B, L, n_lead, grow;
  int32_t* ones[2];
  int64_t n_ones[2];
  int32_t v[kArgInts];
};
static_assert(sizeof(StartJob) + 64 <= kKernelArgBytes, "the job and the LayerNorm's own arguments");

// x_is_float: the input rows are float (the residual stream) even when dtype is bf16.
hipError_t launch_layer_norm(int dtype, bool x_is_float, const void* x, const void* g, const void* b,
                             void* y, int64_t T, int D, float eps, hipStream_t s, const StartJob* job = nullptr);
// LayerNorm of bf16 rows that also writes the rows out as floats (x_float [T, D]).
hipError_t launch_layer_norm_widen(const void* x_bf16, const void* g, const void* b, void* y, float* x_float,
                                   int64_t T, int D, float eps, hipStream_t s, const StartJob* job = nullptr);

// EPI_RESIDUAL: res and y are float (the residual stream) for every dtype; otherwise y has the
// model's dtype.  model_bytes: the weights of the model whose pass this is part of (0: none; decides with the output's
// size whether it is stored past the caches, no result depends on it).
hipError_t launch_linear(int dtype, const void* x, const void* w, const void* bias,
                         const float* res, void* y, int64_t M, int N, int K, int epi,
                         hipStream_t s, int64_t model_bytes = 0);
bool streams_output(int64_t M, int N, int epi, int64_t model_bytes);

// The same with the kernel named by the caller (tests and profiling exercise every kernel at every
// shape this way): GK_AUTO = launch_linear's own choice, GK_FMA = fp32 arithmetic (any dtype),
// the others bf16 MFMA kernels named by block tile (rows x columns; of GK_64X64 and GK_128_K64 the first of several) and K step.  Returns
// hipErrorInvalidValue if the kernel does not take the shape (K % 32 / K % 64, N % 8).
enum gemm_kernel_id {
  GK_AUTO = 0, GK_FMA = 1, GK_128_K32 = 2, GK_128_K64 = 3, GK_192X256 = 4, GK_256X256 = 5, GK_320X256 = 6,
  GK_64X64 = 7, GK_160X256 = 8, GK_224X256 = 9, GK_288X256 = 10, GK_COUNT = 11
};
// The tiles that kernels 7 and 3 run a shape in (pure host): their results are the same bits.
enum SmallTile { ST_64X64 = 0, ST_32X32 = 1, ST_32X64 = 2, ST_96X64 = 3 };
SmallTile pick_small_tile(int64_t M, int N, int K, int splits);
int wide_rows(int64_t M, int N, int K, int splits);   // 128 or 160
int linear_kernel_choice(int dtype, int64_t M, int N, int K, int epi);   // the id launch_linear runs for this shape
hipError_t launch_linear_kernel(int kernel, int dtype, const void* x, const void* w, const void* bias,
                                const float* res, void* y, int64_t M, int N, int K, int epi, hipStream_t s);

// Split-K form of the residual linear for bf16 models: splitk_factor picks S (1 = do not split);
// launch_linear_splitk writes S float partial products part[S][M][N] of x W^T, each over K / S;
// launch_splitk_reduce_ln then forms x_out = res + bias + sum_s part[s] (s ascending) and, when
// y != nullptr, y = LayerNorm(x_out) with gamma g, beta b in bf16 (the next block's first norm).
int splitk_factor(int dtype, int64_t M, int N, int K, int max_split = 8);
hipError_t launch_linear_splitk(const void* x, const void* w, float* part, int64_t M, int N, int K, int S,
                                hipStream_t s);
// A weight that wgs workgroups beside a launch's own read into the last-level cache for the next linear (wgs = 0: none).
struct WarmWeight { const void* w = nullptr; int64_t bytes = 0; int wgs = 0; };
hipError_t launch_splitk_reduce_ln(const float* part, int S, const void* bias, const float* res, float* x_out,
                                   int64_t M, int D, const void* g, const void* b, void* y, float eps,
                                   hipStream_t s, const WarmWeight& warm = WarmWeight{});

hipError_t launch_attention(int dtype, const void* qkv, const int32_t* sizes,
                            const int32_t* d_off, int B, int max_n, int long_blocks, int D, int H, bool size_bias,
                            void* o, hipStream_t s);
// How a launch of the bf16 attention cuts up its work (pure host): keys staged at a time, waves per head and row block, of which kg share
// 32 rows, whether the row blocks of a head go to one XCD.  The results are the same bits in every shape.
struct AttnShape {
  int kc, nw, kg;
  bool by_head;
};
AttnShape attention_shape(int dh, int H, int B, int max_n, int long_blocks, int others);
// long_blocks of these launches: blocks of 128 rows of the queries that are longer than half the longest one, max_n.
inline int attention_long_blocks(const int* n, int B, int max_n) {
  int blocks = 0;
  for (int q = 0; q < B; ++q)
    if (2 * n[q] > max_n) blocks += (n[q] + 127) / 128;
  return blocks;
}

// Attention and the merge plan of one layer in a single launch (bf16 models of head width 64, and f32 models, whose launch
// takes the selection only; the plan's metric is the head mean of the keys in qkv).  Returns hipErrorInvalidValue, having launched nothing, for what attention_plan_how
// does not take.
// With sel_best / sel_bcol (device, nb arrays of sel_stride entries, one per packed token row) the launch runs only the
// plan's selection (every A token's best match), in na x nb workgroups per query, and leaves it there; the lists are then
// written by the first B workgroups of launch_linear_plan_tail, beside the attention output projection.  With both NULL
// it runs the whole plan, one workgroup per query, whose metric rows must fit the LDS.
struct FusedPlan { int na, nb; };   // na = 0: not taken
FusedPlan attention_plan_how(int dtype, int B, int max_n, int D, int H, bool lists_elsewhere);
hipError_t launch_attention_plan(int dtype, const void* qkv, const int32_t* sizes, const int32_t* d_off, const int32_t* d_out_off,
                                 const int32_t* d_reff, const int32_t* d_troff, int B, int max_n, int long_blocks, int D, int H,
                                 bool size_bias, int n_lead, void* o, int32_t* src_list, int32_t* row_ptr,
                                 int32_t* trace_src, int32_t* trace_dst, float* sel_best, int32_t* sel_bcol,
                                 int64_t sel_stride, hipStream_t s);

// What the list phases of the merge plan (merge_plan_lists) need when they run inside another kernel's launch.
struct PlanTail {
  const int32_t *in_off, *out_off, *reff, *troff;   // device: per-query offsets in / out, r_eff, trace offsets
  int32_t *src_list, *row_ptr, *trace_src, *trace_dst;
  const float* best;                                // the selection's result: nb arrays of `stride` entries, one per
  const int32_t* bcol;                              // packed token row
  int64_t stride;
  int nb;
  int B;                                            // queries = leading workgroups that run the lists
};
// y = x W^T + bias + res (operands of the model's type, float residual in and out) as launch_linear with EPI_RESIDUAL, and in
// the same launch the list phases of the merge plan for tail.B queries of at most max_n tokens.
// hipErrorInvalidValue, having launched nothing, when no kernel with such a form takes the shape.  linear_plan_tail_fits: whether
// the launch's last round has B workgroup slots to spare (pure host); if not, the lists are better written elsewhere.
bool linear_plan_tail_fits(int dtype, const void* x, const void* w, int64_t M, int N, int K, int B);
hipError_t launch_linear_plan_tail(int dtype, const void* x, const void* w, const void* bias, const float* res, void* y,
                                   int64_t M, int N, int K, const PlanTail& tail, int max_n, hipStream_t s);

// The metric of token i is the mean over H heads of src[i * row_stride + col_off + h * dm + c]
// (dtype = type of src), normalised to unit length inside the kernel.  The kernel keeps a query's unit
// metric rows in LDS when merge_plan_lds_bytes(max_n, dm) <= 160 KB; otherwise in `rows`, a device
// buffer of merge_plan_rows_bytes(T, dm) bytes for the T packed tokens (16-byte aligned; may be NULL
// when every query fits LDS, else the launch fails with hipErrorInvalidValue).
hipError_t launch_merge_plan(int dtype, const void* src, int64_t row_stride, int col_off, int H, int dm,
                             const int32_t* d_in_off, const int32_t* d_out_off, const int32_t* d_reff,
                             const int32_t* d_troff, int B, int max_n, int n_lead, int32_t* src_list,
                             int32_t* row_ptr, int32_t* trace_src, int32_t* trace_dst, float* rows, hipStream_t s);
// The same for a metric of its own ([T, dm], one "head"), the query's numbers from a host plan:
// in_off [B+1] | out_off [B+1] | r_eff [B] | trace_off [B].
hipError_t launch_merge_plan_host(int dtype, const void* metric, int dm, const int32_t* plan, size_t count,
                                  const int32_t* d_plan, int B, int max_n, int n_lead, int32_t* src_list,
                                  int32_t* row_ptr, int32_t* trace_src, int32_t* trace_dst, float* rows, hipStream_t s);
// The merging module as an operator of its own in two launches that share out a query's work between workgroups: the selection
// (every A token's best match into best / bcol, an entry per packed token row), then the lists, in LDS, with the averages.
// Arguments as above; D columns of x.  token_merge_in_two: whether B queries of up to max_n tokens are run this way (pure host);
// if not, the two launchers return hipErrorInvalidValue.
bool token_merge_in_two(int B, int max_n, int dm);
hipError_t launch_merge_select_host(int dtype, const void* metric, int dm, const int32_t* plan, size_t count, const int32_t* d_plan,
                                    int B, int max_n, int n_lead, float* best, int32_t* bcol, hipStream_t s);
hipError_t launch_merge_lists_apply_host(int dtype, const void* x, const int32_t* sizes, int dm, const float* best, const int32_t* bcol,
                                         const int32_t* plan, size_t count, const int32_t* d_plan, int B, int max_n, int D,
                                         void* x_out, int32_t* sizes_out, int32_t* trace_src, int32_t* trace_dst, hipStream_t s);
size_t merge_plan_lds_bytes(int max_n, int dm);
size_t merge_plan_rows_bytes(int64_t T, int dm);

// dtype: type of x and x_out (0 = float, 1 = bf16).
hipError_t launch_merge_apply(int dtype, const void* x, const int32_t* sizes,
                              const int32_t* src_list, const int32_t* row_ptr, int64_t T_in,
                              int64_t T_out, int D, void* x_out, int32_t* sizes_out,
                              hipStream_t s);

// merge-apply on the float residual stream fused with the following LayerNorm: writes the merged
// rows x_out (float), their sizes, and y = LN(x_out) in the model's dtype (gamma, beta of that dtype).
hipError_t launch_merge_apply_ln(int dtype, const float* x, const int32_t* sizes, const int32_t* src_list,
                                 const int32_t* row_ptr, int64_t T_in, int64_t T_out, int D, float* x_out,
                                 int32_t* sizes_out, const void* g, const void* b, void* y, float eps,
                                 hipStream_t s, const WarmWeight& warm = WarmWeight{});

}  // namespace otas
