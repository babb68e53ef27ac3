// The merging module (Sec. II-C): bipartite matching on cosine similarity, top-r edges, then a
// size-weighted average and an order-preserving compaction.
//
//   merge_plan_kernel  -- one workgroup per query.  It forms the row-normalised metric vectors
//       (head mean of the keys) in LDS and from them computes, in integers, everything the data
//       movement needs: for every surviving token the
//       list of input rows that are averaged into it.  Written as a CSR over the *output* rows of
//       the whole packed batch: row_ptr[j] .. row_ptr[j+1] indexes src_list, whose first entry is
//       the surviving token itself followed by its merged sources in ascending position.
//   merge_apply_kernel -- one or two 16-byte chunks of one output row per thread: gathers the listed rows,
//       accumulates size * x in fp32 in list order, divides by the summed size.  Reads every input
//       row once and writes every output row once, with no atomics, so results are deterministic.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "merge_plan_body.h"
#include "plan_args.h"

namespace otas {

// Everything but the metric rows.
static inline size_t plan_small_lds_bytes(int max_n) {
  const size_t nA = (max_n + 1) / 2, nB = max_n / 2;
  return sizeof(float) * (3 * nA + nB + 2 * (size_t)max_n + 32 + 8 + 2 * 512);
}
size_t merge_plan_lds_bytes(int max_n, int dm) {
  return sizeof(float) * (size_t)max_n * plan_row_floats(dm) + plan_small_lds_bytes(max_n);
}
size_t merge_plan_rows_bytes(int64_t T, int dm) { return sizeof(float) * (size_t)T * plan_row_floats(dm); }

// One workgroup of 1024 threads per query: merge_plan_body (merge_plan_body.h).  P: where the query's numbers come from.
struct PlanPointers {
  const int32_t *in_off, *out_off, *reff, *troff;   // device arrays
  __device__ PlanQuery query(int q, int) const { return plan_query(in_off, out_off, reff, troff, q); }
};
template <typename I> struct PlanInts {             // in_off [B+1] | out_off [B+1] | r_eff [B] | trace_off [B]
  I v;
  __device__ PlanQuery query(int q, int B) const {
    return PlanQuery{v[q], v[q + 1] - v[q], v[B + 1 + q], v[2 * B + 2 + q], v[3 * B + 2 + q]};
  }
};
template <typename T, bool ROWS_IN_LDS, typename P>
__global__ __launch_bounds__(kPlanThreads) void merge_plan_kernel(
    const T* __restrict__ src, int64_t row_stride, int col_off, int H, int dm, const P plan, int B, int n_lead,
    int32_t* __restrict__ src_list, int32_t* __restrict__ row_ptr, int32_t* __restrict__ trace_src,
    int32_t* __restrict__ trace_dst, float* rows) {
  extern __shared__ float lds[];
  const PlanQuery pq = plan.query((int)blockIdx.x, B);
  merge_plan_body<T, ROWS_IN_LDS>(src, row_stride, col_off, H, dm, pq, n_lead, src_list, row_ptr, trace_src, trace_dst,
                                  rows, lds, (int)threadIdx.x);
}

template <typename P>
static hipError_t merge_plan(int dtype, const void* src, int64_t row_stride, int col_off, int H, int dm, const P& plan,
                             int B, int max_n, int n_lead, int32_t* src_list, int32_t* row_ptr, int32_t* trace_src,
                             int32_t* trace_dst, float* rows, hipStream_t s) {
  if (B <= 0 || max_n <= 0) return hipSuccess;
  if (dm % 4 != 0 || dm > 128 || max_n > kPlanThreads) return hipErrorInvalidValue;
  const bool in_lds = merge_plan_lds_bytes(max_n, dm) <= 160 * 1024;
  if (!in_lds && !rows) return hipErrorInvalidValue;
  const size_t lds = in_lds ? merge_plan_lds_bytes(max_n, dm) : plan_small_lds_bytes(max_n);
#define OTAS_PLAN(TYPE, IN_LDS)                                                                                  \
  do {                                                                                                           \
    auto kern = merge_plan_kernel<TYPE, IN_LDS, P>;                                                              \
    hipError_t e = set_max_dynamic_lds((const void*)kern, 160 * 1024);                                           \
    if (e != hipSuccess) return e;                                                                               \
    kern<<<dim3(B), dim3(kPlanThreads), lds, s>>>((const TYPE*)src, row_stride, col_off, H, dm, plan, B, n_lead, \
                                                  src_list, row_ptr, trace_src, trace_dst, rows);                \
  } while (0)
  if (dtype == 0) {
    if (in_lds) OTAS_PLAN(float, true); else OTAS_PLAN(float, false);
  } else {
    if (in_lds) OTAS_PLAN(bf16_t, true); else OTAS_PLAN(bf16_t, false);
  }
#undef OTAS_PLAN
  return hipGetLastError();
}

hipError_t launch_merge_plan(int dtype, const void* src, int64_t row_stride, int col_off, int H, int dm,
                             const int32_t* d_in_off, const int32_t* d_out_off, const int32_t* d_reff,
                             const int32_t* d_troff, int B, int max_n, int n_lead, int32_t* src_list,
                             int32_t* row_ptr, int32_t* trace_src, int32_t* trace_dst, float* rows, hipStream_t s) {
  return merge_plan(dtype, src, row_stride, col_off, H, dm, PlanPointers{d_in_off, d_out_off, d_reff, d_troff}, B, max_n,
                    n_lead, src_list, row_ptr, trace_src, trace_dst, rows, s);
}

hipError_t launch_merge_plan_host(int dtype, const void* metric, int dm, const int32_t* plan, size_t count,
                                  const int32_t* d_plan, int B, int max_n, int n_lead, int32_t* src_list,
                                  int32_t* row_ptr, int32_t* trace_src, int32_t* trace_dst, float* rows, hipStream_t s) {
  return with_plan(plan, count, d_plan, [&](const auto& v) {
    return merge_plan(dtype, metric, dm, 0, 1, dm, PlanInts<std::decay_t<decltype(v)>>{v}, B, max_n, n_lead, src_list,
                      row_ptr, trace_src, trace_dst, rows, s);
  });
}

// ------------------------------------------------------------------------------------ apply
constexpr int64_t kApplyThreads = 256 * 2048;   // what the chip holds at a time
// A thread takes U chunks of an output row, `per` apart (per = chunks of a row / U, rounded up): the chain list bounds ->
// sources -> rows costs the launch a round trip each per round of workgroups the chip holds, so a large call has fewer
// threads with more loads each.  11584 x
// 768 rows out of 12608 (MI355X): 8.5 us with one chunk a thread and 64-bit indices, 8.2 so; a call 23.7 -> 23.35.
template <typename T, int U>
__global__ __launch_bounds__(256) void merge_apply_kernel(const T* __restrict__ x, const int32_t* __restrict__ sizes,
                                                          const int32_t* __restrict__ src_list,
                                                          const int32_t* __restrict__ row_ptr, int64_t T_in,
                                                          int64_t T_out, int D, T* __restrict__ x_out,
                                                          int32_t* __restrict__ sizes_out) {
  constexpr int V = Vec<T>::N;
  const int chunks = D / V, per = (chunks + U - 1) / U;
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;   // a launch holds fewer than 2^32 threads
  const int64_t j = t / (uint32_t)per;
  if (j >= T_out) return;
  const int c0 = (int)(t - (uint32_t)j * (uint32_t)per);
  const int beg = row_ptr[j];
  const int end = (j + 1 < T_out) ? row_ptr[j + 1] : (int)T_in;
  const int first = src_list[beg];
  if (end - beg == 1) {  // untouched token: plain copy
    const T* p = x + (size_t)first * D;
    Vec<T> v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = load_vec<T>(p + min(c0 + u * per, chunks - 1) * V);
    if (c0 == 0) sizes_out[j] = sizes ? sizes[first] : 1;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c0 + u * per < chunks) store_vec<T>(x_out + (size_t)j * D + (c0 + u * per) * V, v[u]);
    return;
  }
  float acc[U][V];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int k = 0; k < V; ++k) acc[u][k] = 0.f;
  int tot = 0;
  for (int e = beg; e < end; ++e) {
    const int srow = src_list[e];
    const int sz = sizes ? sizes[srow] : 1;
    const float w = (float)sz;
    tot += sz;
    const T* p = x + (size_t)srow * D;
    Vec<T> v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = load_vec<T>(p + min(c0 + u * per, chunks - 1) * V);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < V; ++k) acc[u][k] = fmaf(w, v[u].get(k), acc[u][k]);
  }
  const float denom = (float)tot;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (c0 + u * per < chunks) {
      Vec<T> o;
#pragma unroll
      for (int k = 0; k < V; ++k) o.set(k, acc[u][k] / denom);
      store_vec<T>(x_out + (size_t)j * D + (c0 + u * per) * V, o);
    }
  if (c0 == 0) sizes_out[j] = tot;
}

template <typename T>
static hipError_t merge_apply(const void* x, const int32_t* sizes, const int32_t* src_list, const int32_t* row_ptr,
                              int64_t T_in, int64_t T_out, int D, void* x_out, int32_t* sizes_out, hipStream_t s) {
  const int64_t chunks = D / Vec<T>::N, all = T_out * chunks;
  const int U = all > kApplyThreads ? 2 : 1;
  const int64_t tasks = T_out * ((chunks + U - 1) / U);
  const dim3 grid((unsigned)((tasks + 255) / 256)), block(256);
  if (tasks > ((int64_t)1 << 32) - 256) return hipErrorInvalidValue;   // more threads than a launch holds
#define OTAS_APPLY(UU)                                                                                          \
  merge_apply_kernel<T, UU><<<grid, block, 0, s>>>((const T*)x, sizes, src_list, row_ptr, T_in, T_out, D,       \
                                                   (T*)x_out, sizes_out)
  if (U == 1) OTAS_APPLY(1);
  else OTAS_APPLY(2);
#undef OTAS_APPLY
  return hipGetLastError();
}

hipError_t launch_merge_apply(int dtype, const void* x, const int32_t* sizes, const int32_t* src_list,
                              const int32_t* row_ptr, int64_t T_in, int64_t T_out, int D, void* x_out,
                              int32_t* sizes_out, hipStream_t s) {
  if (T_out <= 0) return hipSuccess;
  return dtype == 0 ? merge_apply<float>(x, sizes, src_list, row_ptr, T_in, T_out, D, x_out, sizes_out, s)
                    : merge_apply<bf16_t>(x, sizes, src_list, row_ptr, T_in, T_out, D, x_out, sizes_out, s);
}

}  // namespace otas
