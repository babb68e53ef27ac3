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
// The merging module as an operator of its own runs both in other proportions where token_merge_in_two says so
// (launch_merge_select_host, then launch_merge_lists_apply_host):
//   merge_select_kernel      -- the plan's selection, a query's A tokens dealt to several workgroups.
//   merge_lists_apply_kernel -- several workgroups per query, each of which works out the query's lists for itself, in
//       LDS, and averages its share of the output rows.
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

// ------------------------------------------------------------------------------ the operator in two launches
// merge_plan_kernel gives a query one CU, and with it go, one after the other, 5 us of fetching and normalising, 5 of comparing
// and 4 of list making (197 tokens) while most CUs have nothing to do.  Here the A tokens are dealt in blocks of 32 to `na` workgroups a
// query (each compares its blocks with all B tokens), and the lists are made again, in LDS, by every workgroup that
// applies them: nothing but the selection goes through memory.  The lists and sums are what the two other kernels make.
// Measured on MI355X (us a call, bf16, D = 768, merge_plan_kernel and merge_apply_kernel / these two): one query of 50 / 197 / 401 / 577
// tokens 13.0 / 13.1, 16.6 / 14.7, 30.8 / 19.2, 57.9 / 23.1; 16 of them 13.1 / 13.6, 18.0 / 16.2, 34.1 / 21.2, 66.0 / 26.5; 64 14.0 / 14.6, 22.4 /
// 20.1, 43.1 / 34.3, 81.2 / 62.7.  Up to 64 queries, which have four workgroups each that apply.  With three (66 ... 85 queries of 129 ... 577
// tokens, 45 calls at each of three widths) bf16 gains 8 % in the mean (0.96 ... 1.46 times) and float 1 % (0.87 ... 1.33: 85 of 401 at
// D = 1280 loses most); with two (96 ... 128) 0.94 ... 1.10 and 0.85 ... 1.01 times; with one (144) 0.70 ... 0.95.  Workgroups of 256, 512 and 1024 threads that
// apply, 1024, 256 and 256 of them in all: 64 of 197 22.5, 21.6, 20.1.
constexpr int kSelectThreads = 512, kListsApplyThreads = 1024;
constexpr int kOperatorQueries = 64, kOperatorTokens = 129;   // up to so many queries, from so many tokens on

template <typename T, typename P>
__global__ __launch_bounds__(kSelectThreads) void merge_select_kernel(const T* __restrict__ metric, int dm, const P plan, int B,
                                                                      int n_lead, float* __restrict__ best,
                                                                      int32_t* __restrict__ bcol, int na) {
  extern __shared__ float lds[];
  const int q = (int)blockIdx.x / na, a = (int)blockIdx.x - q * na;
  merge_plan_select<T, true, true, kSelectThreads>(metric, dm, 0, 1, dm, plan.query(q, B), n_lead, nullptr, lds, best, bcol,
                                                   (int)threadIdx.x, PlanPart{a, na, 0, 1, 0});
}

// LDS: what merge_plan_lists needs | src [n] | row [n].
template <typename T, typename P>
__global__ __launch_bounds__(kListsApplyThreads) void merge_lists_apply_kernel(
    const T* __restrict__ x, const int32_t* __restrict__ sizes, const float* __restrict__ best, const int32_t* __restrict__ bcol,
    const P plan, int B, int D, T* __restrict__ x_out, int32_t* __restrict__ sizes_out, int32_t* __restrict__ trace_src,
    int32_t* __restrict__ trace_dst, int parts, int lists_words) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr int V = Vec<T>::N, NT = kListsApplyThreads, TB = 4;
  const int q = (int)blockIdx.x / parts, part = (int)blockIdx.x - q * parts, tid = threadIdx.x;
  PlanQuery pq = plan.query(q, B);
  const int i0 = pq.i0, o0 = pq.o0, n = pq.n;
  if (n <= 0) return;
  const int n_out = n - pq.r_eff;
  int32_t* src = reinterpret_cast<int32_t*>(lds) + lists_words;   // the query's rows from 0, like the entries of `row`
  int32_t* row = src + n;
  pq.i0 = pq.o0 = 0;
  merge_plan_lists<NT, true>(lds, best + i0, bcol + i0, 1, 0, pq, src, row, part ? nullptr : trace_src, trace_dst, tid);
  __syncthreads();
  // A thread takes TB chunks at a time, a workgroup's threads neighbouring ones, and requests what most rows need, one source, for all
  // of them before it waits.
  const int share = (n_out + parts - 1) / parts, j0 = part * share, rows = min(share, n_out - j0);
  const int chunks = D / V, total = rows * chunks;
  const T* xq = x + (size_t)i0 * D;
  for (int t0 = tid; t0 < total; t0 += NT * TB) {
    int j[TB], c[TB], beg[TB], cnt[TB], sz[TB];
    Vec<T> v[TB];
#pragma unroll
    for (int u = 0; u < TB; ++u) {
      const int t = min(t0 + u * NT, total - 1);   // past the end: the last one again, not stored
      const int jj = t / chunks;
      j[u] = j0 + jj;
      c[u] = (t - jj * chunks) * V;
      beg[u] = row[j[u]];
      cnt[u] = (j[u] + 1 < n_out ? row[j[u] + 1] : n) - beg[u];
      const int first = src[beg[u]];
      v[u] = load_vec<T>(xq + (size_t)first * D + c[u]);
      sz[u] = sizes ? sizes[i0 + first] : 1;
    }
#pragma unroll
    for (int u = 0; u < TB; ++u) {
      if (t0 + u * NT >= total) break;
      T* po = x_out + (size_t)(o0 + j[u]) * D + c[u];
      if (cnt[u] > 1) {
        float acc[V];
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] = fmaf((float)sz[u], v[u].get(k), 0.f);
        for (int e = beg[u] + 1; e < beg[u] + cnt[u]; ++e) {
          const int srow = src[e], z = sizes ? sizes[i0 + srow] : 1;
          const Vec<T> w = load_vec<T>(xq + (size_t)srow * D + c[u]);
          sz[u] += z;
#pragma unroll
          for (int k = 0; k < V; ++k) acc[k] = fmaf((float)z, w.get(k), acc[k]);
        }
        const float denom = (float)sz[u];
#pragma unroll
        for (int k = 0; k < V; ++k) v[u].set(k, acc[k] / denom);
      }
      store_vec<T>(po, v[u]);
      if (c[u] == 0) sizes_out[o0 + j[u]] = sz[u];
    }
  }
}

// Workgroups per query of the two launches; na = 0: not run this way.  As many for the selection as there are blocks of A tokens
// while the launch has a CU for each, and enough to keep a workgroup's metric rows in 64 KB of LDS where they would not fit otherwise
// (160 KB at most).  For the rows one per CU, up to 16: all but their copying is the same work in each.
struct OperatorParts { int na, parts; };
static OperatorParts operator_parts(int B, int max_n, int dm) {
  const int bA = ((max_n + 1) / 2 + 31) / 32;
  int na = 1;
  while (na < bA && ((int64_t)2 * na * B <= 256 || plan_select_lds_bytes(max_n, dm, na, 1) > 64 * 1024)) na *= 2;
  if (na > bA) na = bA;
  if (B <= 0 || B > kOperatorQueries || max_n < kOperatorTokens || plan_select_lds_bytes(max_n, dm, na, 1) > 160 * 1024) return OperatorParts{0, 0};
  return OperatorParts{na, 256 / B > 16 ? 16 : 256 / B};
}

bool token_merge_in_two(int B, int max_n, int dm) {
  return B > 0 && max_n > 0 && max_n <= kPlanThreads && dm > 0 && dm % 4 == 0 && dm <= 128 && operator_parts(B, max_n, dm).na > 0;
}

hipError_t launch_merge_select_host(int dtype, const void* metric, int dm, const int32_t* plan, size_t count, const int32_t* d_plan,
                                    int B, int max_n, int n_lead, float* best, int32_t* bcol, hipStream_t s) {
  if (!token_merge_in_two(B, max_n, dm)) return hipErrorInvalidValue;
  const int na = operator_parts(B, max_n, dm).na;
  const size_t lds = plan_select_lds_bytes(max_n, dm, na, 1);
  return with_plan(plan, count, d_plan, [&](const auto& v) {
    typedef PlanInts<std::decay_t<decltype(v)>> P;
    const P p{v};
#define OTAS_SELECT(TYPE)                                                                                       \
  do {                                                                                                          \
    auto kern = merge_select_kernel<TYPE, P>;                                                                   \
    hipError_t e = set_max_dynamic_lds((const void*)kern, 160 * 1024);                                          \
    if (e != hipSuccess) return e;                                                                              \
    kern<<<dim3(B * na), dim3(kSelectThreads), lds, s>>>((const TYPE*)metric, dm, p, B, n_lead, best, bcol, na); \
  } while (0)
    if (dtype == 0) OTAS_SELECT(float); else OTAS_SELECT(bf16_t);
#undef OTAS_SELECT
    return hipGetLastError();
  });
}

hipError_t launch_merge_lists_apply_host(int dtype, const void* x, const int32_t* sizes, int dm, const float* best, const int32_t* bcol,
                                         const int32_t* plan, size_t count, const int32_t* d_plan, int B, int max_n, int D,
                                         void* x_out, int32_t* sizes_out, int32_t* trace_src, int32_t* trace_dst, hipStream_t s) {
  if (!token_merge_in_two(B, max_n, dm)) return hipErrorInvalidValue;
  const int parts = operator_parts(B, max_n, dm).parts;
  const size_t lists = (plan_lists_lds_bytes(max_n) + 15) & ~(size_t)15, lds = lists + 8 * (size_t)max_n;
  return with_plan(plan, count, d_plan, [&](const auto& v) {
    typedef PlanInts<std::decay_t<decltype(v)>> P;
    const P p{v};
#define OTAS_LISTS_APPLY(TYPE)                                                                                        \
  merge_lists_apply_kernel<TYPE, P><<<dim3(B * parts), dim3(kListsApplyThreads), lds, s>>>(                           \
      (const TYPE*)x, sizes, best, bcol, p, B, D, (TYPE*)x_out, sizes_out, trace_src, trace_dst, parts, (int)(lists / 4))
    if (dtype == 0) OTAS_LISTS_APPLY(float); else OTAS_LISTS_APPLY(bf16_t);
#undef OTAS_LISTS_APPLY
    return hipGetLastError();
  });
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
