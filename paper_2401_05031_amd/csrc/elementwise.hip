// HBM-bound row kernels: integer fill/copy, the prompting module's ragged concatenation
// (Sec. II-B / III-B), LayerNorm (Sec. II-A "normalization"), and the merging module's data
// movement fused with the LayerNorm behind it (Sec. II-C).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "plan_args.h"

namespace otas {

// ---------------------------------------------------------------------------------- fill / copy
__global__ void fill_i32_kernel(int32_t* p, int32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ void copy_i32_kernel(const int32_t* __restrict__ a, int32_t* __restrict__ b, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}
// One wave that stays busy for `ticks` periods of the constant-rate wall clock (a kernel of known
// duration, used to calibrate what an event pair adds to a launch).  The iteration cap makes the loop end
// whatever the clock does.
__global__ void spin_kernel(int64_t ticks, int32_t* sink) {
  const int64_t t0 = wall_clock64();
  int32_t it = 0;
  while (it < (1 << 22) && wall_clock64() - t0 < ticks) ++it;
  if (threadIdx.x == 0) sink[0] = it;
}
hipError_t launch_spin(int64_t ticks, int32_t* sink, hipStream_t s) {
  spin_kernel<<<dim3(1), dim3(64), 0, s>>>(ticks, sink);
  return hipGetLastError();
}
// One wave that `samples` times sleeps 4 x 8128 shader clocks (s_sleep 127 = 127 x 64 clocks; a sleeping wave
// needs no issue slots, so the waves it shares a SIMD with do not stretch it) and stores how many periods of the
// constant-rate wall clock that took: 4 * 8128 / ticks[s] = shader clocks per wall-clock period while whatever else
// is in flight on the chip runs.  Ends by itself after `samples` samples.
__global__ void clock_probe_kernel(uint32_t* ticks, int32_t samples) {
  for (int32_t s = 0; s < samples; ++s) {
    const uint64_t t0 = wall_clock64();
    asm volatile("s_sleep 127\n s_sleep 127\n s_sleep 127\n s_sleep 127");
    const uint64_t t1 = wall_clock64();
    if (threadIdx.x == 0) ticks[s] = (uint32_t)(t1 - t0);
  }
}
hipError_t launch_clock_probe(uint32_t* ticks, int32_t samples, hipStream_t s) {
  clock_probe_kernel<<<dim3(1), dim3(64), 0, s>>>(ticks, samples);
  return hipGetLastError();
}
hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  fill_i32_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(p, v, n);
  return hipGetLastError();
}
hipError_t launch_copy_i32(const int32_t* a, int32_t* b, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  copy_i32_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(a, b, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------- prepend
// One 16-byte chunk per thread.  blockIdx.y = query; blockIdx.x strides over the query's
// (row, chunk) pairs.  Output row i of a query comes from: i < n_lead -> token i;
// i < n_lead + P -> prompt i - n_lead; else token i - P.
// plan: tok_off [B+1] | prm_beg [B] | prm_cnt [B] | out_off [B+1].  gx = gridDim.x, 256 threads: asked for as gridDim and
// blockDim they would add 256 bytes of implicit arguments to the plan's.
template <typename T, typename P>
__global__ __launch_bounds__(256) void prepend_kernel(const T* __restrict__ tokens, const T* __restrict__ prompts, T* __restrict__ out,
                               const P plan, int B, int D, int n_lead, int gx) {
  constexpr int V = Vec<T>::N;
  const int q = blockIdx.y;
  const int o0 = plan[3 * B + 1 + q], n_out = plan[3 * B + 2 + q] - o0;
  const int t0 = plan[q], p0 = plan[B + 1 + q], Pq = plan[2 * B + 1 + q];   // the query's rows of the prompt tensor
  const int chunks = D / V;
  const int total = n_out * chunks;
  for (int t = blockIdx.x * 256 + threadIdx.x; t < total; t += gx * 256) {
    const int i = t / chunks, c = (t - i * chunks) * V;
    const T* src;
    if (i < n_lead) src = tokens + (size_t)(t0 + i) * D;
    else if (i < n_lead + Pq) src = prompts + (size_t)(p0 + i - n_lead) * D;
    else src = tokens + (size_t)(t0 + i - Pq) * D;
    store_vec<T>(out + (size_t)(o0 + i) * D + c, load_vec<T>(src + c));
  }
}

hipError_t launch_prepend(int dtype, const void* tokens, const void* prompts, void* out, const int32_t* plan,
                          size_t count, const int32_t* d_plan, int B, int max_n_out, int D, int n_lead, hipStream_t s) {
  if (B <= 0 || max_n_out <= 0) return hipSuccess;
  const int V = dtype == 0 ? 4 : 8;
  const int64_t tasks = (int64_t)max_n_out * (D / V);
  unsigned gx = (unsigned)((tasks + 255) / 256);
  if (gx > 64) gx = 64;
  dim3 grid(gx, B), block(256);
  return with_plan(plan, count, d_plan, [&](const auto& pl) {
    typedef std::decay_t<decltype(pl)> P;
    if (dtype == 0)
      prepend_kernel<float, P><<<grid, block, 0, s>>>((const float*)tokens, (const float*)prompts, (float*)out, pl, B, D,
                                                      n_lead, (int)gx);
    else
      prepend_kernel<bf16_t, P><<<grid, block, 0, s>>>((const bf16_t*)tokens, (const bf16_t*)prompts, (bf16_t*)out, pl, B,
                                                       D, n_lead, (int)gx);
    return hipGetLastError();
  });
}

// ---------------------------------------------------------------------------------- per-layer prompting
// The prompting module in front of a layer l >= 1 (Sec. III-B: it sits before the normalisation of
// every layer), on the float residual stream.  grow = false: rows n_lead .. n_lead + P - 1 of every
// query are overwritten with this layer's prompts (x_new == x_old, only those rows are touched).
// grow = true: the P prompts are inserted at row n_lead, the old rows are copied around them into
// x_new (a different buffer; old_off / new_off are the packed offsets before and after).
// 4 floats per thread; blockIdx.y = query.
template <typename T>
__global__ void deep_prompt_kernel(const float* __restrict__ x_old, float* __restrict__ x_new,
                                   const T* __restrict__ prompts, const int32_t* __restrict__ old_off,
                                   const int32_t* __restrict__ new_off, const int32_t* __restrict__ prm_off,
                                   int D, int n_lead, bool grow) {
  const int q = blockIdx.y;
  const int p0 = prm_off[q], P = prm_off[q + 1] - p0;
  const int o0 = new_off[q], n_new = new_off[q + 1] - o0, i0 = old_off[q];
  const int chunks = D / 4;
  const int first = grow ? 0 : n_lead, rows = grow ? n_new : P;   // rows this launch writes
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < rows * chunks; t += gridDim.x * blockDim.x) {
    const int i = first + t / chunks, c = (t % chunks) * 4;
    Vec<float> v;
    if (i >= n_lead && i < n_lead + P) {
      const T* src = prompts + (size_t)(p0 + i - n_lead) * D + c;
#pragma unroll
      for (int k = 0; k < 4; ++k) v.set(k, to_float(src[k]));
    } else {
      v = load_vec<float>(x_old + (size_t)(i0 + (i < n_lead ? i : i - P)) * D + c);
    }
    store_vec<float>(x_new + (size_t)(o0 + i) * D + c, v);
  }
}

hipError_t launch_deep_prompt(int dtype, const float* x_old, float* x_new, const void* prompts,
                              const int32_t* d_old_off, const int32_t* d_new_off, const int32_t* d_prm_off, int B,
                              int max_rows, int D, int n_lead, bool grow, hipStream_t s) {
  if (B <= 0 || max_rows <= 0) return hipSuccess;
  if (D % 4 != 0 || (grow && x_old == x_new)) return hipErrorInvalidValue;
  const int64_t tasks = (int64_t)max_rows * (D / 4);
  unsigned gx = (unsigned)((tasks + 255) / 256);
  if (gx > 64) gx = 64;
  dim3 grid(gx, B), block(256);
  if (dtype == 0)
    deep_prompt_kernel<float><<<grid, block, 0, s>>>(x_old, x_new, (const float*)prompts, d_old_off, d_new_off,
                                                     d_prm_off, D, n_lead, grow);
  else
    deep_prompt_kernel<bf16_t><<<grid, block, 0, s>>>(x_old, x_new, (const bf16_t*)prompts, d_old_off, d_new_off,
                                                      d_prm_off, D, n_lead, grow);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------- LayerNorm
// The row kernels below are chains of memory round trips and wave reductions, at small batches nothing else: each requests
// all it will need (the row's chunks, gamma, beta) before it waits for anything.  Loads are not masked: lanes past the
// end of the row repeat its last chunk, and what they hold is neither summed nor stored.
// Against masked loads, each chunk waited for before the next and gamma, beta after the reductions (MI355X, same bits): a
// ViT-B pass of one query 528 -> 522 us, of 64 without merging 3.00 -> 2.97 ms, with r = 16 1.956 -> 1.945.
__device__ inline int wave_index() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }   // row addresses stay scalar
template <typename T, int NCH> struct RowChunks {   // chunk lane + 64 i of 8 columns of a row
  Vec<T> v[NCH][8 / Vec<T>::N];
  __device__ inline void load(const T* __restrict__ p, int chunks, int lane) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = min(lane + 64 * i, chunks - 1);
#pragma unroll
      for (int u = 0; u < 8 / Vec<T>::N; ++u) v[i][u] = load_vec<T>(p + c * 8 + u * Vec<T>::N);
    }
  }
  __device__ inline float get(int i, int k) const { return v[i][k / Vec<T>::N].get(k % Vec<T>::N); }
};

// Row l of the plan (StartJob in kernels.h) by one workgroup of 256 threads, two queries a thread.
__device__ inline void start_plan_row(const StartJob& job, int l) {
  __shared__ int wave_tot[2][4];
  const int B = job.B, L = job.L, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool merge = job.kind == START_MERGE;
  int n[2], k[2], gone = 0;   // this row's length and removals of the thread's queries; tokens removed before layer l
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int q = 2 * tid + j;
    n[j] = k[j] = 0;
    if (q >= B) continue;
    const int n0 = job.v[q], r = job.v[B + q];
    if (merge) {
      n[j] = n0;
      for (int i = 0; i <= l; ++i) {
        k[j] = max(0, min(r, (n[j] - job.n_lead) / 2));
        if (i < l) n[j] -= k[j];
      }
      gone += n0 - n[j];
    } else {
      n[j] = l == L ? r : n0 + (job.grow ? l * r : 0);
    }
  }
  int sn = n[0] + n[1], sk = k[0] + k[1];
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int a = __shfl_up(sn, o, kWave), b = __shfl_up(sk, o, kWave);
    gone += __shfl_xor(gone, o, kWave);
    if (lane >= o) { sn += a; sk += b; }
  }
  __shared__ int gone_tot[4];
  if (lane == 63) { wave_tot[0][wave] = sn; wave_tot[1][wave] = sk; }
  if (lane == 0) gone_tot[wave] = gone;
  __syncthreads();
  int on = sn - n[0] - n[1], ok = sk - k[0] - k[1] + gone_tot[0] + gone_tot[1] + gone_tot[2] + gone_tot[3];
  for (int w = 0; w < wave; ++w) { on += wave_tot[0][w]; ok += wave_tot[1][w]; }
  int32_t* off = job.plan + (size_t)l * (B + 1);
  int32_t* reff = job.plan + (size_t)(L + 1) * (B + 1) + (size_t)l * B;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int q = 2 * tid + j;
    if (q >= B) break;
    off[q] = on;
    on += n[j];
    if (q == B - 1) off[B] = on;
    if (merge && l < L) {
      reff[q] = k[j];
      reff[(size_t)L * B + q] = ok;
      ok += k[j];
    }
  }
}
constexpr int kOnesPerBlock = 256 * 16;
__host__ __device__ static inline int64_t ones_blocks(int64_t n) { return (n + kOnesPerBlock - 1) / kOnesPerBlock; }
__device__ inline void start_job(const StartJob& job, int64_t blk) {
  if (blk <= job.L) { start_plan_row(job, (int)blk); return; }
  blk -= job.L + 1;
  const int which = blk < ones_blocks(job.n_ones[0]) ? 0 : 1;
  if (which) blk -= ones_blocks(job.n_ones[0]);
  int32_t* p = job.ones[which];
  for (int64_t i = blk * kOnesPerBlock + threadIdx.x; i < min((blk + 1) * kOnesPerBlock, job.n_ones[which]); i += 256) p[i] = 1;
}
struct NoJob {};

// One wave per row, the row held in registers (NCH chunks per lane), two-pass statistics
// in fp32 (mean, then the biased variance of the centred values).
// XT = type of the input row (the residual stream is float), T = type of gamma, beta and the output.
// Each lane owns chunks of 8 consecutive columns (two 16-byte loads of a float row).
// J: StartJob for a pass's first LayerNorm, whose leading job_blocks workgroups set the pass up, else NoJob.
// xw != nullptr: the row is also written out as floats (16-bit tokens entering the float residual
// stream: the widening copy rides on the first block's LayerNorm).
template <typename XT, typename T, int NCH, typename J>
__global__ __launch_bounds__(256) void layer_norm_kernel(const XT* __restrict__ x, const T* __restrict__ g,
                                                         const T* __restrict__ b, T* __restrict__ y,
                                                         int64_t Trows, int D, float eps, float* __restrict__ xw,
                                                         int job_blocks, const J job) {
  int64_t blk = blockIdx.x;
  if constexpr (std::is_same_v<J, StartJob>) {   // the pass's first LayerNorm: the leading workgroups set the pass up
    if (blk < job_blocks) { start_job(job, blk); return; }
    blk -= job_blocks;
  }
  constexpr int V = 8;
  const int lane = threadIdx.x & 63;
  const int64_t row = blk * 4 + wave_index();
  if (row >= Trows) return;
  const int chunks = D / V;
  const XT* xr = x + (size_t)row * D;
  RowChunks<XT, NCH> t;
  RowChunks<T, NCH> gg, bb;
  t.load(xr, chunks, lane);
  gg.load(g, chunks, lane);
  bb.load(b, chunks, lane);
  __builtin_amdgcn_sched_barrier(0);
  float v[NCH][V];
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
#pragma unroll
    for (int k = 0; k < V; ++k) v[i][k] = t.get(i, k);
    if (lane + 64 * i < chunks) {
#pragma unroll
      for (int k = 0; k < V; ++k) sum += v[i][k];
    }
  }
  if (xw) {
    float* wr = xw + (size_t)row * D;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = lane + 64 * i;
      if (c < chunks) {
        Vec<float> lo, hi;
#pragma unroll
        for (int k = 0; k < 4; ++k) { lo.set(k, v[i][k]); hi.set(k, v[i][4 + k]); }
        store_vec<float>(wr + c * V, lo);
        store_vec<float>(wr + c * V + 4, hi);
      }
    }
  }
  const float mean = wave_sum(sum) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
    if (c < chunks) {
#pragma unroll
      for (int k = 0; k < V; ++k) { const float d = v[i][k] - mean; sq += d * d; }
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + eps);
  T* yr = y + (size_t)row * D;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
    if (c < chunks) {
#pragma unroll
      for (int k0 = 0; k0 < V; k0 += Vec<T>::N) {
        Vec<T> o;
#pragma unroll
        for (int k = 0; k < Vec<T>::N; ++k) o.set(k, (v[i][k0 + k] - mean) * rstd * gg.get(i, k0 + k) + bb.get(i, k0 + k));
        store_vec<T>(yr + c * V + k0, o);
      }
    }
  }
}

template <typename XT, typename T>
static hipError_t layer_norm_dispatch(const void* x, const void* g, const void* b, void* y, int64_t Trows,
                                      int D, float eps, hipStream_t s, const StartJob* job, float* xw = nullptr) {
  const int chunks = D / 8;
  const int nch = (chunks + 63) / 64;
  const int64_t extra = job ? job->L + 1 + ones_blocks(job->n_ones[0]) + ones_blocks(job->n_ones[1]) : 0;
  dim3 grid((unsigned)((Trows + 3) / 4 + extra)), block(256);
#define OTAS_LN(N)                                                                                               \
  do {                                                                                                           \
    if (job)                                                                                                     \
      layer_norm_kernel<XT, T, N, StartJob><<<grid, block, 0, s>>>((const XT*)x, (const T*)g, (const T*)b, (T*)y,  \
                                                                   Trows, D, eps, xw, (int)extra, *job);         \
    else                                                                                                         \
      layer_norm_kernel<XT, T, N, NoJob><<<grid, block, 0, s>>>((const XT*)x, (const T*)g, (const T*)b, (T*)y,    \
                                                                Trows, D, eps, xw, 0, NoJob{});                  \
  } while (0)
  if (nch <= 1) OTAS_LN(1);
  else if (nch <= 2) OTAS_LN(2);
  else if (nch <= 3) OTAS_LN(3);
  else if (nch <= 4) OTAS_LN(4);
  else if (nch <= 8) OTAS_LN(8);
  else return hipErrorInvalidValue;
#undef OTAS_LN
  return hipGetLastError();
}

hipError_t launch_layer_norm(int dtype, bool x_is_float, const void* x, const void* g, const void* b, void* y,
                             int64_t T, int D, float eps, hipStream_t s, const StartJob* job) {
  if (T <= 0) return hipSuccess;
  if (dtype == 0) return layer_norm_dispatch<float, float>(x, g, b, y, T, D, eps, s, job);
  return x_is_float ? layer_norm_dispatch<float, bf16_t>(x, g, b, y, T, D, eps, s, job)
                    : layer_norm_dispatch<bf16_t, bf16_t>(x, g, b, y, T, D, eps, s, job);
}

hipError_t launch_layer_norm_widen(const void* x_bf16, const void* g, const void* b, void* y, float* x_float,
                                   int64_t T, int D, float eps, hipStream_t s, const StartJob* job) {
  if (T <= 0) return hipSuccess;
  return layer_norm_dispatch<bf16_t, bf16_t>(x_bf16, g, b, y, T, D, eps, s, job, x_float);
}

// Workgroups past the launch's rows read the weight of the next linear, one word of every cache line once.  What that gains is
// the way from HBM to the last-level cache under a kernel that leaves HBM idle: the lines end up in one XCD's L2, and
// which one matters little.  Each XCD the columns of its own tiles: 0 - 4 % slower from 800 rows on, as those overlap and the
// weight is read two to four times.  Each XCD an eighth, which are its tiles' columns up to 512 rows (us a pass, eighths /
// plain, MI355X): ViT-B, eight models in turn, one query 508 / 506, two 537 / 533; ViT-L one 1117 / 1108, two 1214 / 1208; ViT-H 50 rows
// 1454 / 1448, 200 2186 / 2177, 400 2389 / 2399, 430 1576 / 1576.
__device__ inline void warm_weight(const WarmWeight& w, int first) {
  const int64_t lines = w.bytes >> 7;
  for (int64_t l = (int64_t)((int)blockIdx.x - first) * 256 + threadIdx.x; l < lines; l += (int64_t)w.wgs * 256) {
    const uint32_t v = *reinterpret_cast<const uint32_t*>(static_cast<const char*>(w.w) + (l << 7));
    asm volatile("" ::"v"(v));
  }
}

// ---------------------------------------------------------------------------------- merge-apply + LayerNorm
// The merging module's data movement (Sec. II-C: size-weighted average of every surviving token
// with the tokens merged into it, survivors in their original order) fused with the LayerNorm that
// follows it in the block.  One wave per OUTPUT row: it gathers the rows listed for it
// (row_ptr / src_list, the surviving row first, then its sources in ascending position), forms
// sum(size * x) / sum(size) in fp32 in list order, writes the merged residual row and its size,
// and normalises the row it still holds in registers.  Same arithmetic, in the same order, as
// merge_apply_kernel followed by layer_norm_kernel.
template <typename T, int NCH>
__global__ __launch_bounds__(256) void merge_apply_ln_kernel(
    const float* __restrict__ x, const int32_t* __restrict__ sizes, const int32_t* __restrict__ src_list,
    const int32_t* __restrict__ row_ptr, int64_t T_in, int64_t T_out, int D, float* __restrict__ x_out,
    int32_t* __restrict__ sizes_out, const T* __restrict__ g, const T* __restrict__ b, T* __restrict__ y, float eps,
    WarmWeight warm) {
  constexpr int V = 8;
  if ((int)blockIdx.x >= (int)gridDim.x - warm.wgs) return warm_weight(warm, (int)gridDim.x - warm.wgs);
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave_index();
  if (row >= T_out) return;
  const int chunks = D / V;
  const int beg = row_ptr[row];
  const int end = (row + 1 < T_out) ? row_ptr[row + 1] : (int)T_in;
  RowChunks<T, NCH> gg, bb;
  gg.load(g, chunks, lane);
  bb.load(b, chunks, lane);
  float v[NCH][V];
#pragma unroll
  for (int i = 0; i < NCH; ++i)
#pragma unroll
    for (int k = 0; k < V; ++k) v[i][k] = 0.f;
  int tot = 0;
  if (end - beg == 1) {   // untouched token: the row itself
    const int srow = src_list[beg];
    tot = sizes ? sizes[srow] : 1;
    RowChunks<float, NCH> a;
    a.load(x + (size_t)srow * D, chunks, lane);
#pragma unroll
    for (int i = 0; i < NCH; ++i)
#pragma unroll
      for (int k = 0; k < V; ++k) v[i][k] = a.get(i, k);
  } else {
    // Every lane fetches one list entry and its size, so the rows' addresses are in registers before
    // the first row is requested; the rows are then loaded two at a time and accumulated in list order.
    for (int e0 = beg; e0 < end; e0 += 64) {
      const int cnt = min(64, end - e0);
      const int my_src = lane < cnt ? src_list[e0 + lane] : 0;
      const int my_sz = lane < cnt ? (sizes ? sizes[my_src] : 1) : 0;
      for (int e = 0; e < cnt; e += 2) {
        const bool two = e + 1 < cnt;   // the same for the whole wave
        const int e1 = two ? e + 1 : e;
        const int s0 = __builtin_amdgcn_readlane(my_src, e), s1 = __builtin_amdgcn_readlane(my_src, e1);
        const int z0 = __builtin_amdgcn_readlane(my_sz, e), z1 = __builtin_amdgcn_readlane(my_sz, e1);
        RowChunks<float, NCH> a0, a1;
        a0.load(x + (size_t)s0 * D, chunks, lane);
        a1.load(x + (size_t)s1 * D, chunks, lane);
        const float w0 = (float)z0, w1 = (float)z1;
        tot += z0;
#pragma unroll
        for (int i = 0; i < NCH; ++i)
#pragma unroll
          for (int k = 0; k < V; ++k) v[i][k] = fmaf(w0, a0.get(i, k), v[i][k]);
        if (two) {
          tot += z1;
#pragma unroll
          for (int i = 0; i < NCH; ++i)
#pragma unroll
            for (int k = 0; k < V; ++k) v[i][k] = fmaf(w1, a1.get(i, k), v[i][k]);
        }
      }
    }
    const float denom = (float)tot;
#pragma unroll
    for (int i = 0; i < NCH; ++i)
#pragma unroll
      for (int k = 0; k < V; ++k) v[i][k] = v[i][k] / denom;
  }
  if (lane == 0) sizes_out[row] = tot;
  float* xo = x_out + (size_t)row * D;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
    if (c < chunks) {
      Vec<float> lo, hi;
#pragma unroll
      for (int k = 0; k < 4; ++k) { lo.set(k, v[i][k]); hi.set(k, v[i][4 + k]); }
      store_vec<float>(xo + c * V, lo);
      store_vec<float>(xo + c * V + 4, hi);
#pragma unroll
      for (int k = 0; k < V; ++k) sum += v[i][k];
    }
  }
  const float mean = wave_sum(sum) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
    if (c < chunks) {
#pragma unroll
      for (int k = 0; k < V; ++k) { const float d = v[i][k] - mean; sq += d * d; }
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + eps);
  T* yr = y + (size_t)row * D;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
    if (c < chunks) {
#pragma unroll
      for (int k0 = 0; k0 < V; k0 += Vec<T>::N) {
        Vec<T> o;
#pragma unroll
        for (int k = 0; k < Vec<T>::N; ++k) o.set(k, (v[i][k0 + k] - mean) * rstd * gg.get(i, k0 + k) + bb.get(i, k0 + k));
        store_vec<T>(yr + c * V + k0, o);
      }
    }
  }
}

template <typename T>
static hipError_t merge_apply_ln_dispatch(const float* x, const int32_t* sizes, const int32_t* src_list,
                                          const int32_t* row_ptr, int64_t T_in, int64_t T_out, int D, float* x_out,
                                          int32_t* sizes_out, const void* g, const void* b, void* y, float eps,
                                          hipStream_t s, const WarmWeight& warm) {
  const int nch = (D / 8 + 63) / 64;
  dim3 grid((unsigned)((T_out + 3) / 4 + warm.wgs)), block(256);
#define OTAS_MLN(N)                                                                                               \
  merge_apply_ln_kernel<T, N><<<grid, block, 0, s>>>(x, sizes, src_list, row_ptr, T_in, T_out, D, x_out, sizes_out, \
                                                     (const T*)g, (const T*)b, (T*)y, eps, warm)
  if (nch <= 1) OTAS_MLN(1);
  else if (nch <= 2) OTAS_MLN(2);
  else if (nch <= 3) OTAS_MLN(3);
  else if (nch <= 4) OTAS_MLN(4);
  else if (nch <= 8) OTAS_MLN(8);
  else return hipErrorInvalidValue;
#undef OTAS_MLN
  return hipGetLastError();
}

hipError_t launch_merge_apply_ln(int dtype, const float* x, const int32_t* sizes, const int32_t* src_list,
                                 const int32_t* row_ptr, int64_t T_in, int64_t T_out, int D, float* x_out,
                                 int32_t* sizes_out, const void* g, const void* b, void* y, float eps, hipStream_t s,
                                 const WarmWeight& warm) {
  if (T_out <= 0) return hipSuccess;
  return dtype == 0 ? merge_apply_ln_dispatch<float>(x, sizes, src_list, row_ptr, T_in, T_out, D, x_out, sizes_out, g,
                                                     b, y, eps, s, warm)
                    : merge_apply_ln_dispatch<bf16_t>(x, sizes, src_list, row_ptr, T_in, T_out, D, x_out, sizes_out,
                                                      g, b, y, eps, s, warm);
}

// ---------------------------------------------------------------------------------- split-K reduce + LayerNorm
// Second half of a split-K residual linear: one wave per row adds the S float partial products in
// split order, then the bias and the residual row, writes the new residual row, and (LN) normalises
// the row it still holds in registers with the next block's first LayerNorm.  x_out may be res.
template <int NCH, bool LN>
__global__ __launch_bounds__(256) void splitk_reduce_ln_kernel(const float* __restrict__ part, int S,
                                                               const bf16_t* __restrict__ bias, const float* res,
                                                               float* x_out, int64_t M, int D,
                                                               const bf16_t* __restrict__ g,
                                                               const bf16_t* __restrict__ b, bf16_t* __restrict__ y,
                                                               float eps, WarmWeight warm) {
  constexpr int V = 8;
  if ((int)blockIdx.x >= (int)gridDim.x - warm.wgs) return warm_weight(warm, (int)gridDim.x - warm.wgs);
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave_index();
  if (row >= M) return;
  const int chunks = D / V;
  const size_t split_stride = (size_t)M * D;
  const float* pr = part + (size_t)row * D;
  float* xo = x_out + (size_t)row * D;
  // requested with the first partial results and used after all of them
  RowChunks<bf16_t, NCH> bv, gg, bb;
  RowChunks<float, NCH> p0, rv;
  p0.load(pr, chunks, lane);
  bv.load(bias, chunks, lane);
  rv.load(res + (size_t)row * D, chunks, lane);
  if (LN) {
    gg.load(g, chunks, lane);
    bb.load(b, chunks, lane);
  }
  float v[NCH][V];
#pragma unroll
  for (int i = 0; i < NCH; ++i)
#pragma unroll
    for (int k = 0; k < V; ++k) v[i][k] = p0.get(i, k);
  // the other partial results, as many as fit in flight together (all of them for S <= 8 and D <= 1024): the additions
  // keep the order sp = 1, 2, ... (S is the same for the whole launch: the tests on it are scalar branches)
  constexpr int UB = NCH <= 2 ? 7 : NCH <= 4 ? 3 : 1;
  for (int sp = 1; sp < S; sp += UB) {
    RowChunks<float, NCH> ps[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u)
      if (sp + u < S) ps[u].load(pr + (size_t)(sp + u) * split_stride, chunks, lane);
#pragma unroll
    for (int u = 0; u < UB; ++u)
      if (sp + u < S) {
#pragma unroll
        for (int i = 0; i < NCH; ++i)
#pragma unroll
          for (int k = 0; k < V; ++k) v[i][k] += ps[u].get(i, k);
      }
  }
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
#pragma unroll
    for (int k = 0; k < V; ++k) v[i][k] = (v[i][k] + bv.get(i, k)) + rv.get(i, k);
    if (c < chunks) {
      Vec<float> olo, ohi;
#pragma unroll
      for (int k = 0; k < 4; ++k) { olo.set(k, v[i][k]); ohi.set(k, v[i][4 + k]); }
      store_vec<float>(xo + c * V, olo);
      store_vec<float>(xo + c * V + 4, ohi);
#pragma unroll
      for (int k = 0; k < V; ++k) sum += v[i][k];
    }
  }
  if (!LN) return;
  const float mean = wave_sum(sum) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
    if (c < chunks) {
#pragma unroll
      for (int k = 0; k < V; ++k) { const float d = v[i][k] - mean; sq += d * d; }
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + eps);
  bf16_t* yr = y + (size_t)row * D;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + 64 * i;
    if (c < chunks) {
      Vec<bf16_t> o;
#pragma unroll
      for (int k = 0; k < V; ++k) o.set(k, (v[i][k] - mean) * rstd * gg.get(i, k) + bb.get(i, k));
      store_vec<bf16_t>(yr + c * V, o);
    }
  }
}

hipError_t launch_splitk_reduce_ln(const float* part, int S, const void* bias, const float* res, float* x_out,
                                   int64_t M, int D, const void* g, const void* b, void* y, float eps,
                                   hipStream_t s, const WarmWeight& warm) {
  if (M <= 0) return hipSuccess;
  if (S < 1 || D % 8 != 0) return hipErrorInvalidValue;
  const int nch = (D / 8 + 63) / 64;
  dim3 grid((unsigned)((M + 3) / 4 + warm.wgs)), block(256);
#define OTAS_RED(N)                                                                                              \
  do {                                                                                                           \
    if (y)                                                                                                       \
      splitk_reduce_ln_kernel<N, true><<<grid, block, 0, s>>>(part, S, (const bf16_t*)bias, res, x_out, M, D,    \
                                                              (const bf16_t*)g, (const bf16_t*)b, (bf16_t*)y, eps, warm); \
    else                                                                                                         \
      splitk_reduce_ln_kernel<N, false><<<grid, block, 0, s>>>(part, S, (const bf16_t*)bias, res, x_out, M, D,   \
                                                               nullptr, nullptr, nullptr, eps, warm);            \
  } while (0)
  if (nch <= 1) OTAS_RED(1);
  else if (nch <= 2) OTAS_RED(2);
  else if (nch <= 3) OTAS_RED(3);
  else if (nch <= 4) OTAS_RED(4);
  else if (nch <= 8) OTAS_RED(8);
  else return hipErrorInvalidValue;
#undef OTAS_RED
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------- model ends
// Front end of the vision transformer (Sec. II-A): the image [C, Hi, Wi] is cut into p x p patches
// (row by row), every patch flattened channel-major into one row of the patch matrix [N, C p p]
// (the layout of a [D, C, p, p] projection weight); the linear projection is the GEMM kernel;
// embed_finish then builds [class token | projected patches] + position embedding.
// Both are passes over memory whose time went into the index arithmetic of a thread per element, most of it divisions of 64
// bits.  Now a thread moves V elements, 16 bytes, where rows and pointers allow it (V = 1 otherwise), and what does not
// differ inside a workgroup or wave is worked out once for it.  Patchify: `blocks` workgroups for the p rows of one channel that
// make up a row of patches, threads patch by patch, so that they write runs of p p elements and find the other 2 p bytes
// of an image row's cache line in their own L1.  Embed_finish: a wave per row.
// Measured on MI355X (us, an element per thread / 16 bytes): 24 images of 224 x 224 in bf16, patches of 16, D = 768: 17.4 / 6.4 and 10.2 / 5.6; 6 in float 6.1 / 5.1 and 5.1 / 5.2.
template <typename T, int V>
__global__ __launch_bounds__(256) void patchify_kernel(const T* __restrict__ img, T* __restrict__ out, int C, int Hi, int Wi, int p,
                                                       int blocks) {
  const int pv = p / V;                                   // threads per row of a patch
  const int band = (int)blockIdx.x / blocks;              // (image, row of patches, channel)
  const int k = ((int)blockIdx.x - band * blocks) * 256 + (int)threadIdx.x;
  if (k >= Wi / V * p) return;
  const int nw = Wi / p, nh = Hi / p;
  const int px = k / (p * pv), in = k - px * p * pv, i = in / pv, j = (in - i * pv) * V;
  const int bh = band / C, c = band - bh * C, b = bh / nh, py = bh - b * nh;
  const T* src = img + (((size_t)b * C + c) * Hi + (size_t)py * p + i) * Wi + (size_t)px * p + j;
  T* dst = out + (((size_t)bh * nw + px) * C + c) * p * p + (size_t)i * p + j;
  if constexpr (V == 1) *dst = *src;
  else store_vec<T>(dst, load_vec<T>(src));
}

template <typename T, int V>
__global__ __launch_bounds__(256) void embed_finish_kernel(const T* __restrict__ proj, const T* __restrict__ cls,
                                                           const T* __restrict__ pos, T* __restrict__ tokens, int N, int D, int n_lead,
                                                           int rows) {
  const int row = (int)blockIdx.x * 4 + wave_index(), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int n = n_lead + N, b = row / n, i = row - b * n;
  const T* src = i < n_lead ? cls : proj + ((size_t)b * N + (i - n_lead)) * D;
  const T* at = pos + (size_t)i * D;
  T* dst = tokens + (size_t)row * D;
  for (int d = lane * V; d < D; d += 64 * V) {
    if constexpr (V == 1) dst[d] = from_float<T>(to_float(src[d]) + to_float(at[d]));
    else {
      const Vec<T> x = load_vec<T>(src + d), y = load_vec<T>(at + d);
      Vec<T> o;
#pragma unroll
      for (int e = 0; e < V; ++e) o.set(e, x.get(e) + y.get(e));
      store_vec<T>(dst + d, o);
    }
  }
}

// Launches work on B images in as many pieces as it takes to keep a grid of 256 threads a workgroup below the 2^32 threads it can
// have: short rows (4 x 4 pixels in one patch: 16 threads of 256 have an element) reach that before the elements do.
template <typename F>
static hipError_t launch_images(int64_t B, int64_t workgroups_per_image, F&& launch) {
  int64_t most = ((1 << 24) - 1) / workgroups_per_image;
  if (most < 1) most = 1;
  for (int64_t b = 0; b < B; b += most) launch(b, (int)(B - b < most ? B - b : most));
  return hipGetLastError();
}

static bool on_16_bytes(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <typename T>
static hipError_t patchify(const T* img, T* out, int B, int C, int Hi, int Wi, int p, hipStream_t s) {
  constexpr int V = Vec<T>::N;   // p % V == 0: every row of the image and of the patch matrix begins on 16 bytes
  const bool wide = p % V == 0 && on_16_bytes(img) && on_16_bytes(out);
  if (B <= 0 || C <= 0 || Hi / p <= 0 || Wi / p <= 0) return hipSuccess;
  const int64_t per_band = ((int64_t)Wi * p / (wide ? V : 1) + 255) / 256, per_image = per_band * (Hi / p) * C;
  const int64_t pixels = (int64_t)C * Hi * Wi;
  return launch_images(B, per_image, [&](int64_t b, int images) {
    const dim3 grid((unsigned)(per_image * images)), block(256);
    if (wide) patchify_kernel<T, V><<<grid, block, 0, s>>>(img + b * pixels, out + b * pixels, C, Hi, Wi, p, (int)per_band);
    else patchify_kernel<T, 1><<<grid, block, 0, s>>>(img + b * pixels, out + b * pixels, C, Hi, Wi, p, (int)per_band);
  });
}

hipError_t launch_patchify(int dtype, const void* img, void* out, int B, int C, int Hi, int Wi, int p, hipStream_t s) {
  return dtype == 0 ? patchify((const float*)img, (float*)out, B, C, Hi, Wi, p, s)
                    : patchify((const bf16_t*)img, (bf16_t*)out, B, C, Hi, Wi, p, s);
}

template <typename T>
static hipError_t embed_finish(const T* proj, const T* cls, const T* pos, T* tokens, int B, int N, int D, int n_lead,
                               hipStream_t s) {
  constexpr int V = Vec<T>::N;
  const bool wide = D % V == 0 && on_16_bytes(proj) && on_16_bytes(cls) && on_16_bytes(pos) && on_16_bytes(tokens);
  const int n = n_lead + N;
  if (B <= 0 || n <= 0 || D <= 0) return hipSuccess;
  return launch_images(B, (n + 3) / 4, [&](int64_t b, int images) {
    const int rows = images * n;
    const T* from = proj + b * N * D;
    T* to = tokens + b * n * D;
    const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
    if (wide) embed_finish_kernel<T, V><<<grid, block, 0, s>>>(from, cls, pos, to, N, D, n_lead, rows);
    else embed_finish_kernel<T, 1><<<grid, block, 0, s>>>(from, cls, pos, to, N, D, n_lead, rows);
  });
}

hipError_t launch_embed_finish(int dtype, const void* proj, const void* cls, const void* pos, void* tokens, int B,
                               int N, int D, int n_lead, hipStream_t s) {
  return dtype == 0 ? embed_finish((const float*)proj, (const float*)cls, (const float*)pos, (float*)tokens, B, N, D, n_lead, s)
                    : embed_finish((const bf16_t*)proj, (const bf16_t*)cls, (const bf16_t*)pos, (bf16_t*)tokens, B, N, D, n_lead, s);
}

// Back end (Sec. III-B: every task has its own head): the first row of a query's output is normalised (final LayerNorm,
// two-pass fp32 statistics, stored in the model's dtype like every GEMM operand) and multiplied with its task's head
// [K, D].  grid (B, ceil((k_max - c0) / 32)): queries in the first dimension, whose limit no batch reaches (the second one
// ends at 65535).  Eight classes per wave: every wave holds the whole row in registers and normalises it for itself, its
// lanes share a class's row in the same pieces of 8 columns, fp32 accumulate, one butterfly per class.
// Bound by latency: the row, gamma, beta and the first pieces of the weights are requested together and no wave waits
// for another.  Measured on MI355X against one workgroup per query with one class per thread, each walking its row
// alone (us): one query with 10 classes 15.7 -> 5.7, seven queries with up to 100 19.6 -> 6.8.
constexpr int kHeadClasses = 32;
template <typename T, int NCH, typename P>
__global__ __launch_bounds__(256) void task_head_kernel(const float* __restrict__ x, const P plan, int B,
                                                        const T* __restrict__ g, const T* __restrict__ bta, int D,
                                                        float eps, float* __restrict__ logits, int k_max, int c0) {
  constexpr int V = 8, NC = kHeadClasses / 4;
  const int q = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* xr = x + (size_t)plan[q] * D;
  // plan: first rows [B] | task [B] | pad to an even count | per task {w, b, K, pad} (6 ints)
  const int rec = ((2 * B + 1) & ~1) + 6 * plan[B + q];
  const T* w = reinterpret_cast<const T*>((uint64_t)(uint32_t)plan[rec] | (uint64_t)(uint32_t)plan[rec + 1] << 32);
  const T* b = reinterpret_cast<const T*>((uint64_t)(uint32_t)plan[rec + 2] | (uint64_t)(uint32_t)plan[rec + 3] << 32);
  const int K = plan[rec + 4];
  const int k0 = c0 + blockIdx.y * kHeadClasses + wave * NC;
  if (k0 >= K) {   // classes beyond the task's count read 0
    if (lane < NC && k0 + lane < k_max) logits[(size_t)q * k_max + k0 + lane] = 0.f;
    return;
  }
  auto load8 = [](const T* p, float (&o)[V]) {
#pragma unroll
    for (int k = 0; k < V; k += Vec<T>::N) {
      const Vec<T> t = load_vec<T>(p + k);
#pragma unroll
      for (int e = 0; e < Vec<T>::N; ++e) o[k + e] = t.get(e);
    }
  };
  const int chunks = D / V;
  float v[NCH][V], gg[NCH][V], bb[NCH][V];
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = min(lane + 64 * i, chunks - 1);   // lanes past the end repeat the last chunk and are left out of the sums
    const Vec<float> lo = load_vec<float>(xr + c * V), hi = load_vec<float>(xr + c * V + 4);
    load8(g + c * V, gg[i]);
    load8(bta + c * V, bb[i]);
#pragma unroll
    for (int k = 0; k < 4; ++k) { v[i][k] = lo.get(k); v[i][4 + k] = hi.get(k); }
  }
  auto weights = [&](int i, Vec<T> (&wv)[NC][V / Vec<T>::N]) {
    const int c = min(lane + 64 * i, chunks - 1);
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int k = 0; k < V / Vec<T>::N; ++k)
        wv[j][k] = load_vec<T>(w + (size_t)min(k0 + j, K - 1) * D + c * V + k * Vec<T>::N);
  };
  Vec<T> wv[NC][V / Vec<T>::N];
  weights(0, wv);
#pragma unroll
  for (int i = 0; i < NCH; ++i)
    if (lane + 64 * i < chunks) {
#pragma unroll
      for (int k = 0; k < V; ++k) sum += v[i][k];
    }
  const float mean = wave_sum(sum) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
    if (lane + 64 * i < chunks) {
#pragma unroll
      for (int k = 0; k < V; ++k) { const float d = v[i][k] - mean; sq += d * d; }
    }
  const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + eps);
  float acc[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) acc[j] = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    if (i > 0) weights(i, wv);
    if (lane + 64 * i < chunks) {
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const float h = to_float(from_float<T>((v[i][k] - mean) * rstd * gg[i][k] + bb[i][k]));
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[j] = fmaf(h, wv[j][k / Vec<T>::N].get(k % Vec<T>::N), acc[j]);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NC; ++j) acc[j] = wave_sum(acc[j]);
#pragma unroll
  for (int j = 0; j < NC; ++j)
    if (lane == j && k0 + j < k_max) logits[(size_t)q * k_max + k0 + j] = k0 + j < K ? acc[j] + to_float(b[k0 + j]) : 0.f;
}

hipError_t launch_task_heads(int dtype, const float* x, const int32_t* plan, size_t count, const int32_t* d_plan,
                             const void* g, const void* b, int B, int D, float eps, float* logits, int k_max,
                             hipStream_t s) {
  if (B <= 0 || k_max <= 0) return hipSuccess;
  const int nch = (D / 8 + 63) / 64;
  const int blocks = (k_max - 1) / kHeadClasses + 1;
  return with_plan(plan, count, d_plan, [&](const auto& pl) {
    typedef std::decay_t<decltype(pl)> P;
    for (int done = 0; done < blocks; done += 65535) {
      const dim3 grid((unsigned)B, (unsigned)std::min(blocks - done, 65535)), block(256);
#define OTAS_HEAD(TYPE, N)                                                                                              \
  task_head_kernel<TYPE, N, P><<<grid, block, 0, s>>>(x, pl, B, (const TYPE*)g, (const TYPE*)b, D, eps, logits, k_max, \
                                                      done * kHeadClasses)
#define OTAS_HEADS(N) do { if (dtype == 0) OTAS_HEAD(float, N); else OTAS_HEAD(bf16_t, N); } while (0)
      if (nch <= 1) OTAS_HEADS(1);
      else if (nch <= 2) OTAS_HEADS(2);
      else if (nch <= 4) OTAS_HEADS(4);
      else if (nch <= 8) OTAS_HEADS(8);
      else return hipErrorInvalidValue;
#undef OTAS_HEADS
#undef OTAS_HEAD
    }
    return hipGetLastError();
  });
}

}  // namespace otas
