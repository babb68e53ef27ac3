// Multi-head attention of Sec. II-A over a ragged batch: per query q and head h,
//   O_h = softmax(Q_h K_h^T / sqrt(d_h) [+ ln size_j]) V_h,   heads concatenated into [T, D].
// qkv is the packed [T, 3D] output of the QKV projection (columns Q | K | V, heads contiguous).
//
//   * attention_f32_kernel  -- fp32 MFMA, fp32 arithmetic throughout (f32 models, and the fallback for head widths
//                              the bf16 kernel does not take).
//   * attention_mfma_kernel -- bf16 MFMA with one head's K and V staged in LDS (bf16 models).
#include <algorithm>
#include <cstdlib>

#include "common.h"
#include "kernels.h"
#include "merge_plan_body.h"

namespace otas {

// ------------------------------------------------------------------------------ true fp32 on the matrix cores
// f32 models, and bf16 models of head widths the bf16 kernel is not built for: fp32 products, sums and exponentials
// (v_mfma_f32_32x32x2_f32, expf).  grid (ceil(max_n / 32), H, B), four waves: a workgroup owns 32 query rows of one
// head, wave w the key blocks w, w + 4, ... of 32 keys with an online softmax of its own; the four partial results
// (row maximum, row sum, O) are combined through LDS in wave order, so a row's result depends on its own query alone.
// Both products are computed transposed, as in the bf16 kernel below: a lane owns one query row, and the
// accumulator element e of lane half h of the first product is key 8 (e / 4) + 4 h + (e & 3), which the second
// product takes as k-slot h of its MFMA e straight from registers.  K, V and Q go from global memory to registers
// (no wave shares a key block with another): per key block 2 x 32 MFMAs of 64 clocks at head width 64;
// what bounds it, at few waves per SIMD, is the chain load -> logits -> softmax -> product (the matrix pipe is busy 19 %
// of the time at 6 x 201 tokens, 12 heads).
// Measured on MI355X against one wave per query row on the vector ALU (us): 6 x 201 tokens, 12 heads of 64
// 119 -> 21.6; 2 x 201 tokens, 3 heads 31 -> 12.
template <typename T, int DT>
__device__ __forceinline__ void attention_f32_body(const T* __restrict__ qkv, const int32_t* __restrict__ sizes,
                                                   const int32_t* __restrict__ off, int D, int H, float scale,
                                                   T* __restrict__ o, const int q, const int h, const int xblk, float* lds) {
  constexpr int NG = 4 * DT;             // groups of 8 columns of a head, zero-filled past its width
  constexpr int LDO = 32 * DT + 4;
  float* ml = lds;                       // [4][2][32] row maximum and sum of every wave
  float* osh = lds + 256;                // [4][32][LDO]
  const int dh = D / H;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, fr = lane & 31, fk = lane >> 5;
  const int base = off[q], n = off[q + 1] - base;
  const int row0 = xblk * 32;
  if (row0 >= n) return;                 // the whole workgroup
  const size_t ld = (size_t)3 * D;
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  floatx4 qf[NG];
  {
    const T* p = qkv + (size_t)(base + min(row0 + fr, n - 1)) * ld + h * dh + 4 * fk;
#pragma unroll
    for (int g = 0; g < NG; ++g) qf[g] = 8 * g + 4 * fk < dh ? load4<T>(p + 8 * g) : zero;   // dh % 4 == 0
  }
  floatx16 oacc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[t][e] = 0.f;
  float m_run = -INFINITY, l_part = 0.f;
  const int nblk = (n + 31) >> 5;
  for (int b = wave; b < nblk; b += 4) {
    const int kb = b * 32;
    // keys past the end repeat the last one: their logits become -inf
    const T* pk = qkv + (size_t)(base + min(kb + fr, n - 1)) * ld + D + h * dh + 4 * fk;
    floatx4 kf[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) kf[g] = 8 * g + 4 * fk < dh ? load4<T>(pk + 8 * g) : zero;
    float vf[DT][16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int key = min(kb + 8 * (e >> 2) + 4 * fk + (e & 3), n - 1);
      const T* pv = qkv + (size_t)(base + key) * ld + 2 * D + h * dh;
#pragma unroll
      for (int t = 0; t < DT; ++t) vf[t][e] = to_float(pv[min(32 * t + fr, dh - 1)]);   // rows past dh are not stored
    }
    floatx16 s;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g)
      if (8 * g < dh) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[g][u], qf[g][u], s, 0, 0, 0);
      }
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int key = kb + 8 * (e >> 2) + 4 * fk + (e & 3);
      float v = s[e] * scale;
      if (sizes) v += logf((float)sizes[base + min(key, n - 1)]);
      s[e] = key < n ? v : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    mx = xor32_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;   // no key of weight so far (sizes 0, logits below the range): all 0
    const float alpha = expf(m_run - m_ref);                // 0 on the first block
    m_run = m_new;
    l_part *= alpha;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[t][e] *= alpha;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = expf(s[e] - m_ref);
      l_part += s[e];
    }
    if (kb + 32 > n) {   // values past the end: zero, or an infinite last one would turn the row to NaN (0 x inf)
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int t = 0; t < DT; ++t) vf[t][e] = kb + 8 * (e >> 2) + 4 * fk + (e & 3) < n ? vf[t][e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e)
#pragma unroll
      for (int t = 0; t < DT; ++t) oacc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[t][e], s[e], oacc[t], 0, 0, 0);
  }
  const float l_run = xor32_sum(l_part);
  if (fk == 0) {
    ml[wave * 64 + fr] = m_run;
    ml[wave * 64 + 32 + fr] = l_run;
  }
  __syncthreads();
  float m_all = -INFINITY;
#pragma unroll
  for (int w = 0; w < 4; ++w) m_all = fmaxf(m_all, ml[w * 64 + fr]);   // wave 0 always has a key block
  const float f = expf(m_run - m_all);                                 // 0 for a wave without one
  float* mine = osh + (wave * 32 + fr) * LDO;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<floatx4*>(mine + 32 * t + 8 * g + 4 * fk) =
          floatx4{oacc[t][4 * g] * f, oacc[t][4 * g + 1] * f, oacc[t][4 * g + 2] * f, oacc[t][4 * g + 3] * f};
  __syncthreads();
  const int r = tid >> 3;                // 8 threads per row
  if (row0 + r >= n) return;
  float mr = -INFINITY, l = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) mr = fmaxf(mr, ml[w * 64 + r]);
#pragma unroll
  for (int w = 0; w < 4; ++w) l += ml[w * 64 + 32 + r] * expf(ml[w * 64 + r] - mr);
  const float inv = 1.0f / l;
  for (int d = (tid & 7) * 4; d < dh; d += 32) {
    floatx4 v = zero;
#pragma unroll
    for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const floatx4*>(osh + (w * 32 + r) * LDO + d);
    Quad<T> out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out.x[e] = from_float<T>(v[e] * inv);
    *reinterpret_cast<Quad<T>*>(o + (size_t)(base + row0 + r) * D + h * dh + d) = out;
  }
}

template <typename T, int DT>
__global__ __launch_bounds__(256) void attention_f32_kernel(const T* __restrict__ qkv, const int32_t* __restrict__ sizes,
                                                               const int32_t* __restrict__ off, int D, int H, float scale,
                                                               T* __restrict__ o) {
  extern __shared__ __attribute__((aligned(16))) float f32_smem[];
  attention_f32_body<T, DT>(qkv, sizes, off, D, H, scale, o, (int)blockIdx.z, (int)blockIdx.y, (int)blockIdx.x, f32_smem);
}

// Together with the selection of the layer's merge plan, as attention_plan_kernel below does for bf16 models: the first
// B na nb workgroups select, the others are attention's, H heads and xblks row blocks a query.  The lists are written by
// the projection's launch.  Two queries of 201 tokens, 3 heads of 64 (MI355X): plan 17.1 and attention 11.9 us one after
// the other, 13.5 in one launch and 2 us more for the projection; the two-layer pass 126 -> 100 us.
template <int DT>
__global__ __launch_bounds__(256) void attention_select_f32_kernel(
    const float* __restrict__ qkv, const int32_t* __restrict__ sizes, const int32_t* __restrict__ off, int D, int H,
    float scale, float* __restrict__ o, int B, int xblks, const int32_t* __restrict__ out_off,
    const int32_t* __restrict__ reff_arr, const int32_t* __restrict__ troff, int n_lead, float* __restrict__ sel_best,
    int32_t* __restrict__ sel_bcol, int64_t sel_stride, int na, int nb) {
  extern __shared__ __attribute__((aligned(16))) float f32_smem[];
  int id = (int)blockIdx.x;
  if (id < B * na * nb) {   // workgroup-uniform
    const int q = id / (na * nb), pp = id % (na * nb);
    merge_plan_select<float, true, true, 256>(qkv, 3 * (int64_t)D, D, H, D / H, plan_query(off, out_off, reff_arr, troff, q),
                                              n_lead, nullptr, f32_smem, sel_best, sel_bcol, (int)threadIdx.x,
                                              PlanPart{pp % na, na, pp / na, nb, sel_stride});
    return;
  }
  id -= B * na * nb;
  const int xblk = id % xblks;
  id /= xblks;
  attention_f32_body<float, DT>(qkv, sizes, off, D, H, scale, o, id / H, id % H, xblk, f32_smem);
}
static size_t attention_f32_lds(int dh) { return sizeof(float) * (256 + 4 * 32 * (32 * (size_t)((dh + 31) / 32) + 4)); }

template <typename T>
static hipError_t attention_f32(const void* qkv, const int32_t* sz, const int32_t* d_off, int B, int max_n, int D,
                                int H, float scale, void* o, hipStream_t s) {
  const int dt = (D / H + 31) / 32;
  dim3 grid((max_n + 31) / 32, H, B), block(256);
  const size_t lds = attention_f32_lds(D / H);
#define OTAS_ATTN(N)                                                                                              \
  do {                                                                                                            \
    auto kern = attention_f32_kernel<T, N>;                                                                       \
    hipError_t e = set_max_dynamic_lds((const void*)kern, (int)lds);                                              \
    if (e != hipSuccess) return e;                                                                                \
    kern<<<grid, block, lds, s>>>((const T*)qkv, sz, d_off, D, H, scale, (T*)o);                                  \
  } while (0)
  if (dt <= 1) OTAS_ATTN(1);
  else if (dt == 2) OTAS_ATTN(2);
  else if (dt == 3) OTAS_ATTN(3);
  else if (dt == 4) OTAS_ATTN(4);
  else return hipErrorInvalidValue;
#undef OTAS_ATTN
  return hipGetLastError();
}

// ------------------------------------------------------------------------------ bf16 MFMA
// grid (ceil(max_n / (32 NW / KG)), H, B), NW waves (4 or 8): each wave owns 32 query rows of one (query, head), or, where KG > 1, KG
// waves share 32 rows (attention_shared_body).
// The keys and values of the head are staged in LDS in chunks of up to KC rows (rows padded
// by 16 bytes so that the 16 lanes served per clock fall on distinct banks); every wave then walks
// the chunk in blocks of 32 keys with an online softmax (running row maximum and sum, fp32).
//
// Both products are computed transposed, so that a lane always owns ONE query row:
//   S^T[key, row] = K[key, :] . Q[row, :]     A operand = K rows (LDS), B operand = Q rows (registers)
//   O^T[d, row]  += V^T[d, key] P^T[key, row] A operand = V^T (LDS, transposing read), B = P^T
// With the 32x32 accumulator layout a lane (row = lane & 31, half = lane >> 5) holds, of a 32-key
// block, the keys 8 (e / 4) + 4 half + (e & 3), e = 0..15: row maxima and sums are reductions over a
// lane's own registers plus one exchange with lane ^ 32, and the probabilities feed the second MFMA
// straight from registers: its k-slot i of half h is defined to be key 16 kk + 8 (i / 4) + 4 h +
// (i & 3), which is exactly what accumulator registers 8 kk .. 8 kk + 7 hold.  V^T is read with the
// same key order by ds_read_b64_tr_b16 (gfx950): in every group of 16 lanes, lane s supplies the
// address of V[k0 + s / 4][d0 + 4 (s & 3) ..+3] and lane i receives V[k0 + 0..3][d0 + i].
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef short short8_t __attribute__((ext_vector_type(8)));

// The steps of a chunk, which the two bodies below share: they are the same arithmetic in the same order in both.
// Stages K and V rows c0 .. c0 + nc_pad - 1 of a head (zero beyond nc) with NT threads.
template <int DH, bool BIAS, int NT>
__device__ __forceinline__ void attention_stage(const bf16_t* __restrict__ qkv, const int32_t* __restrict__ sizes, size_t ld, int D, int h,
                                                int first, int nc, int nc_pad, bf16_t* Ks, bf16_t* Vs, float* lnsz, int tid) {
  constexpr int LD = DH + 8, CPR = DH / 8;    // 16-byte chunks per row
  // batches of 4 chunk pairs per thread: all eight loads of a batch are issued before the first
  // LDS store waits for them, so their latencies overlap
  const int n_chunks = nc_pad * CPR;
  for (int t0 = 0; t0 < n_chunks; t0 += 4 * NT) {
    bf16x8 kv[4], vv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + u * NT + tid;
      const int r = t / CPR, c = (t - r * CPR) * 8;
      const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      kv[u] = zero;
      vv[u] = zero;
      if (t < n_chunks && r < nc) {
        const bf16_t* src = qkv + (size_t)(first + r) * ld + D + h * DH + c;
        kv[u] = *reinterpret_cast<const bf16x8*>(src);
        vv[u] = *reinterpret_cast<const bf16x8*>(src + D);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + u * NT + tid;
      const int r = t / CPR, c = (t - r * CPR) * 8;
      if (t < n_chunks) {
        *reinterpret_cast<bf16x8*>(Ks + r * LD + c) = kv[u];
        *reinterpret_cast<bf16x8*>(Vs + r * LD + c) = vv[u];
      }
    }
  }
  if (BIAS) {
    for (int t = tid; t < nc_pad; t += NT) lnsz[t] = t < nc ? log2f((float)sizes[first + t]) : 0.f;
  }
}

// Q fragments (B operand): lane (row, half) holds Q[row][16 ks + 8 half .. +7]
template <int DH>
__device__ __forceinline__ void attention_query(bf16x8 (&qf)[DH / 16], const bf16_t* qrow) {
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
}

// S^T block: logits of keys kb .. kb + 31
template <int DH>
__device__ __forceinline__ void attention_logits(floatx16& sacc, const bf16_t* Ks, const bf16x8 (&qf)[DH / 16], int kb, int fr, int fk) {
#pragma unroll
  for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    const bf16x8 kf = *reinterpret_cast<const bf16x8*>(Ks + (kb + fr) * (DH + 8) + ks * 16 + fk * 8);
    sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sacc, 0, 0, 0);
  }
}

// The block's largest logit per row.
// Logits in base-2 units, t = s * (scale * log2 e) [+ log2(size)], so that exp(s - m) is one
// v_exp_f32.  Without the size bias the scaling is folded into the exponent's argument,
// exp2(fma(s, scale2, -m)): the maximum is taken over the raw products (scale2 > 0) and scaled
// once per row.  Only the chunk's last block can hold keys past the end.
template <bool BIAS>
__device__ __forceinline__ float attention_block_max(floatx16& sacc, const float* lnsz, float scale2, int kb, int nc, int fk) {
  float mx = -INFINITY;
  if (BIAS) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      sacc[e] = sacc[e] * scale2 + lnsz[kb + 8 * (e >> 2) + 4 * fk + (e & 3)];
  }
  if (kb + 32 > nc) {   // wave-uniform: keys past the end of the sequence
#pragma unroll
    for (int e = 0; e < 16; ++e)
      sacc[e] = (kb + 8 * (e >> 2) + 4 * fk + (e & 3)) < nc ? sacc[e] : -INFINITY;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sacc[e]);
  mx = xor32_max(mx);
  if (!BIAS) mx *= scale2;
  return mx;
}

// The block's weights in place of its logits, and their sum over the lane's keys.
template <bool BIAS>
__device__ __forceinline__ float attention_weights(floatx16& sacc, float scale2, float m) {
  float psum = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const float pv = BIAS ? __builtin_amdgcn_exp2f(sacc[e] - m) : __builtin_amdgcn_exp2f(fmaf(sacc[e], scale2, -m));
    sacc[e] = pv;
    psum += pv;
  }
  return psum;
}

// V^T fragment (A operand) of tile t of O^T for the 16 keys from kb + 16 kk on.
// transposing reads: lane s of each 16-lane group points at V[k0 + s/4][d0 + 4 (s & 3)]
template <int DH>
__device__ __forceinline__ bf16x8 attention_values(const bf16_t* Vs, int kb, int kk, int t, int lane) {
  constexpr int LD = DH + 8;
  const int s16 = lane & 15, d0 = ((lane >> 4) & 1) * 16, k0 = kb + 16 * kk + 4 * (lane >> 5);
  const bf16_t* vp = Vs + (k0 + (s16 >> 2)) * LD + t * 32 + d0 + 4 * (s16 & 3);
  const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t*)(vp));
  const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t*)(vp + 8 * LD));
  const short8_t both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  bf16x8 vf;
  __builtin_memcpy(&vf, &both, 16);
  return vf;
}

// Tile t of the lane's output row.
template <int DH>
__device__ __forceinline__ void attention_store(bf16_t* orow, const floatx16& oacc, float inv, int t, int fk) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int d = t * 32 + g * 8 + fk * 4;
    if (d < DH) {
      bf16x4 ov = {(bf16_t)(oacc[g * 4 + 0] * inv), (bf16_t)(oacc[g * 4 + 1] * inv),
                   (bf16_t)(oacc[g * 4 + 2] * inv), (bf16_t)(oacc[g * 4 + 3] * inv)};
      *reinterpret_cast<bf16x4*>(orow + d) = ov;
    }
  }
}

// LDS of a head on NW waves: keys (and, in their place, weights: shared body) | values | log2 sizes | block maxima, sums and factors.
// The reads of V^T's last tile may run past DH: four more rows keep them in bounds.
constexpr size_t attention_keys_bytes(int dh, int kc, int nw, int kg) {
  const size_t keys = (size_t)kc * (dh + 8) * sizeof(bf16_t), weights = kg > 1 ? (size_t)nw / kg * kc * 32 * sizeof(bf16_t) : 0;
  return keys > weights ? keys : weights;
}
constexpr size_t attention_lds_bytes(int dh, int kc, int nw, int kg) {
  const size_t stats = kg > 1 ? (size_t)nw / kg * kc * 4 * sizeof(float) : 0;
  return (attention_keys_bytes(dh, kc, nw, kg) + (size_t)(kc + 4) * (dh + 8) * sizeof(bf16_t) + kc * sizeof(float) + stats + 15) & ~(size_t)15;
}

// One (query q, head h, block xblk of 32 NW query rows) on NW waves: tid = thread index among those 64 NW
// threads, smem = their LDS region.  Every __syncthreads() below is reached by all threads of the workgroup
// that share q and xblk (the trip counts depend on the query's length and xblk only), so a workgroup may run
// several heads of one query side by side, each on its own NW waves and LDS region.
template <int DH, bool BIAS, int KC, int NW>
__device__ __forceinline__ void attention_mfma_body(const bf16_t* __restrict__ qkv, const int32_t* __restrict__ sizes,
                                                    const int32_t* __restrict__ off, int D, float scale,
                                                    bf16_t* __restrict__ o, const int q, const int h, const int xblk,
                                                    unsigned char* smem, const int tid) {
  constexpr int KS = DH / 16;             // k-steps of Q K^T
  constexpr int DT = (DH + 31) / 32;      // 32-row tiles of O^T
  constexpr int LD = DH + 8;              // LDS row stride in elements (16 bytes of padding)
  bf16_t* Ks = reinterpret_cast<bf16_t*>(smem);           // [KC][LD]
  bf16_t* Vs = Ks + KC * LD;                              // [KC + 4][LD]
  float* lnsz = reinterpret_cast<float*>(Vs + (KC + 4) * LD);  // [KC] log2(size) of the chunk's keys

  const int lane = tid & 63, wave = tid >> 6;
  const int base = off[q], n = off[q + 1] - base;
  constexpr int NT = 64 * NW;             // threads: NW waves of 32 query rows each
  const int row0 = xblk * (32 * NW);
  if (row0 >= n) return;
  const size_t ld = (size_t)3 * D;
  const int fr = lane & 31, fk = lane >> 5;
  const int my_row = row0 + wave * 32 + fr;
  const bool wave_active = row0 + wave * 32 < n;

  bf16x8 qf[KS];
  attention_query<DH>(qf, qkv + (size_t)(base + (my_row < n ? my_row : n - 1)) * ld + h * DH + fk * 8);

  floatx16 oacc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[t][e] = 0.f;
  float m_run = -INFINITY, l_part = 0.f;
  const float scale2 = scale * 1.44269504088896340736f;   // logits are kept in units of ln 2

  for (int c0 = 0; c0 < n; c0 += KC) {
    const int nc = min(KC, n - c0);
    const int nc_pad = (nc + 31) & ~31;
    if (c0 > 0) __syncthreads();   // everyone is done with the previous chunk
    attention_stage<DH, BIAS, NT>(qkv, sizes, ld, D, h, base + c0, nc, nc_pad, Ks, Vs, lnsz, tid);
    __syncthreads();
    if (!wave_active) continue;

    // The key blocks are software-pipelined inside the wave: the MFMA chain of block b + 1's logits is
    // issued before the softmax arithmetic of block b starts, so the matrix pipe works under the VALU
    // instructions of the same wave (the kernel runs at two to four waves per SIMD and is bound by
    // these dependency waits, not by VALU or MFMA throughput).
    auto s_block = [&](floatx16& sacc, int kb) { attention_logits<DH>(sacc, Ks, qf, kb, fr, fk); };
    auto softmax_pv = [&](floatx16& sacc, int kb) {
      const float mx = attention_block_max<BIAS>(sacc, lnsz, scale2, kb, nc, fk);
      if (__any(mx > m_run)) {   // some row's maximum moved: rescale what has been accumulated
        const float m_new = fmaxf(m_run, mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first block (m_run = -inf)
        m_run = m_new;
        l_part *= alpha;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[t][e] *= alpha;
      }
      l_part += attention_weights<BIAS>(sacc, scale2, m_run);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {   // two k-steps of 16 keys
        bf16x8 pf;
#pragma unroll
        for (int i = 0; i < 8; ++i) pf[i] = (bf16_t)sacc[8 * kk + i];
#pragma unroll
        for (int t = 0; t < DT; ++t)
          oacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(attention_values<DH>(Vs, kb, kk, t, lane), pf, oacc[t], 0, 0, 0);
      }
    };
    const int nblk = nc_pad >> 5;
    floatx16 s_even, s_odd;
    s_block(s_even, 0);
    for (int b = 0; b < nblk; b += 2) {
      if (b + 1 < nblk) s_block(s_odd, (b + 1) * 32);
      __builtin_amdgcn_sched_barrier(0);
      softmax_pv(s_even, b * 32);
      if (b + 1 < nblk) {
        if (b + 2 < nblk) s_block(s_even, (b + 2) * 32);
        __builtin_amdgcn_sched_barrier(0);
        softmax_pv(s_odd, (b + 1) * 32);
      }
    }
  }
  if (!wave_active) return;
  const float l_tot = xor32_sum(l_part);
  if (my_row < n) {
    const float inv = 1.0f / l_tot;
    bf16_t* orow = o + (size_t)(base + my_row) * D + h * DH;
#pragma unroll
    for (int t = 0; t < DT; ++t) attention_store<DH>(orow, oacc[t], inv, t, fk);
  }
}

// The same with a row block's 32 rows on KG waves, of which NW / KG are side by side in the rows: wave kg has every KG-th block of a
// chunk's keys (logits, maximum; then, knowing the maxima of the blocks in front, weights, their sum and the factor that rescales
// what came before, all left in LDS) and tile kg of O^T, to which it adds the chunk's products block by block.  What depends on the
// order of the keys, the running maximum, the rescaling, the row sum and the products, is done block after block as by the one wave
// above: the same bits.  The next chunk's keys and values are on their way while this one is worked on.
template <int DH, bool BIAS, int KC, int NW, int KG>
__device__ __forceinline__ void attention_shared_body(const bf16_t* __restrict__ qkv, const int32_t* __restrict__ sizes,
                                                      const int32_t* __restrict__ off, int D, float scale,
                                                      bf16_t* __restrict__ o, const int q, const int h, const int xblk,
                                                      unsigned char* smem, const int tid) {
  constexpr int KS = DH / 16, DT = (DH + 31) / 32, LD = DH + 8, NT = 64 * NW, RW = NW / KG;
  constexpr int NB = KC / 32, OWN = NB / KG;   // blocks of a chunk, and of them a wave's
  constexpr int CPR = DH / 8, PIECES = KC * CPR / NT;   // 16-byte pieces of a row; of a chunk's keys, a thread's
  static_assert(DT <= KG && NB % KG == 0, "a tile of O^T to a wave, the same number of blocks to each");
  static_assert(KC * CPR % NT == 0 && KC <= NT, "the same number of pieces to each thread, one size at most");
  bf16_t* Ks = reinterpret_cast<bf16_t*>(smem);                                                      // [KC][LD]
  bf16_t* Vs = reinterpret_cast<bf16_t*>(smem + attention_keys_bytes(DH, KC, NW, KG));               // [KC + 4][LD]
  float* lnsz = reinterpret_cast<float*>(Vs + (KC + 4) * LD);                                        // [KC]

  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / RW, rw = wave % RW;
  bf16x8* weights = reinterpret_cast<bf16x8*>(smem) + rw * NB * 2 * 64;   // [NB][2][64], in place of the keys
  float* maxima = lnsz + KC + rw * NB * 32;                               // [NB][32]
  float* sums = lnsz + KC + RW * NB * 32 + rw * NB * 64;                  // [NB][64]
  float* factors = lnsz + KC + RW * NB * 96 + rw * NB * 32;               // [NB][32]
  const int base = off[q], n = off[q + 1] - base;
  const int row0 = xblk * (32 * RW);
  if (row0 >= n) return;
  const size_t ld = (size_t)3 * D;
  const int fr = lane & 31, fk = lane >> 5;
  const int my_row = row0 + rw * 32 + fr;
  const bool wave_active = row0 + rw * 32 < n;

  bf16x8 kv[PIECES], vv[PIECES];
  int sz = 0;
  auto fetch = [&](int c0) {   // rows past the end are zero
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
      const int t = u * NT + tid, r = t / CPR, c = (t - r * CPR) * 8;
      const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      kv[u] = zero;
      vv[u] = zero;
      if (c0 + r < n) {
        const bf16_t* src = qkv + (size_t)(base + c0 + r) * ld + D + h * DH + c;
        kv[u] = *reinterpret_cast<const bf16x8*>(src);
        vv[u] = *reinterpret_cast<const bf16x8*>(src + D);
      }
    }
    if (BIAS) sz = tid < KC && c0 + tid < n ? sizes[base + c0 + tid] : 1;
  };
  fetch(0);
  bf16x8 qf[KS];
  attention_query<DH>(qf, qkv + (size_t)(base + (my_row < n ? my_row : n - 1)) * ld + h * DH + fk * 8);

  floatx16 oacc;
#pragma unroll
  for (int e = 0; e < 16; ++e) oacc[e] = 0.f;
  float m_run = -INFINITY, l_part = 0.f;
  const float scale2 = scale * 1.44269504088896340736f;

  for (int c0 = 0; c0 < n; c0 += KC) {
    const int nc = min(KC, n - c0), nblk = (nc + 31) >> 5;
    if (c0 > 0) __syncthreads();   // everyone is done with the previous chunk
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
      const int t = u * NT + tid, r = t / CPR, c = (t - r * CPR) * 8;
      *reinterpret_cast<bf16x8*>(Ks + r * LD + c) = kv[u];
      *reinterpret_cast<bf16x8*>(Vs + r * LD + c) = vv[u];
    }
    if (BIAS && tid < KC) lnsz[tid] = log2f((float)sz);
    __syncthreads();
    if (c0 + KC < n) fetch(c0 + KC);
    floatx16 sacc[OWN];
    if (wave_active) {
#pragma unroll
      for (int j = 0; j < OWN; ++j) {
        const int b = kg + j * KG;
        if (b < nblk) {
          attention_logits<DH>(sacc[j], Ks, qf, b * 32, fr, fk);
          const float mx = attention_block_max<BIAS>(sacc[j], lnsz, scale2, b * 32, nc, fk);
          if (fk == 0) maxima[b * 32 + fr] = mx;
        }
      }
    }
    __syncthreads();   // the maxima are there, and the keys no longer needed
    if (wave_active) {
      float mx[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) mx[b] = b < nblk ? maxima[b * 32 + fr] : -INFINITY;
      float m = m_run, before[OWN], mine[OWN];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if (b % KG == kg) before[b / KG] = m;
        m = fmaxf(m, mx[b]);
        if (b % KG == kg) mine[b / KG] = m;
      }
      m_run = m;
#pragma unroll
      for (int j = 0; j < OWN; ++j) {
        const int b = kg + j * KG;
        if (b < nblk) {
          if (fk == 0) factors[b * 32 + fr] = __builtin_amdgcn_exp2f(before[j] - mine[j]);   // 0 on the first block
          sums[b * 64 + lane] = attention_weights<BIAS>(sacc[j], scale2, mine[j]);
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) {
            bf16x8 pf;
#pragma unroll
            for (int i = 0; i < 8; ++i) pf[i] = (bf16_t)sacc[j][8 * kk + i];
            weights[(b * 2 + kk) * 64 + lane] = pf;
          }
        }
      }
    }
    __syncthreads();
    if (wave_active && kg < DT) {
      struct Block { bf16x8 w[2], v[2]; float factor, sum; } cur, next;   // operands are read a block ahead
      auto read = [&](Block& x, int b) {
        x.factor = factors[b * 32 + fr];
        x.sum = sums[b * 64 + lane];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          x.w[kk] = weights[(b * 2 + kk) * 64 + lane];
          x.v[kk] = attention_values<DH>(Vs, b * 32, kk, kg, lane);
        }
      };
      read(cur, 0);
      for (int b = 0; b < nblk; ++b) {
        read(next, min(b + 1, nblk - 1));
        if (__any(cur.factor != 1.f)) {
          l_part *= cur.factor;
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[e] *= cur.factor;
        }
        l_part += cur.sum;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) oacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.v[kk], cur.w[kk], oacc, 0, 0, 0);
        cur = next;
      }
    }
  }
  if (wave_active && kg < DT) {
    const float l_tot = xor32_sum(l_part);
    if (my_row < n) attention_store<DH>(o + (size_t)(base + my_row) * D + h * DH, oacc, 1.0f / l_tot, kg, fk);
  }
}

template <int DH, bool BIAS, int KC, int NW, int KG>
__device__ __forceinline__ void attention_head(const bf16_t* __restrict__ qkv, const int32_t* __restrict__ sizes,
                                               const int32_t* __restrict__ off, int D, float scale, bf16_t* __restrict__ o, int q,
                                               int h, int xblk, unsigned char* smem, int tid) {
  if constexpr (KG == 1) attention_mfma_body<DH, BIAS, KC, NW>(qkv, sizes, off, D, scale, o, q, h, xblk, smem, tid);
  else attention_shared_body<DH, BIAS, KC, NW, KG>(qkv, sizes, off, D, scale, o, q, h, xblk, smem, tid);
}

// Which head (counted through all queries) and row block workgroup id has.  Workgroups go to the eight XCDs in turn: BY_HEAD gives
// the xblks row blocks of a head, which read the same keys and values, to one XCD and so to one L2, eight heads at a time (the
// heads past the last eight are dealt out).  The eight change places from group to group: lengths that alternate would
// otherwise leave the long queries to half of the XCDs (32 of 577 and 197 tokens in turn 2632 us a pass, 2672 without).
struct HeadBlock { int head, x; };
template <bool BY_HEAD>
__device__ __forceinline__ HeadBlock head_block(unsigned id, unsigned xblks, unsigned heads) {
  if (!BY_HEAD) return HeadBlock{(int)(id / xblks), (int)(id % xblks)};
  const unsigned eights = heads & ~7u;
  const bool whole = id < eights * xblks;
  const unsigned k = whole ? id >> 3 : id - eights * xblks, p = k / xblks;
  return HeadBlock{(int)(whole ? p * 8 + ((id + p) & 7) : eights + p), (int)(k - p * xblks)};
}

template <int DH, bool BIAS, int KC, int NW, int KG, bool BY_HEAD>
__global__ __launch_bounds__(64 * NW, DH <= 64 && KG == 1 ? 4 : 2) void attention_mfma_kernel(const bf16_t* __restrict__ qkv,
                                                             const int32_t* __restrict__ sizes,
                                                             const int32_t* __restrict__ off, int D, float scale,
                                                             bf16_t* __restrict__ o) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  int q = (int)blockIdx.z, h = (int)blockIdx.y, x = (int)blockIdx.x;
  if constexpr (BY_HEAD) {
    const HeadBlock b = head_block<true>(x + gridDim.x * (h + gridDim.y * q), gridDim.x, gridDim.y * gridDim.z);
    q = b.head / (int)gridDim.y;
    h = b.head - q * (int)gridDim.y;
    x = b.x;
  }
  attention_head<DH, BIAS, KC, NW, KG>(qkv, sizes, off, D, scale, o, q, h, x, smem, (int)threadIdx.x);
}

// Attention and the merge plan of a layer in ONE launch (both only read the layer's QKV projection, and
// kernels of one stream do not overlap): the first workgroups run the plan -- workgroup q the whole plan of query q
// (merge_plan_body), or, when sel_best is given, na x nb workgroups per query only its selection
// (merge_plan_select: the lists are then written beside the next launch) -- the others run attention, each on
// 8 / NW heads of one (query, row block) side by side.  The plan workgroups come first in dispatch order, so their
// long serial chains start at once and the attention workgroups fill the other CUs.  Workgroups of 512 threads:
// attention then has the shape of the stand-alone kernel (one head of eight waves, or two of four: heads in one
// workgroup share its barriers, and four heads in lock-step in 1024-thread workgroups cost attention a fifth of its
// speed), and a plan workgroup shares its CU with an attention workgroup instead of taking the CU.  Head width 64
// only (four waves per SIMD leave 128 registers per lane; two where waves share row blocks, of launches with a CU for nearly every
// workgroup).
// grid.x = B * na * nb + xblks * (H / G) * B with G = 8 / NW (na = nb = 1 for the whole plan).
constexpr int kFusedThreads = 512;
template <bool BIAS, int KC, int NW, int KG, bool BY_HEAD>
__global__ __launch_bounds__(kFusedThreads, KG == 1 ? 4 : 2) void attention_plan_kernel(
    const bf16_t* __restrict__ qkv, const int32_t* __restrict__ sizes, const int32_t* __restrict__ off, int D, int H,
    float scale, bf16_t* __restrict__ o, int B, int xblks, const int32_t* __restrict__ out_off,
    const int32_t* __restrict__ reff_arr, const int32_t* __restrict__ troff, int n_lead,
    int32_t* __restrict__ src_list, int32_t* __restrict__ row_ptr, int32_t* __restrict__ trace_src,
    int32_t* __restrict__ trace_dst, float* __restrict__ sel_best, int32_t* __restrict__ sel_bcol, int64_t sel_stride,
    int na, int nb, int unit_lds) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int DH = 64, WT = kFusedThreads, G = WT / 64 / NW;
  if ((int)blockIdx.x < B * na * nb) {   // workgroup-uniform
    const int q = (int)blockIdx.x / (na * nb), pp = (int)blockIdx.x % (na * nb);
    const PlanQuery pq = plan_query(off, out_off, reff_arr, troff, q);
    if (sel_best)   // the selection only: the lists are written beside the output projection
      merge_plan_select<bf16_t, true, true, WT>(qkv, 3 * (int64_t)D, D, H, DH, pq, n_lead, nullptr,
                                                reinterpret_cast<float*>(smem), sel_best, sel_bcol, (int)threadIdx.x,
                                                PlanPart{pp % na, na, pp / na, nb, sel_stride});
    else
      merge_plan_body<bf16_t, true, WT>(qkv, 3 * (int64_t)D, D, H, DH, pq, n_lead, src_list, row_ptr, trace_src,
                                        trace_dst, nullptr, reinterpret_cast<float*>(smem), (int)threadIdx.x);
    return;
  }
  const int hg = H / G;
  const HeadBlock b = head_block<BY_HEAD>(blockIdx.x - B * na * nb, xblks, B * hg);
  const int hgrp = b.head % hg, q = b.head / hg, xblk = b.x;
  const int unit = (int)threadIdx.x / (64 * NW), tid = (int)threadIdx.x % (64 * NW);
  attention_head<64, BIAS, KC, NW, KG>(qkv, sizes, off, D, scale, o, q, hgrp * G + unit, xblk, smem + (size_t)unit * unit_lds, tid);
}

// Without shared keys: sequences of up to 128 rows (and those beyond 256) take four waves per workgroup, keys and values
// staged 128 at a time ((128 + 132) rows of DH + 8 bf16 = 37 KB at DH = 64, so four workgroups share
// a CU and cover each other's MFMA-dependency and barrier waits).  Sequences of 129 .. 256 rows: one
// workgroup of eight waves per (query, head) instead of two of four, with the head's keys and values
// staged once and in one piece (75 KB at DH = 64, two workgroups per CU): one load phase per
// workgroup instead of two (measured on MI355X, batch 64, 12 heads: 26.3 us against 27.2 at n = 197,
// 18.2 against 20.6 at n = 133).  On its own and at DH = 64 two
// workgroups of four are faster where every one finds a CU (7 / 10 queries, 12 heads, 165 tokens 7.2 / 7.3 -> 7.0 / 7.3, 197 8.3 / 8.4 -> 7.5 / 7.8, 256 9.5 /
// 9.7 -> 8.0 / 8.5; 133 6.3 / 6.4 -> 6.5 / 7.0).  At DH = 64 the same form takes longer sequences whose last block of 256 rows is more than half full
// (of 320, where it is not, 16 / 32 / 64 queries 18.3 / 27.9 / 45.5 -> 20.2 / 32.1 / 53.3): beside a selection always (passes of 10 / 24 of 485
// and 197 tokens with r = 23 1148 / 1829 -> 1137 / 1799, 16 of 650 with r = 16 2663 -> 2645), on its own where it halves the rounds of the
// CUs, all queries having as many blocks.  us, four waves / eight (12 heads): 400 tokens, rounds 1 / 1 (5 queries) 12.7 / 13.7, 2 / 1 (8) 17.0 /
// 14.3, 3 / 2 (13) 23.1 / 23.8, 4 / 2 (19) 29.3 / 25.9, 5 / 3 (24) 35.8 / 36.0, 8 / 4 (42) 52.0 / 46.7; 900 tokens, 2 / 1 (4) 31.3 / 29.3, 3 / 2 (7) 41.9 / 44.0, 4 / 2 (9)
// 53.1 / 46.1, 5 / 3 (12) 66.3 / 69.2, 7 / 4 (18) 87.7 / 91.6.  With workgroups that have no rows it depends on where these fall: 650 and 197 in turn, 16
// heads, 5 queries 24.4 / 21.1, 8 27.6 / 33.5, 20 48.8 / 52.7.
//
// Launches that leave CUs idle last as long as a wave's chain of key blocks (logits, softmax, product, 0.6 us each): four waves share a
// row block (attention_shared_body), in blocks of 32 rows while each of these finds a CU of its own, in blocks of 64 while those do.
// Measured, us without and with (12 heads): one query of 101 / 197 / 256 / 577 tokens 5.0 / 8.0 / 9.1 / 14.2 -> 4.0 / 5.3 / 5.4 / 10.7, with sizes
// of 197 8.6 -> 5.5; three of 197 8.1 -> 5.6; blocks of 64, five of 197 8.2 -> 6.5, seven of 165 7.2 -> 5.9, three of 400 11.4 -> 9.7.  Past those
// lines a CU's second workgroup waits for its registers: seven of 197 8.3 and 11.2, four of 400 11.5 and 19.0, ten of 577 and 197 in
// turn 27.0 and 41.5.  Two waves a row block are nowhere faster than the better of the two.  Keys 256 at a time beyond 128 rows: one query
// of 197 / 400 5.6 / 8.5 -> 5.3 / 8.1, but of 101 4.0 -> 4.5 and at DH = 80 no faster.  Beside a selection of up to 256 rows, which is what such a
// launch lasts, sharing gains nothing (passes of one / two / four queries of 197 tokens with r = 16 448 / 492 / 557 us and 448 / 490 / 557; ViT-L,
// one with r = 8, 1026 and 1031); beyond 256 rows attention lasts longest (one of 577
// 785 -> 732, of 401 633 -> 592, two of 577 and 197 795 -> 696: blocks of 64 whether or not the selection leaves each a CU, 770 where it must).
// others: workgroups beside attention's, those of the plan's selection.
//
// Row blocks of a head beyond 256 rows go to one XCD (us a pass, dealt out -> by head; ViT-B unless said): beside a
// selection (10 / 32 / 64 queries of 577 and 197 tokens in turn with r = 23 1291 / 2660 / 4744 -> 1282 / 2632 / 4659);
// with shared row blocks, whose launch is less than one round of the CUs (two / three of 325 and 3 prompts 636 / 738 -> 628 /
// 730), though not for a lone query (257 448.4 -> 451.8); and from 448 blocks of 128 rows of long queries (long_blocks: those
// longer than half the longest) on (8 / 64 of 577 1652 / 8555 -> 1627 / 8432, 64 of 325 4560 -> 4499, ViT-H 32 of 257 10837 ->
// 10679). Between, a chip of 1 to 2 workgroups a CU lasts as long as its fullest XCD: 5 of 513 tokens (300 blocks) 1222 -> 1238,
// 10 of 325 (360) 1255 -> 1265, 24 of 325 and 50 in turn (432) 1579 -> 1583, but 8 of 513 (480) 1624 -> 1610, 14 of 257 (504)
// 1357 -> 1354.
AttnShape attention_shape(int dh, int H, int B, int max_n, int long_blocks, int others) {
  auto blocks = [&](int rows) { return (int64_t)B * H * ((max_n + rows - 1) / rows); };
  auto shape = [&](int kc, int nw, int kg) {
    return AttnShape{kc, nw, kg, max_n > 256 && B > 1 && (others > 0 || kg > 1 || (int64_t)H * long_blocks >= 448)};
  };
  if (dh <= 80 && max_n > (others > 0 ? 256 : 64)) {
    if (blocks(32) <= 256) return shape(dh == 64 && max_n > 128 ? 256 : 128, 4, 4);
    if (dh == 64 && max_n > 128 && blocks(64) <= 256) return shape(256, 8, 4);
  }
  const int last = (max_n - 1) % 256 + 1;   // rows of the last block of 256
  auto rounds = [&](int rows) { return (blocks(rows) + 255) / 256; };
  if (others == 0 && dh == 64 && max_n > 160 && rounds(128) == 1) return shape(128, 4, 1);
  const bool halves = long_blocks == (int64_t)B * ((max_n + 127) / 128) && rounds(128) >= 2 * rounds(256);
  if (max_n > 128 && last > 128 && (max_n <= 256 || (dh == 64 && (others > 0 || halves)))) return shape(dh <= 64 ? 256 : 128, 8, 1);
  return shape(128, 4, 1);
}

template <int DH, bool BIAS>
static hipError_t attention_mfma_b(const void* qkv, const int32_t* sz, const int32_t* d_off, int B, int max_n, int long_blocks,
                                   int D, int H, float scale, void* o, hipStream_t s) {
  const AttnShape sh = attention_shape(DH, H, B, max_n, long_blocks, 0);
#define OTAS_ATTN(KC, NWV, KG)                                                                                    \
  if (sh.kc == KC && sh.nw == NWV && sh.kg == KG) {                                                               \
    constexpr size_t lds = attention_lds_bytes(DH, KC, NWV, KG);                                                  \
    constexpr int rows = 32 * NWV / KG;                                                                           \
    constexpr bool longer = DH <= 64 || NWV == 4;   /* whether the form takes more than 256 rows */                 \
    auto kern = sh.by_head ? attention_mfma_kernel<DH, BIAS, KC, NWV, KG, longer>                                 \
                           : attention_mfma_kernel<DH, BIAS, KC, NWV, KG, false>;                                 \
    hipError_t e = set_max_dynamic_lds((const void*)kern, (int)lds);                                              \
    if (e != hipSuccess) return e;                                                                                \
    dim3 grid((max_n + rows - 1) / rows, H, B), block(64 * NWV);                                                  \
    kern<<<grid, block, lds, s>>>((const bf16_t*)qkv, sz, d_off, D, scale, (bf16_t*)o);                           \
    return hipGetLastError();                                                                                     \
  }
  OTAS_ATTN(128, 4, 1)
  if constexpr (DH <= 80) { OTAS_ATTN(128, 4, 4) }
  OTAS_ATTN((DH <= 64 ? 256 : 128), 8, 1)   // wider heads: two pieces
  if constexpr (DH == 64) {
    OTAS_ATTN(256, 4, 4)
    OTAS_ATTN(256, 8, 4)
  }
#undef OTAS_ATTN
  return hipErrorInvalidValue;
}

template <int DH>
static hipError_t attention_mfma(const void* qkv, const int32_t* sz, const int32_t* d_off, int B, int max_n, int long_blocks,
                                 int D, int H, float scale, void* o, hipStream_t s) {
  return sz ? attention_mfma_b<DH, true>(qkv, sz, d_off, B, max_n, long_blocks, D, H, scale, o, s)
            : attention_mfma_b<DH, false>(qkv, sz, d_off, B, max_n, long_blocks, D, H, scale, o, s);
}

// LDS of the fused kernel's attention workgroups as the number of the selection's is chosen by: one head of eight waves with
// all keys staged for 129 .. 256 rows, else two heads of four waves with 128 keys each (75 KB either way; longer
// sequences in pieces of 256 take no more, two heads of shared row blocks 155 KB, with a CU for every workgroup).
static size_t fused_attention_lds(int max_n) {
  return max_n > 128 && max_n <= 256 ? attention_lds_bytes(64, 256, 8, 1) : 2 * attention_lds_bytes(64, 128, 4, 1);
}

// How launch_attention_plan runs this case (pure host; not at all: na = 0).  Below two tokens there is nothing to select.
FusedPlan attention_plan_how(int dtype, int B, int max_n, int D, int H, bool lists_elsewhere) {
  FusedPlan how = {0, 0};
  if (B <= 0 || H <= 0 || D <= 0 || max_n < 2 || max_n > kPlanThreads) return how;
  if (dtype == 0) {   // f32 models: the selection only
    const int dh = D / H;
    if (!lists_elsewhere || D % H != 0 || dh % 4 != 0 || dh > 128) return how;
    const PlanParts p = plan_parts(B, max_n, dh, attention_f32_lds(dh));
    if (plan_select_lds_bytes(max_n, dh, p.a, p.b) > 160 * 1024) return how;
    return FusedPlan{p.a, p.b};
  }
  if (D != 64 * H) return how;
  const int G = (max_n > 128 && max_n <= 256) ? 1 : 2;   // heads per workgroup: 8 waves / (8 or 4 waves per head)
  if (H % G != 0) return how;
  if (lists_elsewhere) {
    const PlanParts p = plan_parts(B, max_n, 64, fused_attention_lds(max_n));
    if (plan_select_lds_bytes(max_n, 64, p.a, p.b) > 160 * 1024) return how;
    how.na = p.a;
    how.nb = p.b;
  } else if (merge_plan_lds_bytes(max_n, 64) <= 160 * 1024) {
    how.na = how.nb = 1;
  }
  return how;
}

// Attention of a layer together with the layer's merge plan (bf16, head width 64, H a multiple of the heads a
// workgroup takes); hipErrorInvalidValue for what attention_plan_how does not take -- the caller then launches
// the two kernels one after the other.
hipError_t launch_attention_plan(int dtype, const void* qkv, const int32_t* sizes, const int32_t* d_off, const int32_t* d_out_off,
                                 const int32_t* d_reff, const int32_t* d_troff, int B, int max_n, int long_blocks, int D, int H,
                                 bool size_bias, int n_lead, void* o, int32_t* src_list, int32_t* row_ptr,
                                 int32_t* trace_src, int32_t* trace_dst, float* sel_best, int32_t* sel_bcol,
                                 int64_t sel_stride, hipStream_t s) {
  if (B <= 0 || max_n <= 0) return hipSuccess;
  if ((sel_best == nullptr) != (sel_bcol == nullptr)) return hipErrorInvalidValue;
  const FusedPlan how = attention_plan_how(dtype, B, max_n, D, H, sel_best != nullptr);
  if (how.na == 0) return hipErrorInvalidValue;
  if (dtype == 0) {
    const int dh = D / H, xblks = (max_n + 31) / 32;
    const size_t sel_lds = plan_select_lds_bytes(max_n, dh, how.na, how.nb), attn_lds = attention_f32_lds(dh);
    const dim3 grid((unsigned)(B * how.na * how.nb + xblks * H * B));
#define OTAS_FUSED(N)                                                                                             \
  do {                                                                                                            \
    auto kern = attention_select_f32_kernel<N>;                                                                   \
    hipError_t e = set_max_dynamic_lds((const void*)kern, 160 * 1024);                                            \
    if (e != hipSuccess) return e;                                                                                \
    kern<<<grid, dim3(256), attn_lds > sel_lds ? attn_lds : sel_lds, s>>>(                                        \
        (const float*)qkv, size_bias ? sizes : nullptr, d_off, D, H, 1.0f / sqrtf((float)dh), (float*)o, B, xblks, \
        d_out_off, d_reff, d_troff, n_lead, sel_best, sel_bcol, sel_stride, how.na, how.nb);                      \
  } while (0)
    if (dh <= 32) OTAS_FUSED(1);
    else if (dh <= 64) OTAS_FUSED(2);
    else if (dh <= 96) OTAS_FUSED(3);
    else OTAS_FUSED(4);
#undef OTAS_FUSED
    return hipGetLastError();
  }
  const size_t plan_lds = sel_best ? plan_select_lds_bytes(max_n, 64, how.na, how.nb) : merge_plan_lds_bytes(max_n, 64);
  const float scale = 1.0f / sqrtf(64.0f);
  const int32_t* sz = size_bias ? sizes : nullptr;
  const AttnShape sh = attention_shape(64, H, B, max_n, long_blocks, B * how.na * how.nb);
#define OTAS_FUSED(BIASV, KC, NWV, KG)                                                                            \
  if ((sz != nullptr) == BIASV && sh.kc == KC && sh.nw == NWV && sh.kg == KG) {                                   \
    constexpr int G = kFusedThreads / 64 / NWV, rows = 32 * NWV / KG;                                             \
    constexpr size_t unit = attention_lds_bytes(64, KC, NWV, KG), attn_lds = G * unit;                            \
    const size_t lds = attn_lds > plan_lds ? attn_lds : plan_lds;                                                 \
    if (H % G != 0) return hipErrorInvalidValue;                                                                  \
    auto kern = sh.by_head ? attention_plan_kernel<BIASV, KC, NWV, KG, true>                                      \
                           : attention_plan_kernel<BIASV, KC, NWV, KG, false>;                                    \
    hipError_t e = set_max_dynamic_lds((const void*)kern, 160 * 1024);                                            \
    if (e != hipSuccess) return e;                                                                                \
    const int xblks = (max_n + rows - 1) / rows;                                                                  \
    dim3 grid((unsigned)(B * how.na * how.nb + xblks * (H / G) * B)), block(kFusedThreads);                       \
    kern<<<grid, block, lds, s>>>((const bf16_t*)qkv, sz, d_off, D, H, scale, (bf16_t*)o, B, xblks, d_out_off,    \
                                  d_reff, d_troff, n_lead, src_list, row_ptr, trace_src, trace_dst, sel_best,     \
                                  sel_bcol, sel_stride, how.na, how.nb, (int)unit);                               \
    return hipGetLastError();                                                                                     \
  }
#define OTAS_FUSED_BIAS(BIASV)              \
  OTAS_FUSED(BIASV, 128, 4, 1)              \
  OTAS_FUSED(BIASV, 256, 8, 1)              \
  OTAS_FUSED(BIASV, 256, 4, 4)              \
  OTAS_FUSED(BIASV, 256, 8, 4)
  OTAS_FUSED_BIAS(true)
  OTAS_FUSED_BIAS(false)
#undef OTAS_FUSED_BIAS
#undef OTAS_FUSED
  return hipErrorInvalidValue;
}

hipError_t launch_attention(int dtype, const void* qkv, const int32_t* sizes, const int32_t* d_off, int B,
                            int max_n, int long_blocks, int D, int H, bool size_bias, void* o, hipStream_t s) {
  if (B <= 0 || max_n <= 0) return hipSuccess;
  const int dh = D / H;
  const float scale = 1.0f / sqrtf((float)dh);
  const int32_t* sz = size_bias ? sizes : nullptr;
  if (dtype != 0) {
    if (dh == 64) return attention_mfma<64>(qkv, sz, d_off, B, max_n, long_blocks, D, H, scale, o, s);
    if (dh == 80) return attention_mfma<80>(qkv, sz, d_off, B, max_n, long_blocks, D, H, scale, o, s);
    if (dh == 96) return attention_mfma<96>(qkv, sz, d_off, B, max_n, long_blocks, D, H, scale, o, s);
    if (dh == 128) return attention_mfma<128>(qkv, sz, d_off, B, max_n, long_blocks, D, H, scale, o, s);
  }
  return dtype == 0 ? attention_f32<float>(qkv, sz, d_off, B, max_n, D, H, scale, o, s)
                    : attention_f32<bf16_t>(qkv, sz, d_off, B, max_n, D, H, scale, o, s);
}

}  // namespace otas
