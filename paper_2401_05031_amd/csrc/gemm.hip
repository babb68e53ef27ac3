// Linear layers of the encoder block (Sec. II-A: per-head Q/K/V projections, the linear after
// the concatenated heads, and the MLP):  Y[M,N] = epilogue(X[M,K] W[N,K]^T + bias[N]).
//
// Kernels:
//   * gemm_f32_kernel, gemm_f32_small_kernel -- true fp32 on the matrix cores: f32 models, and the fallback for bf16
//                          shapes the bf16 kernels do not take.
//   * bf16 MFMA (v_mfma_f32_16x16x32_bf16), fp32 accumulate, operand tiles loaded straight into
//     swizzled LDS stages, fused bias / GELU / residual epilogue (bf16 models).  The 32x32x16 form does the same FLOP in
//     half the instructions but draws more power per FLOP, and large products run at the clock the power allows (a loop
//     of nothing but MFMAs on random operands: 1.91 against 1.82 PFLOP/s; 67072 x 3840 x 1280 544 against 573 us).
//       gemm_mfma_k32_kernel     128 x 128, K step 32, three workgroups per CU (K that is no multiple of 64)
//       gemm_mfma128k64_kernel   128 or 160 x 128, K step 64, two per CU (also split-K)
//       gemm_mfma256w8_kernel    160, 192, 224, 256, 288 or 320 x 256, eight waves, one per CU
//       gemm_mfma64_kernel       64 x 64, 32 x 32, 32 x 64 or 96 x 64, K step 64 (64 x 64 also 32), for products of very few rows (also
//                                split-K)
//     pick_mfma_kernel chooses among them with a cost model fitted to measured launch times; splitk_factor
//     decides by a rule of its own whether the MLP's second linear is split over K.
//     Each kernel has a PLAN form for the attention output projection, whose first workgroups write the lists
//     of the layer's merge plan (merge_plan_lists) instead of computing a tile.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "merge_plan_body.h"

namespace otas {

// At most n of this wave's loads still in flight.
#define OTAS_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))
// vmcnt(0) and lgkmcnt(0): this wave's loads have landed AND its LDS reads have returned.
#define OTAS_WAIT_LOADS_AND_LDS() __builtin_amdgcn_s_waitcnt(7 << 4)
// lgkmcnt(0) only (vmcnt, expcnt at their maxima).
#define OTAS_WAIT_LDS() __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (3 << 14))
// A barrier that this wave reaches with at most VM of its loads and none of its LDS reads still under way: what the reads were
// of may be overwritten after it, by loads or by another wave's stores.  The barrier alone does not wait, and the
// instructions that use what was read, with the compiler's wait for it, may be scheduled behind it.
template <int VM>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | (7 << 4) | ((VM >> 4) << 14));   // lgkmcnt(0)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
#define OTAS_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define OTAS_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// Output element type: the residual epilogue writes the float residual stream, the others the
// model's storage type.
template <typename T, int EPI> struct OutType { typedef T type; };
template <typename T> struct OutType<T, EPI_RESIDUAL> { typedef float type; };
template <typename T> struct OutType<T, EPI_PARTIAL> { typedef float type; };

template <int EPI>
__device__ inline float epilogue_value(float acc, float bias, const float* res, size_t idx) {
  float v = acc + bias;
  if (EPI == EPI_GELU) v = gelu_exact(v);
  if (EPI == EPI_RESIDUAL) v += res[idx];
  return v;
}

// Tile order.  Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2, and inside
// an XCD the ~32 resident workgroups are consecutive in that XCD's sequence.  Give XCD x the
// sequence positions s = id / 8 of one contiguous band of tiles, and inside the band walk groups of
// GM tile rows column by column, so that the tiles in flight on one XCD form a compact block that
// shares activation and weight panels through that L2.
template <int GM = 8>
__device__ inline void tile_of_block(int bid, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
  const int nblk = tiles_m * tiles_n;
  const int per = nblk >> 3;
  int t = bid;
  if (bid < per * 8) t = (bid & 7) * per + (bid >> 3);   // full bands; the remainder keeps its id
  const int group = GM * tiles_n;
  const int g = t / group, idx = t - g * group;
  const int rows = min(GM, tiles_m - g * GM);            // the last group may be shorter
  tile_n = idx / rows;
  tile_m = g * GM + (idx - tile_n * rows);
}

// The list phases of the merge plan inside a GEMM launch (PLAN variants of the kernels below): the launch's first
// pt.B workgroups each write the lists of one query and leave; the others compute tiles as if those did not exist.
// The attention output projection runs this way: the lists depend on the selection made beside attention one
// launch earlier, and the projection leaves CUs idle at the batch sizes this matters for.
template <int NT>
__device__ __forceinline__ void plan_tail_run(const PlanTail& pt, unsigned char* smem, int q, int tid) {
  merge_plan_lists<NT, true>(reinterpret_cast<float*>(smem), pt.best, pt.bcol, pt.nb, pt.stride,
                             plan_query(pt.in_off, pt.out_off, pt.reff, pt.troff, q), pt.src_list, pt.row_ptr,
                             pt.trace_src, pt.trace_dst, tid);
}
// The same for a grid of tile columns x tile rows: the workgroups of the first rows of the grid, as many as B takes, are the
// plan's (those past B have nothing to do).  True: this workgroup is done; else tile_row is its row of tiles.
template <int NT, bool PLAN>
__device__ __forceinline__ bool plan_tail_or_tile_row(const PlanTail& pt, unsigned char* smem, int& tile_row) {
  tile_row = (int)blockIdx.y;
  if constexpr (PLAN) {
    const int rows = (pt.B + (int)gridDim.x - 1) / (int)gridDim.x;
    if (tile_row < rows) {
      const int q = tile_row * (int)gridDim.x + (int)blockIdx.x;
      if (q < pt.B) plan_tail_run<NT>(pt, smem, q, (int)threadIdx.x);
      return true;
    }
    tile_row -= rows;
  }
  return false;
}

// ------------------------------------------------------------------------------ true fp32 on the matrix cores
// f32 models, and the fallback for bf16 shapes the bf16 MFMA kernels do not take (operands widened on the way in):
// v_mfma_f32_16x16x4_f32, whose products and sums are fp32 (256 FLOP per clock and CU, 157 TFLOP/s on the chip; the
// four lane groups of an operand hold neighbouring 16-byte pieces of a row, so a wave's load covers 64 bytes of 16 rows,
// where the 32x32x2 form takes 32 bytes of 32 rows and twice as long).
// Two kernels with the same arithmetic in the same order, so that a row's result does not depend on which one the
// batch's row count picks: K is cut into four quarters (multiples of 32), each quarter is summed from zero in
// ascending order, and the quarters are added as ((q0 + q1) + q2) + q3.
//   gemm_f32_dma_kernel    f32, K a multiple of 128.  64 x 64 tile, eight waves of 32 x 32: four for each half of K, so that
//                          a CU with a single workgroup has two waves per SIMD.  Operands straight into LDS, the next
//                          k-tile's fragments read behind this one's MFMAs.  With several tiles per CU the matrix pipe is
//                          busy 93 % of the time (4616 x 768 x 3072: 123 TFLOP/s on 876 tiles, 3.4 a CU); what a pass of
//                          1206 rows loses beyond that are the last tiles of 228 to 912 on 256 CUs.  A third stage (one
//                          workgroup per CU) is slower (4616 x 2304 x 768 133 -> 157 us), bands of tiles per XCD change
//                          nothing.
//   gemm_f32_kernel        the same tile for any other K % 8 == 0 and for bf16 operands: staged through registers (columns past K
//                          are zeroed there), the fragments of a k-tile waited for after its barrier.
//   gemm_f32_small_kernel  32 x 32 tile, four waves, one quarter of K each, operands straight into registers, the four
//                          sums added through LDS.  With few tiles a launch lasts as long as one wave's chain of
//                          MFMAs (32 clocks per column of K); a quarter of K per wave makes that four times
//                          shorter, at twice the operand bytes per FLOP.
// Measured on MI355X (us; tiles of 4 x 4 FMAs per thread on the vector ALU, gemm_f32_kernel, gemm_f32_dma_kernel): 1206 x 768
// x 3072 + residual 205, 68, 48; 1206 x 3072 x 768 + GELU 90, 73, 53; 1206 x 2304 x 768 -, 54, 40; 1206 x 768 x 768 + residual
// -, 20.7, 16.2.  gemm_f32_small_kernel: 402 x 192 x 768 51 -> 9, 402 x 576 x 192 16 -> 5.
constexpr int kF32SmallTiles = 512, kF32SmallTilesStaged = 600;
__host__ __device__ static inline int f32_quarter(int K) { return ((K + 3) / 4 + 31) & ~31; }

// Four consecutive outputs of row m from column n (N % 8 == 0: inside or outside as a whole).
template <typename T, int EPI>
__device__ inline void f32_epilogue4(floatx4 v, const T* __restrict__ bias, const float* res,
                                     typename OutType<T, EPI>::type* Y, int64_t m, int n, int64_t M, int N) {
  typedef typename OutType<T, EPI>::type OT;
  if (m >= M || n >= N) return;
  const size_t idx = (size_t)m * N + n;
  const floatx4 b = load4<T>(bias + n);
  Quad<OT> o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o.x[e] = from_float<OT>(epilogue_value<EPI>(v[e], b[e], res, idx + e));
  *reinterpret_cast<Quad<OT>*>(Y + idx) = o;
}

constexpr int kF32Ld = 36;   // LDS row stride in floats
constexpr size_t kF32Lds = sizeof(float) * 2 * 2 * 2 * 64 * kF32Ld;   // [K half][operand][stage][64][36]

template <typename T, int EPI>
__global__ __launch_bounds__(512) void gemm_f32_kernel(const T* __restrict__ A, const T* __restrict__ W,
                                                       const T* __restrict__ bias, const float* res,
                                                       typename OutType<T, EPI>::type* Y, int64_t M, int N, int K) {
  // rows of 32 floats padded to 36: the 16 lanes served per clock read 16 bytes of 16 consecutive rows, 9 r mod 16
  // sixteen-byte groups apart, i.e. all 64 banks once
  constexpr int LD = kF32Ld;
  extern __shared__ __attribute__((aligned(16))) float f32_lds[];
  const int lane = threadIdx.x & 63, fr = lane & 15, fk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int half = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1, tid = threadIdx.x & 255;
  float* As = f32_lds + half * (2 * 2 * 64 * LD);   // [2][64][LD]
  float* Ws = As + 2 * 64 * LD;
  const int64_t m0 = (int64_t)blockIdx.y * 64;
  const int n0 = blockIdx.x * 64;
  const int lr = tid >> 3, lk = (tid & 7) * 4;   // staging: rows lr, lr + 32; columns lk .. lk + 3
  // K-tile kt is requested two k-tiles ahead (a k-tile is 0.43 us of MFMAs, less than a load takes), into
  // registers slot kt & 1, and stored to LDS stage kt & 1 one k-tile ahead.
  const int qt = f32_quarter(K) / 32, KT = 2 * qt, k_beg = half * KT * 32;
  // Loads are never masked and the loop has no branch around one (the compiler would wait for all loads in flight):
  // rows past the end repeat the last one, columns past K are read at K - 4 and zeroed on their way to LDS.
  floatx4 ra[2][2], rw[2][2];
  const T *pa[2], *pw[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    pa[j] = A + (size_t)min(m0 + lr + 32 * j, M - 1) * K;
    pw[j] = W + (size_t)min(n0 + lr + 32 * j, N - 1) * K;
  }
  auto fetch = [&](int slot, int kt) {
    const int k = min(k_beg + kt * 32 + lk, K - 4);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      ra[slot][j] = load4<T>(pa[j] + k);
      rw[slot][j] = load4<T>(pw[j] + k);
    }
  };
  auto stage = [&](int slot, int kt) {
    const bool in = k_beg + kt * 32 + lk < K;   // K % 8 == 0
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      *reinterpret_cast<floatx4*>(As + (slot * 64 + lr + 32 * j) * LD + lk) = in ? ra[slot][j] : zero;
      *reinterpret_cast<floatx4*>(Ws + (slot * 64 + lr + 32 * j) * LD + lk) = in ? rw[slot][j] : zero;
    }
  };
  floatx4 acc[2][2], first[2][2];   // [row block][column block] of 16 x 16: the quarter being summed, the half's first one
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = first[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
  fetch(0, 0);
  fetch(1, 1);
  stage(0, 0);
  __syncthreads();
  auto step = [&](int st, int kt) {
    floatx4 a[2][2], w[2][2];   // [block][16-column half of the k-tile]
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i][g] = *reinterpret_cast<const floatx4*>(As + (st * 64 + wm * 32 + 16 * i + fr) * LD + 16 * g + 4 * fk);
        w[i][g] = *reinterpret_cast<const floatx4*>(Ws + (st * 64 + wn * 32 + 16 * i + fr) * LD + 16 * g + 4 * fk);
      }
    fetch(st, kt + 2);
    __builtin_amdgcn_sched_barrier(0);   // else the loads sink below the MFMAs that are to cover them
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i >> 1][i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i & 1][g][u], a[i >> 1][g][u], acc[i >> 1][i & 1], 0, 0, 0);
    if (kt + 1 == qt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        first[i >> 1][i & 1] = acc[i >> 1][i & 1];
        acc[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    }
    stage(st ^ 1, kt + 1);   // everyone left that stage before the barrier of the previous k-tile
    __syncthreads();
  };
  for (int kt = 0; kt < KT; kt += 2) {
    step(0, kt);
    step(1, kt + 1);
  }
  // the second half's two quarters go to the first half's waves through LDS: [quarter][64][64 + 4]
  constexpr int LDX = 68;
  const int row = wm * 32 + fr, col = wn * 32 + 4 * fk;
  if (half) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float* p = f32_lds + (row + 16 * (i >> 1)) * LDX + col + 16 * (i & 1);
      *reinterpret_cast<floatx4*>(p) = first[i >> 1][i & 1];
      *reinterpret_cast<floatx4*>(p + 64 * LDX) = acc[i >> 1][i & 1];
    }
  }
  __syncthreads();
  if (half) return;
  // W rows were the first operand: a lane holds, of output row fr, the columns 4 fk .. + 3 of every 16 x 16 block
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float* p = f32_lds + (row + 16 * (i >> 1)) * LDX + col + 16 * (i & 1);
    floatx4 v = first[i >> 1][i & 1] + acc[i >> 1][i & 1];
    v += *reinterpret_cast<const floatx4*>(p);
    v += *reinterpret_cast<const floatx4*>(p + 64 * LDX);
    f32_epilogue4<T, EPI>(v, bias, res, Y, m0 + row + 16 * (i >> 1), n0 + col + 16 * (i & 1), M, N);
  }
}

// The same tile and the same arithmetic for f32 operands whose K is a multiple of 128 (quarters of whole k-tiles: nothing to
// zero).  Operand tiles go straight into LDS (see "direct-to-LDS kernels" below; rows of 32 floats are 128 bytes, so chunk
// c of row r sits at c ^ ((r >> 1) & 7) as in the bf16 kernels), and a wave reads the fragments of k-tile t + 1 into a
// second set of registers behind the MFMAs of k-tile t: after a barrier the MFMAs start at once, and nothing of a stage is
// needed any more when its next tile is requested.  Both halves of K share the barrier.
template <typename T, int EPI, bool PLAN = false>
__global__ __launch_bounds__(512, 4) void gemm_f32_dma_kernel(const T* __restrict__ A, const T* __restrict__ W,
                                                              const T* __restrict__ bias, const float* res, float* Y,
                                                              int64_t M, int N, int K, PlanTail pt) {
  static_assert(std::is_same<T, float>::value, "the operands go to LDS as they are");
  constexpr int BK = 32, TILE = 64 * BK, NS = 2;   // floats of an operand tile
  extern __shared__ __attribute__((aligned(16))) float f32_lds[];
  const int tid = threadIdx.x, lane = tid & 63, fr = lane & 15, fk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = wave >> 2, w4 = wave & 3, wm = w4 >> 1, wn = w4 & 1;
  float* st_base = f32_lds + half * (NS * 2 * TILE);   // [NS][A 64 x 32 | W 64 x 32]
  int tile_row;
  if (plan_tail_or_tile_row<512, PLAN>(pt, reinterpret_cast<unsigned char*>(f32_lds), tile_row)) return;
  const int64_t m0 = (int64_t)tile_row * 64;
  const int n0 = blockIdx.x * 64;
  const int qt = K / 128, KT = 2 * qt;   // k-tiles of a quarter and of a half
  // wave w4 loads rows 16 w4 .. of both operand tiles, 8 rows of 128 bytes per instruction
  uint32_t a_off[2], w_off[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = w4 * 16 + j * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    const int64_t a_last = M - 1 - m0;   // rows past the end repeat the last row
    const int w_last = N - 1 - n0;
    const uint32_t ra = (uint32_t)(row < a_last ? row : a_last), rw = (uint32_t)(row < w_last ? row : w_last);
    a_off[j] = (ra * (uint32_t)K + (uint32_t)c * 4u) * (uint32_t)sizeof(float);
    w_off[j] = (rw * (uint32_t)K + (uint32_t)c * 4u) * (uint32_t)sizeof(float);
  }
  const char* a_base = reinterpret_cast<const char*>(A + (size_t)m0 * K + (size_t)half * KT * BK);
  const char* w_base = reinterpret_cast<const char*>(W + (size_t)n0 * K + (size_t)half * KT * BK);
  auto dma_one = [&](int kt, int st, int d) {   // d = 0, 1: A rows; 2, 3: W rows
    const size_t kb = (size_t)kt * BK * sizeof(float);
    const int j = d & 1;
    asm volatile("" : "+v"(d < 2 ? a_off[j] : w_off[j]));   // as in gemm_mfma256w8_kernel
    if (d < 2)
      __builtin_amdgcn_global_load_lds(OTAS_GPTR(a_base + kb + a_off[j]),
                                       OTAS_LPTR(st_base + st * 2 * TILE + (w4 * 16 + j * 8) * BK), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(OTAS_GPTR(w_base + kb + w_off[j]),
                                       OTAS_LPTR(st_base + st * 2 * TILE + TILE + (w4 * 16 + j * 8) * BK), 16, 0, 0);
  };
  floatx4 acc[2][2], first[2][2];   // [row block][column block] of 16 x 16: the quarter being summed, the half's first one
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = first[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
  floatx4 fa[2][2][2], fw[2][2][2];   // [k-tile & 1][block][16-column half of the k-tile]
  const int sw = (fr >> 1) & 7;
  auto read_frag = [&](int buf, int st, int x) {   // x = 0 .. 7: in the order the MFMAs need them
    const int g = x >> 2, i = x & 1;
    const float* p = st_base + st * 2 * TILE + (((g << 2) + fk) ^ sw) * 4 + fr * BK;
    if (x & 2) fa[buf][i][g] = *reinterpret_cast<const floatx4*>(p + (wm * 32 + 16 * i) * BK);
    else fw[buf][i][g] = *reinterpret_cast<const floatx4*>(p + TILE + (wn * 32 + 16 * i) * BK);
  };
  // What this wave finishes: rows wm * 32 + 16 half .. of the tile, two blocks of columns.
  const int orow = wm * 32 + 16 * half + fr, ocol = wn * 32 + 4 * fk;
  const int64_t m_out = m0 + orow;
  floatx4 res_v[2];
  auto step = [&](int buf, int kt, auto load, auto next) {   // buf = kt & 1, which is k-tile kt's stage too
    constexpr bool LOAD = decltype(load)::value, NEXT = decltype(next)::value;
    if constexpr (!NEXT && EPI == EPI_RESIDUAL) {   // the residual rows travel under the last k-tile
      const float* p = res + (size_t)(m_out < M ? m_out : M - 1) * N;
#pragma unroll
      for (int j = 0; j < 2; ++j) res_v[j] = *reinterpret_cast<const floatx4*>(p + (n0 + ocol + 16 * j < N ? n0 + ocol + 16 * j : 0));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[i >> 1][i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[buf][i & 1][g][u], fa[buf][i >> 1][g][u],
                                                                    acc[i >> 1][i & 1], 0, 0, 0);
          const int t = g * 16 + u * 4 + i;
          if constexpr (LOAD) { if (t % 2 == 0 && t < 8) dma_one(kt + 2, buf, t / 2); }
          if constexpr (NEXT) { if (t >= 8 && t < 16) read_frag(buf ^ 1, buf ^ 1, t - 8); }
          __builtin_amdgcn_sched_barrier(0);
        }
    if (kt + 1 == qt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        first[i >> 1][i & 1] = acc[i >> 1][i & 1];
        acc[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  // Before k-tile t's barrier a wave has its fragments of t in registers (so its stage may be written again) and its loads
  // of k-tile t + 1 have landed.
  auto sync = [&] {
    OTAS_WAIT_LOADS_AND_LDS();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
#pragma unroll
  for (int d = 0; d < 4; ++d) dma_one(0, 0, d);
#pragma unroll
  for (int d = 0; d < 4; ++d) dma_one(1, 1, d);   // KT >= 2
  OTAS_VMCNT(4);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int x = 0; x < 8; ++x) read_frag(0, 0, x);
  int kt = 0;
  for (; kt < KT - 2; kt += 2) {
    sync();
    step(0, kt, std::true_type(), std::true_type());
    sync();
    step(1, kt + 1, std::true_type(), std::true_type());
  }
  sync();
  step(0, KT - 2, std::false_type(), std::true_type());
  sync();
  step(1, KT - 1, std::false_type(), std::false_type());
  // Each half finishes one row block of 16 of every wave's two: the first half's waves send the sum of their two quarters
  // of the second block, the second half's both of theirs of the first (the order of additions is ((q0 + q1) + q2) + q3).
  constexpr int LDX = 64 + 4;
  float* x01 = f32_lds;                    // [wm][16][LDX]
  float* x2 = f32_lds + 32 * LDX;
  float* x3 = f32_lds + 64 * LDX;
  const int xr = (wm * 16 + fr) * LDX + ocol;
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();            // every wave has its last fragments: the stages may be overwritten
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (half) {
      *reinterpret_cast<floatx4*>(x2 + xr + 16 * j) = first[0][j];
      *reinterpret_cast<floatx4*>(x3 + xr + 16 * j) = acc[0][j];
    } else {
      *reinterpret_cast<floatx4*>(x01 + xr + 16 * j) = first[1][j] + acc[1][j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    floatx4 v;
    if (half) {
      v = *reinterpret_cast<const floatx4*>(x01 + xr + 16 * j);
      v += first[1][j];
      v += acc[1][j];
    } else {
      v = first[0][j] + acc[0][j];
      v += *reinterpret_cast<const floatx4*>(x2 + xr + 16 * j);
      v += *reinterpret_cast<const floatx4*>(x3 + xr + 16 * j);
    }
    const int n = n0 + ocol + 16 * j;
    if (m_out < M && n < N) {   // N % 8 == 0: four columns are inside or outside as a whole
      const floatx4 b = *reinterpret_cast<const floatx4*>(bias + n);
      floatx4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] = v[e] + b[e];
        if (EPI == EPI_GELU) o[e] = gelu_exact(o[e]);
        if (EPI == EPI_RESIDUAL) o[e] += res_v[j][e];
      }
      *reinterpret_cast<floatx4*>(Y + (size_t)m_out * N + n) = o;
    }
  }
}
constexpr size_t kF32DmaLds = sizeof(float) * 2 * 2 * 2 * 64 * 32;   // [K half][stage][operand][64][32]

template <typename T, int EPI, bool PLAN = false>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(const T* __restrict__ A, const T* __restrict__ W,
                                                             const T* __restrict__ bias, const float* res,
                                                             typename OutType<T, EPI>::type* Y, int64_t M, int N,
                                                             int K, PlanTail pt) {
  constexpr int LD = 36, NS = 4;   // batches of 32 columns, NS - 1 of them requested ahead
  __shared__ __attribute__((aligned(16))) float part[4][32][LD];
  static_assert(sizeof(part) >= kPlanListsLdsMax, "plan lists");
  const int tid = threadIdx.x, lane = tid & 63, fr = lane & 15, fk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: the loop below has scalar branches only
  int tile_row;
  if (plan_tail_or_tile_row<256, PLAN>(pt, reinterpret_cast<unsigned char*>(part), tile_row)) return;
  const int64_t m0 = (int64_t)tile_row * 32;
  const int n0 = blockIdx.x * 32;
  const int KQ = f32_quarter(K), k_beg = wave * KQ, k_end = min(K, k_beg + KQ);
  // rows past the end repeat the last one: their outputs are not stored
  const T *pa[2], *pw[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    pa[i] = A + (size_t)min(m0 + 16 * i + fr, M - 1) * K + 4 * fk;
    pw[i] = W + (size_t)min(n0 + 16 * i + fr, N - 1) * K + 4 * fk;
  }
  const int nb = k_end > k_beg ? (k_end - k_beg) / 32 : 0;   // whole batches; the last quarter may have 8, 16 or 24 more columns
  floatx4 ra[NS][2][2], rw[NS][2][2];
  auto fetch = [&](int slot, int b) {   // unmasked: batches past the last repeat it
    const int k = k_beg + 32 * min(b, nb - 1);
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        ra[slot][i][g] = load4<T>(pa[i] + k + 16 * g);
        rw[slot][i][g] = load4<T>(pw[i] + k + 16 * g);
      }
  };
  floatx4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto mfma16 = [&](const floatx4 (&w)[2], const floatx4 (&a)[2]) {   // 16 columns of K
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[i >> 1][i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i & 1][u], a[i >> 1][u], acc[i >> 1][i & 1], 0, 0, 0);
  };
  if (nb > 0) {
#pragma unroll
    for (int j = 0; j < NS - 1; ++j) fetch(j, j);
    auto batch = [&](int j, int b) {   // j = b % NS
      fetch((j + NS - 1) % NS, b + NS - 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const floatx4 w[2] = {rw[j][0][g], rw[j][1][g]}, a[2] = {ra[j][0][g], ra[j][1][g]};
        mfma16(w, a);
      }
    };
    int b = 0;
    for (; b + NS <= nb; b += NS) {   // no branch inside: the compiler would wait for every load in flight at the join
#pragma unroll
      for (int j = 0; j < NS; ++j) batch(j, b + j);
    }
#pragma unroll
    for (int j = 0; j < NS - 1; ++j)
      if (b + j < nb) batch(j, b + j);
  }
  for (int k = k_beg + 32 * nb; k < k_end; k += 16) {   // columns past the end of K are zero, as in gemm_f32_kernel
    const bool in = k + 4 * fk < k_end;
    const int kk = in ? k : k_end - 4 - 4 * fk;
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    floatx4 w[2], a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      w[i] = in ? load4<T>(pw[i] + kk) : zero;
      a[i] = in ? load4<T>(pa[i] + kk) : zero;
    }
    mfma16(w, a);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<floatx4*>(&part[wave][16 * i + fr][16 * j + 4 * fk]) = acc[i][j];
  __syncthreads();
  const int r = tid >> 3, c = (tid & 7) * 4;
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const floatx4*>(&part[w][r][c]);
  f32_epilogue4<T, EPI>(v, bias, res, Y, m0 + r, n0 + c, M, N);
}

// dma: whether the large tiles would be gemm_f32_dma_kernel's.
static bool f32_small_tiles(int64_t M, int N, bool dma) {
  // Up to two workgroups per CU the small tiles finish first, a third round of them is slower than the large tiles' one if
  // those go straight into LDS, about as fast as that of the staged kernel.
  // Measured (us, small against gemm_f32_dma_kernel): K = 768 240 small tiles 8.9 / 15.9, 312 15.6 / 16.2, 504 15.4 / 16.1,
  // 528 21.3 / 16.1; K = 3072 240 small tiles 25.5 / 51.8, 312 49.0 / 52.2, 528 71.5 / 52.6.  Against gemm_f32_kernel, 504, 552, 624,
  // 768 small tiles: f32, K = 192 6.2 / 9.1, 8.4 / 9.3, 8.5 / 9.4, 10.8 / 9.7; 776 14.7 / 22.5, 19.4 / 22.6, 19.5 / 22.7, 20.7 / 22.9; 1056 20.6 /
  // 27.4, 29.4 / 27.5, 29.7 / 27.6, 29.8 / 27.9; 3080 43.0 / 68.9, 60.5 / 68.6, 61.3 / 69.0, 61.7 / 69.1; bf16, K = 776 15.1 / 22.6, 20.3 / 22.7, 20.7 /
  // 22.7, 25.9 / 22.9; 3080 46.4 / 69.9, 67.8 / 69.8, 68.5 / 69.8, 69.1 / 70.1.
  return ((M + 31) / 32) * ((N + 31) / 32) <= (dma ? kF32SmallTiles : kF32SmallTilesStaged);
}

// The direct-to-LDS kernel takes whole k-tiles and rows that begin on 16 bytes.
static bool f32_dma_takes(const void* x, const void* w, int K) {
  return K % 128 == 0 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w)) & 15) == 0;
}

// pt: the launch's first workgroups also write the lists of pt->B queries (f32 operands and EPI_RESIDUAL only).
template <typename T>
static hipError_t linear_f32(const void* x, const void* w, const void* bias, const float* res, void* y,
                             int64_t M, int N, int K, int epi, hipStream_t s, const PlanTail* pt = nullptr) {
  constexpr bool F32 = std::is_same<T, float>::value;
  const bool can_dma = F32 && f32_dma_takes(x, w, K), small = f32_small_tiles(M, N, can_dma), dma = can_dma && !small;
  if (pt && (!F32 || epi != EPI_RESIDUAL || !(small || dma))) return hipErrorInvalidValue;
  const int b = small ? 32 : 64, cols = (N + b - 1) / b;
  const dim3 grid(cols, (unsigned)((M + b - 1) / b + (pt ? (pt->B + cols - 1) / cols : 0)), 1), block(small ? 256 : 512);
  const PlanTail tail = pt ? *pt : PlanTail{};
#define OTAS_GEMM(LDS, KERN, E, ...)                                                                        \
  do {                                                                                                      \
    auto kern = KERN;                                                                                       \
    hipError_t e = LDS ? set_max_dynamic_lds((const void*)kern, (int)(LDS)) : hipSuccess;                   \
    if (e != hipSuccess) return e;                                                                          \
    kern<<<grid, block, LDS, s>>>((const T*)x, (const T*)w, (const T*)bias, res,                            \
                                  (typename OutType<T, E>::type*)y, M, N, K, ##__VA_ARGS__);                \
  } while (0)
#define OTAS_GEMM_EPI(LDS, KERN, E, ...)                                              \
  do {                                                                               \
    if (E == EPI_NONE) OTAS_GEMM(LDS, (KERN<T, EPI_NONE>), EPI_NONE, ##__VA_ARGS__);  \
    else if (E == EPI_GELU) OTAS_GEMM(LDS, (KERN<T, EPI_GELU>), EPI_GELU, ##__VA_ARGS__); \
    else OTAS_GEMM(LDS, (KERN<T, EPI_RESIDUAL>), EPI_RESIDUAL, ##__VA_ARGS__);        \
  } while (0)
  if constexpr (F32) {
    if (pt && small) { OTAS_GEMM(0, (gemm_f32_small_kernel<float, EPI_RESIDUAL, true>), EPI_RESIDUAL, tail); return hipGetLastError(); }
    if (pt) { OTAS_GEMM(kF32DmaLds, (gemm_f32_dma_kernel<float, EPI_RESIDUAL, true>), EPI_RESIDUAL, tail); return hipGetLastError(); }
    if (dma) { OTAS_GEMM_EPI(kF32DmaLds, gemm_f32_dma_kernel, epi, tail); return hipGetLastError(); }
  }
  if (small) OTAS_GEMM_EPI(0, gemm_f32_small_kernel, epi, tail);
  else OTAS_GEMM_EPI(kF32Lds, gemm_f32_kernel, epi);
#undef OTAS_GEMM_EPI
#undef OTAS_GEMM
  return hipGetLastError();
}

// Epilogue shared by the MFMA kernels.  A lane's accumulators are 4-column groups of 16 x 16 blocks (Acc
// below), so storing them directly would touch 16 rows with 16-byte pieces per instruction.  Instead every
// wave transposes its tile through its own LDS region, 32 rows at a time: it writes its accumulators
// as floats into a [32][WN + 4] slab, reads the slab back row-major (16 bytes per lane, WN / 4
// lanes per row) and applies bias / GELU / residual there, where the bias and residual loads and the
// output stores are contiguous runs of a full row segment.  stage: this wave's region of
// 32 * (32 TN + 4) floats, no longer used by anyone else (barrier before the call).
// Residual rows of slab i of a wave's tile, in the layout the slab is read back in.
template <int TN> struct ResSlab {
  static constexpr int LPR = 8 * TN, RPI = 64 / LPR, NIT = 32 / RPI;
  floatx4 v[NIT];
  __device__ inline void load(const float* res, int64_t M, int N, int64_t m_slab, int n_wave, int lane, int rows = 32) {
    // a uniform base and 32-bit offsets: addresses of 64 bits per lane would not fit the registers of the large tiles
    const int64_t m_base = m_slab < M ? m_slab : M - 1;
    const uint32_t last = (uint32_t)(M - 1 - m_base < 31 ? M - 1 - m_base : 31);
    const char* base = reinterpret_cast<const char*>(res + (size_t)m_base * N);
    const int n = n_wave + (lane % LPR) * 4;
    const uint32_t row = lane / LPR, col = n < N ? n : 0;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if (it * RPI >= rows) break;   // a half slab
      const uint32_t r = row + it * RPI;
      v[it] = *reinterpret_cast<const floatx4*>(base + ((r < last ? r : last) * (uint32_t)N + col) * 4u);
    }
  }
};
// The bias of a tile's BN columns waits in LDS for the epilogue: each of the first BN / 8 threads fetches 8 of them
// (bias_fetch) before the operand loads and stores them (bias_stage) once the first of those have landed.  Fetched in the
// epilogue they cost every tile a round trip to L2, or to HBM for the first tiles of a column.
template <int BN>
__device__ inline bf16x8 bias_fetch(const bf16_t* __restrict__ bias, int N, int n0, int tid) {
  const int n = n0 + tid * 8;
  const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
  return tid < BN / 8 && n < N ? *reinterpret_cast<const bf16x8*>(bias + n) : zero;   // N % 8 == 0
}
template <int BN>
__device__ inline void bias_stage(bf16_t* bias_s, const bf16x8& v, int tid) {
  if (tid < BN / 8) *reinterpret_cast<bf16x8*>(bias_s + tid * 8) = v;
}

// A wave's accumulators, RB x CB blocks of 16 x 16 (a lane holds, of block row lane & 15, four
// consecutive columns), as the epilogues see them: slab i (32 rows; the last has 16 where RB is odd) is 2 CB quads per lane;
// quad k sits at row(k), col(k) of the slab and takes bias quad k % CB.
template <int RB, int CB> struct Acc {
  static constexpr int NB = CB, SLABS = (RB + 1) / 2;
  floatx4 v[RB][CB];
  __device__ inline void clear() {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) v[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ inline void mfma(int i, int j, const bf16x8& w, const bf16x8& a) {
    v[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, v[i][j], 0, 0, 0);
  }
  __device__ inline const floatx4& quad(int i, int k) const { return v[2 * i + k / CB][k % CB]; }
  static constexpr __device__ inline int rows(int i) { return 2 * i + 2 <= RB ? 32 : 16; }   // of slab i
  static __device__ inline int row(int k, int lane) { return 16 * (k / CB) + (lane & 15); }
  static __device__ inline int col(int k, int lane) { return 16 * (k % CB) + 4 * (lane >> 4); }
};

// bias_s: the bias of this wave's 32 TN columns in LDS.  first: the residual rows of slab 0, already requested
// (HAVE_FIRST), so that the epilogue does not begin with a round trip to HBM.
template <int EPI, int RB, int CB, bool HAVE_FIRST = false>
__device__ inline void mfma_epilogue(const Acc<RB, CB>& acc, float* stage, const bf16_t* bias_s,
                                     const float* res, typename OutType<bf16_t, EPI>::type* Y, int64_t M, int N,
                                     int64_t m_wave, int n_wave, int lane,
                                     const ResSlab<CB / 2>& first = ResSlab<CB / 2>{}) {
  typedef Acc<RB, CB> A;
  constexpr int TN = CB / 2;
  constexpr int WN = 32 * TN, LDR = WN + 4;
  constexpr int LPR = WN / 4;      // lanes per row when reading back
  constexpr int RPI = 64 / LPR;    // rows per read-back instruction
  constexpr int NIT = 32 / RPI;
  const int rrow = lane / LPR, rcol = (lane % LPR) * 4;
  const int n = n_wave + rcol;
  const bool n_ok = n < N;         // N % 8 == 0: a 4-column group is inside or outside as a whole
  bf16x4 bb = {(bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f};
  if (EPI != EPI_PARTIAL) bb = *reinterpret_cast<const bf16x4*>(bias_s + rcol);
  // The residual rows of slab i + 1 are requested before slab i goes through LDS, so their latency
  // is covered by a whole slab's work instead of being waited for once per slab.  Without the first slab's rows (320-row
  // tiles: no registers for two slabs of them) a slab's rows are requested as it leaves its accumulators.
  ResSlab<TN> rr[2];
  if (EPI == EPI_RESIDUAL && HAVE_FIRST) rr[0] = first;
#pragma unroll
  for (int i = 0; i < A::SLABS; ++i) {
    const int64_t m_slab = m_wave + i * 32;
    if (EPI == EPI_RESIDUAL && HAVE_FIRST && i + 1 < A::SLABS)
      rr[(i + 1) & 1].load(res, M, N, m_slab + 32, n_wave, lane, A::rows(i + 1));
#pragma unroll
    for (int k = 0; k < CB * A::rows(i) / 16; ++k)
      *reinterpret_cast<floatx4*>(stage + A::row(k, lane) * LDR + A::col(k, lane)) = acc.quad(i, k);
    if (EPI == EPI_RESIDUAL && !HAVE_FIRST) {
      __builtin_amdgcn_sched_barrier(0);
      rr[i & 1].load(res, M, N, m_slab, n_wave, lane, A::rows(i));
    }
    // the slab is read back four rows per lane at a time before anything is stored: one LDS wait per group
    // instead of one per store
    constexpr int GRP = NIT < 4 ? NIT : 4;
    floatx4 ag[GRP];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if (it * RPI >= A::rows(i)) break;
      const int row = it * RPI + rrow;
      if (it % GRP == 0) {
#pragma unroll
        for (int u = 0; u < GRP; ++u)
          ag[u] = *reinterpret_cast<const floatx4*>(stage + ((it + u) * RPI + rrow) * LDR + rcol);
      }
      const floatx4 a = ag[it % GRP];
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = EPI == EPI_PARTIAL ? a[e] : a[e] + (float)bb[e];
      if (m_slab + row < M && n_ok) {
        typedef typename OutType<bf16_t, EPI>::type OT;
        OT* yp = reinterpret_cast<OT*>(reinterpret_cast<char*>(Y + (size_t)m_slab * N) +
                                       ((uint32_t)row * (uint32_t)N + (uint32_t)n) * (uint32_t)sizeof(OT));
        static_assert(EPI == EPI_RESIDUAL || EPI == EPI_PARTIAL, "float outputs");
        floatx4 o = {v[0], v[1], v[2], v[3]};
        if (EPI == EPI_RESIDUAL) {
          const floatx4 r = rr[i & 1].v[it];
          o = floatx4{v[0] + r[0], v[1] + r[1], v[2] + r[2], v[3] + r[3]};
        }
        *reinterpret_cast<floatx4*>(yp) = o;
      }
    }
  }
}

// Epilogue for the 16-bit outputs (no residual).  Bias and GELU are applied to the accumulators in
// registers (a lane owns runs of 4 consecutive columns of one row), the results are rounded to bf16
// and only then transposed through the wave's LDS slab, [32][WN + 8] bf16: half the LDS traffic of the
// float slab, and the read-back hands every lane 8 consecutive columns, so the global stores are
// 16 bytes per lane and a row segment of 2 WN bytes goes out in one instruction.
// NT: the output goes past the L2's replacement (see streams_output).
template <int EPI, int RB, int CB, bool NT = false>
__device__ inline void mfma_epilogue_bf16(const Acc<RB, CB>& acc, bf16_t* stage, const bf16_t* bias_s, bf16_t* Y,
                                          int64_t M, int N, int64_t m_wave, int n_wave, int lane) {
  typedef Acc<RB, CB> A;
  constexpr int TN = CB / 2;
  constexpr int WN = 32 * TN, LDR = WN + 8;
  constexpr int LPR = WN / 8;      // lanes per row when reading back
  constexpr int RPI = 64 / LPR;    // rows per read-back instruction
  constexpr int NIT = 32 / RPI;
  const int rrow = lane / LPR, rcol = (lane % LPR) * 8;
  const int n_out = n_wave + rcol;
  const bool n_ok = n_out < N;     // N % 8 == 0: an 8-column group is inside or outside as a whole
  bf16x4 bb[A::NB];
#pragma unroll
  for (int k = 0; k < A::NB; ++k) bb[k] = *reinterpret_cast<const bf16x4*>(bias_s + A::col(k, lane));
#pragma unroll
  for (int i = 0; i < A::SLABS; ++i) {
    const int64_t m_slab = m_wave + i * 32;
#pragma unroll
    for (int k = 0; k < CB * A::rows(i) / 16; ++k) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc.quad(i, k)[e] + (float)bb[k % A::NB][e];
        if (EPI == EPI_GELU) v[e] = gelu_bf16(v[e]);
      }
      const bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
      *reinterpret_cast<bf16x4*>(stage + A::row(k, lane) * LDR + A::col(k, lane)) = o;
    }
    // all of the slab's rows are read back before the first is stored: one LDS wait per slab instead of one per
    // store, and one address computation (the rows of a lane are RPI * N elements apart)
    bf16x8 a[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it)
      if (it * RPI < A::rows(i)) a[it] = *reinterpret_cast<const bf16x8*>(stage + (it * RPI + rrow) * LDR + rcol);
    bf16_t* yp = Y + (size_t)(m_slab + rrow) * N + n_out;
#pragma unroll
    for (int it = 0; it < NIT; ++it)
      if (it * RPI < A::rows(i) && m_slab + it * RPI + rrow < M && n_ok) {
        bf16x8* p = reinterpret_cast<bf16x8*>(yp + (size_t)it * RPI * N);
        if (NT) __builtin_nontemporal_store(a[it], p);
        else *p = a[it];
      }
  }
}

// ------------------------------------------------------------------------------ bf16 MFMA tiles
// All MFMA kernels compute the transposed tile (W rows as the first operand, X rows as the second): a
// lane then holds, for one output row m, runs of 4 consecutive output columns n, which makes the
// epilogue's loads and stores 8- or 16-byte vectors along the row.

// ------------------------------------------------------------------------------ direct-to-LDS kernels
// Operand tiles go from global memory straight into LDS (global_load_lds_dwordx4: 16 bytes per lane,
// each wave instruction fills 1 KB of consecutive LDS; no staging registers, no ds_write) through a
// ring of stages of K step 32.  Loads complete in issue order, so "at most n still in flight"
// (s_waitcnt vmcnt(n)) means everything but the n youngest has landed; a wave waits for its own
// loads, then a raw s_barrier makes every wave's loads visible.  The compiler is kept from moving
// LDS accesses across these points by empty asm memory clobbers.
// Stage layout: rows of 64 B (32 bf16); 16-byte chunk c of row r sits at chunk c ^ ((r >> 2) & 3).
// The DMA writes are linear; a fragment read is served 16 lanes per clock and its 16 consecutive
// rows of one chunk column fall on 16 different (row mod 4, chunk position) pairs, i.e. on all 64
// banks once.  Lane i of a DMA instruction writes LDS row base + i/4, chunk position i%4, so it must
// fetch logical chunk (i%4) ^ ((row >> 2) & 3) of that row.


#define OTAS_PLAN_TAIL_OR_TILE(NT)                          \
  int bid = (int)blockIdx.x;                                \
  if constexpr (PLAN) {                                     \
    if (bid < pt.B) {                                       \
      plan_tail_run<NT>(pt, smem, bid, (int)threadIdx.x);   \
      return;                                               \
    }                                                       \
    bid -= pt.B;                                            \
  }

// ------------------------------------------------------------------------------ (64 TM) x 128, K step 32
// Four waves in a 2 x 2 arrangement, each owning (32 TM) x 64 outputs; block tile (64 TM) x 128.  The
// library runs TM = 2 (128 rows, three workgroups per CU); TM = 3 and 4 (192 / 256 rows, two per CU)
// were measured on MI355X and lose to the 256-wide kernels on every large shape (60 us against 50 us
// for 12608 x 2304 x 768) and win by less than 10 % on a handful of mid-size ones, so they are not
// dispatched.  K step 32, operand tiles loaded straight into a ring of NS = 3 LDS stages by
// global_load_lds_dwordx4 (deeper rings, NS = 4 .. 8, change nothing: a lone workgroup is bound by what
// one CU can stream from L2, about 50 GB/s, not by load latency).  Several workgroups share a CU:
// while one waits at its barrier or for its fragments, or runs its epilogue (bias, GELU, the residual
// traffic), the others keep the matrix pipe busy.
//   iteration t: wait for this wave's loads of tile t, barrier, start the loads of tile t+NS-1 into
//                the stage tile t-1 used, then the MFMAs of tile t.
template <int EPI, int NS, int TM, bool PLAN = false>
__global__ __launch_bounds__(256, TM == 2 ? 3 : 2) void gemm_mfma_k32_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, const bf16_t* __restrict__ bias, const float* res,
    typename OutType<bf16_t, EPI>::type* Y, int64_t M, int N, int K, int tiles_m, int tiles_n, PlanTail pt) {
  constexpr int WM = 32 * TM, BM = 2 * WM, BN = 128, BK = 32, WN = 64, TN = 2;
  constexpr int STAGE_A = BM * BK, STAGE_W = BN * BK;   // elements per stage
  constexpr int RB = 2 * TM, CB = 2 * TN, ND = TM + 2;   // 16-row and 16-column blocks of a wave, loads per tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem);   // [NS][BM][32]
  bf16_t* Ws = As + NS * STAGE_A;                 // [NS][128][32]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: LDS addresses of the DMA stay scalar
  const int wm = wave >> 1, wn = wave & 1;
  int tile_m, tile_n;
  OTAS_PLAN_TAIL_OR_TILE(256)
  tile_of_block(bid, tiles_m, tiles_n, tile_m, tile_n);
  const int64_t m0 = (int64_t)tile_m * BM;
  const int n0 = tile_n * BN;

  // DMA addressing: 16 rows of 64 B per instruction; wave w owns rows w*16*TM .. of the A tile and rows
  // w*32 .. of the W tile.  Global addresses: uniform base (tile origin + k) plus a constant per-lane
  // 32-bit byte offset.
  uint32_t a_off[TM], w_off[2];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int row = wave * (16 * TM) + j * 16 + (lane >> 2);
    const int c = (lane & 3) ^ ((row >> 2) & 3);
    const int64_t a_last = M - 1 - m0;                // rows past the end repeat the last row
    const uint32_t ra = (uint32_t)(row < a_last ? row : a_last);
    a_off[j] = (ra * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = wave * 32 + j * 16 + (lane >> 2);
    const int c = (lane & 3) ^ ((row >> 2) & 3);
    const int w_last = N - 1 - n0;
    const uint32_t rw = (uint32_t)(row < w_last ? row : w_last);
    w_off[j] = (rw * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
  const char* a_base = reinterpret_cast<const char*>(A + (size_t)m0 * K);
  const char* w_base = reinterpret_cast<const char*>(W + (size_t)n0 * K);
  const int KT = K / BK;
  auto dma_one = [&](int kt, int st, int d) {   // d = 0..TM-1: A rows; TM, TM+1: W rows
    const size_t kb = (size_t)((kt < KT ? kt : KT - 1) * BK) * sizeof(bf16_t);
    asm volatile("" : "+v"(d < TM ? a_off[d] : w_off[d - TM]));   // as in gemm_mfma256w8_kernel
    if (d < TM)
      __builtin_amdgcn_global_load_lds(OTAS_GPTR(a_base + kb + a_off[d]),
                                       OTAS_LPTR(As + st * STAGE_A + (wave * (16 * TM) + d * 16) * BK), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(OTAS_GPTR(w_base + kb + w_off[d - TM]),
                                       OTAS_LPTR(Ws + st * STAGE_W + (wave * 32 + (d - TM) * 16) * BK), 16, 0, 0);
  };

  Acc<2 * TM, 2 * TN> acc;
  acc.clear();

  const int fr = lane & 15, fk = lane >> 4;
  const int frag = fr * BK + (fk ^ ((fr >> 2) & 3)) * 8;   // a k-tile is one MFMA deep

  // Prologue: the epilogue's bias and first residual rows, then tiles 0 .. NS-2.  Loads complete in issue order: "at
  // most n in flight" = all but the n youngest have landed.
  bf16_t* bias_s = Ws + NS * STAGE_W;
  const bf16x8 bias_v = bias_fetch<BN>(bias, N, n0, tid);
  ResSlab<TN> first;
  if (EPI == EPI_RESIDUAL) first.load(res, M, N, m0 + wm * WM, n0 + wn * WN, lane);
#pragma unroll
  for (int t = 0; t < NS - 1; ++t)
#pragma unroll
    for (int d = 0; d < ND; ++d) dma_one(t, t, d);

  int st = 0, st_new = NS - 1;
  auto tile = [&](int kt, auto more, auto in_flight) {
    wait_barrier<decltype(in_flight)::value>();
    bf16x8 af[RB], wf[CB];
    wf[0] = *reinterpret_cast<const bf16x8*>(Ws + st * STAGE_W + wn * WN * BK + frag);
#pragma unroll
    for (int i = 0; i < RB; ++i) af[i] = *reinterpret_cast<const bf16x8*>(As + st * STAGE_A + (wm * WM + i * 16) * BK + frag);
    if constexpr (decltype(more)::value) {
#pragma unroll
      for (int d = 0; d < ND; ++d) dma_one(kt + NS - 1, st_new, d);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        acc.mfma(i, j, wf[j], af[i]);
        if (j == 0 && i < CB - 1)
          wf[i + 1] = *reinterpret_cast<const bf16x8*>(Ws + st * STAGE_W + (wn * WN + (i + 1) * 16) * BK + frag);
        __builtin_amdgcn_sched_barrier(0);
      }
    st = st + 1 == NS ? 0 : st + 1;
    st_new = st_new + 1 == NS ? 0 : st_new + 1;
  };
  static_assert(NS == 3, "the last two k-tiles below");
  constexpr std::integral_constant<int, ND * (NS - 2)> NEXT;   // tile kt landed; tile kt+1 may still be in flight
  constexpr std::integral_constant<int, 0> NONE;
  OTAS_VMCNT(NEXT.value);   // tile 0 landed, and everything requested before it
  bias_stage<BN>(bias_s, bias_v, tid);
  tile(0, std::bool_constant<true>(), NEXT);   // KT >= 2; for KT == 2 its request repeats the last tile
  for (int kt = 1; kt < KT - 2; ++kt) tile(kt, std::bool_constant<true>(), NEXT);
  if (KT > 2) tile(KT - 2, std::bool_constant<false>(), NEXT);
  tile(KT - 1, std::bool_constant<false>(), NONE);
  wait_barrier<0>();   // every wave has its last fragments: the stages become the epilogue's staging area
  if constexpr (EPI == EPI_NONE || EPI == EPI_GELU)
    mfma_epilogue_bf16<EPI, 2 * TM, 2 * TN>(acc, reinterpret_cast<bf16_t*>(smem) + wave * 32 * (WN + 8), bias_s + wn * WN, Y, M, N,
                                    m0 + wm * WM, n0 + wn * WN, lane);
  else
    mfma_epilogue<EPI, 2 * TM, 2 * TN, EPI == EPI_RESIDUAL>(acc, reinterpret_cast<float*>(smem) + wave * 32 * (WN + 4),
                                                    bias_s + wn * WN, res, Y, M, N, m0 + wm * WM, n0 + wn * WN, lane, first);
}

template <int NS, int TM>
static hipError_t linear_mfma_k32(const void* x, const void* w, const void* bias, const float* res, void* y,
                                  int64_t M, int N, int K, int epi, hipStream_t s, const PlanTail* pt) {
  constexpr int BM = 64 * TM;
  const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + 127) / 128;
  const size_t lds = ((size_t)NS * (BM + 128) * 32 + 128) * sizeof(bf16_t);   // the stages and the tile's bias
  static_assert(4 * 32 * (64 + 4) * sizeof(float) <= (size_t)NS * (BM + 128) * 32 * sizeof(bf16_t), "epilogue slab");
  static_assert(kPlanListsLdsMax <= (size_t)NS * (BM + 128) * 32 * sizeof(bf16_t), "plan lists");
  dim3 grid((unsigned)(tiles_m * tiles_n + (pt ? pt->B : 0))), block(256);
#define OTAS_MFMA(E, ...)                                                                                         \
  do {                                                                                                            \
    auto kern = gemm_mfma_k32_kernel<E, NS, TM, ##__VA_ARGS__>;                                                   \
    hipError_t e = set_max_dynamic_lds((const void*)kern, (int)lds);                                              \
    if (e != hipSuccess) return e;                                                                                \
    kern<<<grid, block, lds, s>>>((const bf16_t*)x, (const bf16_t*)w, (const bf16_t*)bias, res,                   \
                                  (typename OutType<bf16_t, E>::type*)y, M, N, K, tiles_m, tiles_n,               \
                                  pt ? *pt : PlanTail{});                                                         \
  } while (0)
  if (pt) {
    if (epi != EPI_RESIDUAL) return hipErrorInvalidValue;
    OTAS_MFMA(EPI_RESIDUAL, true);
  } else if (epi == EPI_NONE) OTAS_MFMA(EPI_NONE);
  else if (epi == EPI_GELU) OTAS_MFMA(EPI_GELU);
  else OTAS_MFMA(EPI_RESIDUAL);
#undef OTAS_MFMA
  return hipGetLastError();
}

// ------------------------------------------------------------------------------ 64 x 64 and smaller
// For products of so few rows that 128 x 128 tiles leave most CUs without a workgroup (small serving batches: a
// ViT-B query is 197 rows): block tile (32 RB) x (32 CB), four waves of (16 RB) x (16 CB) in a 2 x 2 arrangement, the same
// direct-to-LDS ring with NS = 4 stages.  64 x 64 is four times the workgroups of the 128 x 128 tiling at twice the operand
// bytes per FLOP.  Such a launch lasts as long as one workgroup's chain of k-tiles, each a barrier, an LDS round trip
// and BK / 16 MFMAs that follow one another; K step 64 halves that chain's barriers and fetches whole cache lines (64 KB
// of LDS, two workgroups per CU); K step 128 (128 KB, one per CU) was no faster with a CU for every tile and slower
// beyond.  K step 32 remains for K that is no multiple of 64.  The other tiles: pick_small_tile.
// Stage layout: 16-byte chunk c of row r sits at chunk c ^ swz(r), which puts the 16 rows that are served per clock on all
// 64 banks once.
// Measured on MI355X (us, 64 x 64, K step 32 / 64 / 128): 197 x 2304 x 768 6.3 / 5.4 / 5.6, 197 x 768 x 768 + residual 6.4 / 5.5 / 5.8,
// 197 x 3072 x 768 + GELU 6.8 / 5.9 / 6.1, 1400 x 768 x 768 9.3 / 8.5 / 11.4, 600 x 3072 x 1024 11.7 / 9.4 / 12.2.
constexpr int kSmallStages = 4;
template <int EPI, int BK, int RB, int CB, bool PLAN = false>
__global__ __launch_bounds__(256, 2) void gemm_mfma64_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, const bf16_t* __restrict__ bias, const float* res,
    typename OutType<bf16_t, EPI>::type* Y, int64_t M, int N, int K, int k_len, int tiles_m, int tiles_n, PlanTail pt) {
  constexpr int WM = 16 * RB, WN = 16 * CB, BM = 2 * WM, BN = 2 * WN, NS = kSmallStages;
  constexpr int CPR = BK / 8;                    // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;                  // rows per DMA instruction
  constexpr int NA = BM / 4 / RPI, NW = BN / 4 / RPI, ND = NA + NW;   // DMA instructions per wave and k-tile
  constexpr int KS = BK / 32;
  constexpr int STAGE_A = BM * BK, STAGE_W = BN * BK;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem);   // [NS][BM][BK]
  bf16_t* Ws = As + NS * STAGE_A;                 // [NS][BN][BK]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int tile_m, tile_n;
  OTAS_PLAN_TAIL_OR_TILE(256)
  tile_of_block(bid, tiles_m, tiles_n, tile_m, tile_n);
  const int64_t m0 = (int64_t)tile_m * BM;
  const int n0 = tile_n * BN;
  auto swz = [](int r) { return BK == 64 ? (r >> 1) & 7 : (r >> 2) & 3; };
  // DMA: wave w loads a quarter of the rows of the A tile and of the W tile, RPI rows per instruction
  uint32_t a_off[NA], w_off[NW];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int row = wave * (BM / 4) + j * RPI + lane / CPR;
    const int c = (lane % CPR) ^ swz(row);
    const int64_t last = M - 1 - m0;
    const uint32_t r = (uint32_t)(row < last ? row : last);
    a_off[j] = (r * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    const int row = wave * (BN / 4) + j * RPI + lane / CPR;
    const int c = (lane % CPR) ^ swz(row);
    const int last = N - 1 - n0;
    const uint32_t r = (uint32_t)(row < last ? row : last);
    w_off[j] = (r * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
  const char* a_base = reinterpret_cast<const char*>(A + (size_t)m0 * K + (size_t)blockIdx.y * k_len);
  const char* w_base = reinterpret_cast<const char*>(W + (size_t)n0 * K + (size_t)blockIdx.y * k_len);
  if (EPI == EPI_PARTIAL) Y += (size_t)blockIdx.y * M * N;
  const int KT = k_len / BK;
  auto dma = [&](int kt, int st) {
    const size_t kb = (size_t)((kt < KT ? kt : KT - 1) * BK) * sizeof(bf16_t);   // no branch: see the prologue
#pragma unroll
    for (int j = 0; j < (NA > NW ? NA : NW); ++j) {
      if (j < NA) {
        asm volatile("" : "+v"(a_off[j]));   // as in gemm_mfma256w8_kernel
        __builtin_amdgcn_global_load_lds(OTAS_GPTR(a_base + kb + a_off[j]),
                                         OTAS_LPTR(As + st * STAGE_A + (wave * (BM / 4) + j * RPI) * BK), 16, 0, 0);
      }
      if (j < NW) {
        asm volatile("" : "+v"(w_off[j]));
        __builtin_amdgcn_global_load_lds(OTAS_GPTR(w_base + kb + w_off[j]),
                                         OTAS_LPTR(Ws + st * STAGE_W + (wave * (BN / 4) + j * RPI) * BK), 16, 0, 0);
      }
    }
  };
  Acc<RB, CB> acc;
  acc.clear();
  const int fr = lane & 15, fk = lane >> 4;
  const int frag_row = fr * BK, sw = swz(fr);   // swz of 16 w + fr is swz of fr
  bf16_t* bias_s = Ws + NS * STAGE_W;
  bf16x8 bias_v;
  if (EPI != EPI_PARTIAL) bias_v = bias_fetch<BN>(bias, N, n0, tid);
  constexpr bool SLAB = CB % 2 == 0;   // one block of columns has an epilogue of its own
  ResSlab<SLAB ? CB / 2 : 1> first;
  if constexpr (EPI == EPI_RESIDUAL && SLAB) first.load(res, M, N, m0 + wm * WM, n0 + wn * WN, lane, RB == 1 ? 16 : 32);
  // Unconditional: behind a branch the compiler cannot count these and waits for all of them where it uses the bias (a pass of six
  // ViT-B queries 0.9 % longer).
#pragma unroll
  for (int t = 0; t < NS - 1; ++t) dma(t, t);
  int st = 0, st_new = NS - 1;
  auto tile = [&](int kt, auto more, auto in_flight) {
    wait_barrier<decltype(in_flight)::value>();
    bf16x8 af[KS][RB], wf[KS][CB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int c = (((ks << 2) + fk) ^ sw) * 8;
#pragma unroll
      for (int i = 0; i < RB; ++i)
        af[ks][i] = *reinterpret_cast<const bf16x8*>(As + st * STAGE_A + (wm * WM + 16 * i) * BK + frag_row + c);
#pragma unroll
      for (int j = 0; j < CB; ++j)
        wf[ks][j] = *reinterpret_cast<const bf16x8*>(Ws + st * STAGE_W + (wn * WN + 16 * j) * BK + frag_row + c);
    }
    if constexpr (decltype(more)::value) dma(kt + NS - 1, st_new);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < RB * CB; ++i) acc.mfma(i / CB, i % CB, wf[ks][i % CB], af[ks][i / CB]);
    st = st + 1 == NS ? 0 : st + 1;
    st_new = st_new + 1 == NS ? 0 : st_new + 1;
  };
  static_assert(NS == 4, "the last three k-tiles below");
  constexpr std::integral_constant<int, ND * (NS - 2)> TWO;   // tile kt landed; the two after it may still be in flight
  constexpr std::integral_constant<int, ND> ONE;
  constexpr std::integral_constant<int, 0> NONE;
  constexpr std::bool_constant<true> MORE;
  constexpr std::bool_constant<false> LAST;
  OTAS_VMCNT(TWO.value);   // tile 0 landed, and everything requested before it
  if (EPI != EPI_PARTIAL) bias_stage<BN>(bias_s, bias_v, tid);
  int kt = 0;
  if (KT < NS) {   // up to three k-tiles: the prologue requested more than there are (they repeat the last one)
    if (KT > 1) tile(kt++, LAST, TWO);
  } else {
    tile(kt++, MORE, TWO);
    for (; kt < KT - 3; ++kt) tile(kt, MORE, TWO);
    tile(kt++, LAST, TWO);
  }
  for (; kt < KT - 1; ++kt) tile(kt, LAST, ONE);
  tile(KT - 1, LAST, NONE);
  wait_barrier<0>();   // every wave has its last fragments: the stages become the epilogue's staging area
  if constexpr (!SLAB) {
    // 32 x 32: all waves leave their block in one slab, a thread finishes four columns of a row
    static_assert(RB == 1 && CB == 1, "256 threads, four outputs each");
    float* slab = reinterpret_cast<float*>(smem);   // [32][36]
    *reinterpret_cast<floatx4*>(slab + (wm * 16 + fr) * 36 + wn * 16 + 4 * fk) = acc.v[0][0];
    __syncthreads();
    const int r = tid >> 3, c = (tid & 7) * 4;
    const floatx4 v = *reinterpret_cast<const floatx4*>(slab + r * 36 + c);
    if (m0 + r < M && n0 + c < N) {
      typedef typename OutType<bf16_t, EPI>::type OT;
      const size_t idx = (size_t)(m0 + r) * N + n0 + c;
      bf16x4 bb = {(bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f};
      if (EPI != EPI_PARTIAL) bb = *reinterpret_cast<const bf16x4*>(bias_s + c);
      floatx4 rr = {0.f, 0.f, 0.f, 0.f};
      if (EPI == EPI_RESIDUAL) rr = *reinterpret_cast<const floatx4*>(res + idx);
      Quad<OT> o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float t = EPI == EPI_PARTIAL ? v[e] : v[e] + (float)bb[e];
        if (EPI == EPI_GELU) t = gelu_bf16(t);
        if (EPI == EPI_RESIDUAL) t += rr[e];
        o.x[e] = from_float<OT>(t);
      }
      *reinterpret_cast<Quad<OT>*>(Y + idx) = o;
    }
  } else if constexpr (EPI == EPI_NONE || EPI == EPI_GELU)
    mfma_epilogue_bf16<EPI, RB, CB>(acc, reinterpret_cast<bf16_t*>(smem) + wave * 32 * (WN + 8), bias_s + wn * WN, Y, M, N,
                                    m0 + wm * WM, n0 + wn * WN, lane);
  else
    mfma_epilogue<EPI, RB, CB, EPI == EPI_RESIDUAL>(acc, reinterpret_cast<float*>(smem) + wave * 32 * (WN + 4),
                                                    bias_s + wn * WN, res, Y, M, N, m0 + wm * WM, n0 + wn * WN, lane, first);
}

template <int BK, int RB, int CB>
static hipError_t linear_mfma64_bk(const void* x, const void* w, const void* bias, const float* res, void* y, int64_t M,
                                   int N, int K, int epi, hipStream_t s, int splits, const PlanTail* pt) {
  constexpr int BM = 32 * RB, BN = 32 * CB;
  constexpr size_t stages = (size_t)kSmallStages * (BM + BN) * BK * sizeof(bf16_t);
  const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
  const size_t lds = stages + BN * sizeof(bf16_t);   // and the tile's bias
  static_assert(4 * 32 * (16 * CB + 4) * sizeof(float) <= stages, "epilogue slab");
  static_assert(kPlanListsLdsMax <= stages, "plan lists");
  dim3 grid((unsigned)(tiles_m * tiles_n + (pt ? pt->B : 0)), (unsigned)splits), block(256);
  const int k_len = K / splits;
#define OTAS_MFMA(E, ...)                                                                                         \
  do {                                                                                                            \
    auto kern = gemm_mfma64_kernel<E, BK, RB, CB, ##__VA_ARGS__>;                                                             \
    hipError_t e = set_max_dynamic_lds((const void*)kern, (int)lds);                                              \
    if (e != hipSuccess) return e;                                                                                \
    kern<<<grid, block, lds, s>>>((const bf16_t*)x, (const bf16_t*)w, (const bf16_t*)bias, res,                   \
                                  (typename OutType<bf16_t, E>::type*)y, M, N, K, k_len, tiles_m, tiles_n,        \
                                  pt ? *pt : PlanTail{});                                                         \
  } while (0)
  if (pt) {
    if (epi != EPI_RESIDUAL || splits != 1) return hipErrorInvalidValue;
    OTAS_MFMA(EPI_RESIDUAL, true);
  } else if (epi == EPI_NONE) OTAS_MFMA(EPI_NONE);
  else if (epi == EPI_GELU) OTAS_MFMA(EPI_GELU);
  else if (epi == EPI_PARTIAL) OTAS_MFMA(EPI_PARTIAL);
  else OTAS_MFMA(EPI_RESIDUAL);
#undef OTAS_MFMA
  return hipGetLastError();
}

// Which of its tiles the small-tile kernel runs (the same bits in each).  A launch lasts as long as the fullest CU's chain
// of k-tiles, and one CU draws its operands at about 75 GB/s whatever the tile: a k-tile costs in proportion to BM + BN.  With
// a CU for every 32 x 32 or 32 x 64 tile those have the shortest chain; where 64 x 64 just takes a second workgroup per CU,
// 96 x 64 takes one.  That tile's stages fill more than half a CU's LDS, so that its second workgroup runs after the first.
// Measured on MI355X, operands from the last-level cache (us, 32 x 32 / 32 x 64 / 64 x 64 / 96 x 64): 197 x 768 x 768 + residual
// 4.1 / 4.4 / 5.1 / 6.2, 600 4.9 / 4.8 / 5.4 / 6.5, 1406 8.7 / 7.6 / 7.6 / 7.0; 197 x 2304 x 768 4.7 / 4.6 / 5.1 / 5.9, 300 5.7 / 5.7 / 5.2 /
// 5.9, 500 8.2 / 7.2 / 6.9 / 6.1, 900 12.5 / 10.8 / 10.4 / 10.9; 101 x 3072 x 768 + GELU 4.6 / 4.6 / 5.3 / 6.3, 394 8.6 / 7.5 / 7.3 / 6.6; eight partial
// products 165 x 768 x 3072 6.0 / 5.8 / 6.2 / 5.3.  32 x 128, 64 x 128, 128 x 64 and rings of six and eight stages win nowhere by
// more than 0.2 us.
struct SmallShape { int bm, bn, slots; };   // slots: workgroups on the chip
static SmallShape small_shape(SmallTile t) {
  return t == ST_32X32 ? SmallShape{32, 32, 1024} : t == ST_32X64 ? SmallShape{32, 64, 768}
         : t == ST_96X64 ? SmallShape{96, 64, 256} : SmallShape{64, 64, 512};
}
SmallTile pick_small_tile(int64_t M, int N, int K, int splits) {
  if (K % (splits * 64) != 0) return ST_64X64;   // K step 32: 64 x 64 only
  struct Cand { SmallTile t; double alpha, first, more; };   // us: launch and epilogue; per column of K, first and later rounds
  static const Cand cands[] = {{ST_64X64, 2.40, 0.0031, 0.0031}, {ST_32X32, 2.85, 0.00155, 0.00155},
                               {ST_32X64, 2.80, 0.00233, 0.00233}, {ST_96X64, 3.00, 0.0039, 0.0064}};
  const int k_len = K / splits;
  double best = 1e30;
  SmallTile pick = ST_64X64;
  for (const Cand& c : cands) {
    const SmallShape sh = small_shape(c.t);
    const int64_t tiles = ((M + sh.bm - 1) / sh.bm) * ((N + sh.bn - 1) / sh.bn) * splits;
    const double cost = c.alpha + k_len * (c.first + c.more * (double)((tiles + 255) / 256 - 1));
    if (cost < best) { best = cost; pick = c.t; }
  }
  return pick;
}

// Whether a launch of `tiles` leaves slots of its last round for B list workgroups.
static bool lists_fit(int64_t tiles, int slots, int B) { return tiles % slots != 0 && tiles % slots + B <= slots; }
// The same tile where lists ride along, unless they would not fit beside it and would beside 64 x 64.
static SmallTile pick_small_tile_with_lists(int64_t M, int N, int K, int B) {
  const SmallTile t = pick_small_tile(M, N, K, 1);
  const SmallShape sh = small_shape(t);
  return lists_fit(((M + sh.bm - 1) / sh.bm) * ((N + sh.bn - 1) / sh.bn), sh.slots, B) ? t : ST_64X64;
}

static hipError_t linear_mfma64(const void* x, const void* w, const void* bias, const float* res, void* y, int64_t M,
                                int N, int K, int epi, hipStream_t s, const PlanTail* pt = nullptr, int splits = 1) {
  if (K % (splits * 64) != 0) return linear_mfma64_bk<32, 2, 2>(x, w, bias, res, y, M, N, K, epi, s, splits, pt);
  switch (pt ? pick_small_tile_with_lists(M, N, K, pt->B) : pick_small_tile(M, N, K, splits)) {
    case ST_32X32: return linear_mfma64_bk<64, 1, 1>(x, w, bias, res, y, M, N, K, epi, s, splits, pt);
    case ST_32X64: return linear_mfma64_bk<64, 1, 2>(x, w, bias, res, y, M, N, K, epi, s, splits, pt);
    case ST_96X64: return linear_mfma64_bk<64, 3, 2>(x, w, bias, res, y, M, N, K, epi, s, splits, pt);
    default: return linear_mfma64_bk<64, 2, 2>(x, w, bias, res, y, M, N, K, epi, s, splits, pt);
  }
}

// ------------------------------------------------------------------------------ 256x256, 8 waves
// The large-shape kernel: block tile 256 x 256, 8 waves of 128 x 64 (2 x 4 arrangement), two LDS
// stages of K step 64 (128 KB; rows of 128 B, i.e. whole cache lines per row and k-tile: streaming
// 64-byte row pieces reaches ~13 TB/s from L2 on MI355X, 128-byte pieces 15-16).  128 accumulator
// registers per lane let two waves share each SIMD, so one wave's barrier / LDS waits are covered by the other's MFMAs, while the L2 traffic per MFMA is half
// that of the 128 x 128 tiling (which is bound by L2 -> LDS bandwidth: streaming operand tiles into
// LDS tops out near 13 TB/s chip-wide on MI355X).
// After each MFMA one piece of later work is issued (a fragment read for the next k-step / next
// tile, or a load instruction of the tile after next), so that this issue overlaps the MFMA's cycles
// in the matrix pipe.  A load is in flight for one whole 64-wide tile before it is needed.
// Stage layout: 16-byte chunk c of row r sits at chunk c ^ ((r >> 1) & 7) (conflict-free for the
// linear DMA writes and for the 16-lanes-per-clock fragment reads).
// The tile height is a template parameter: BM = 32 RB rows (RB = 5 .. 10: 160, 192, .. 320; a wave has RB blocks of 16) by
// 256 columns.  Whole rounds of one workgroup per CU are what this kernel costs, so the launcher picks
// the height whose tile count wastes the least of the last round.
template <int EPI, int RB, bool PLAN = false>
__global__ __launch_bounds__(512, 1) void gemm_mfma256w8_kernel(const bf16_t* __restrict__ A,
                                                                const bf16_t* __restrict__ W,
                                                                const bf16_t* __restrict__ bias, const float* res,
                                                                typename OutType<bf16_t, EPI>::type* Y, int64_t M,
                                                                int N, int K, int tiles_m, int tiles_n, bool stream,
                                                                PlanTail pt) {
  constexpr int WM = 16 * RB, BM = 2 * WM, BN = 256, BK = 64, WN = 64, TN = 2, NS = 2;
  constexpr int STAGE_A = BM * BK, STAGE_W = BN * BK;
  // DMA instructions per wave (8 rows each): NA for the A tile, 4 for W, and where RB is odd one more for A's last 32 rows,
  // which only the first four waves have
  constexpr bool ODD = RB % 2;
  constexpr int NA = BM / 64, ND = NA + 4 + ODD;
  constexpr int CB = 2 * TN, HB = 2;   // 16-column blocks of a wave; row blocks before the barrier
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem);   // [NS][BM][64]
  bf16_t* Ws = As + NS * STAGE_A;                 // [NS][256][64]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: LDS addresses of the DMA stay scalar
  const int wm = wave >> 2, wn = wave & 3;
  int tile_m, tile_n;
  OTAS_PLAN_TAIL_OR_TILE(512)
  // The float outputs have few tile columns and a long K: two rows at a time, an activation panel is still in the L2 for its
  // last column.  us with groups of 8 / 2 / 1 rows: 40000 x 1280 x 5120 518 / 484 / 478, 67072 x 1280 x 5120 865 / 836 / 840,
  // 25216 x 1024 x 4096 233 / 226 / 225, 25216 x 1024 x 1024 84 / 82 / 80, 67072 x 1280 x 1280 295 / 295 / 303.  The other
  // products are no faster that way (12608 x 3072 x 768 + GELU 61.4 / 64.4 / 65.7).
  tile_of_block<EPI == EPI_RESIDUAL ? 2 : 8>(bid, tiles_m, tiles_n, tile_m, tile_n);
  const int64_t m0 = (int64_t)tile_m * BM;
  const int n0 = tile_n * BN;

  // DMA addressing: rows of 128 B (a whole cache line of K per row and k-tile), 8 lanes per row, 8 rows
  // per instruction; wave w owns rows w*8*NA .. of the A tile and rows w*32 .. of the W tile.
  // Lane i writes LDS row base + i/8, chunk position i%8, so it fetches logical chunk
  // (i%8) ^ ((row >> 1) & 7) of that row.
  // Global addresses are a uniform base (tile origin + k, scalar registers) plus a per-lane 32-bit
  // byte offset that never changes, so issuing a load costs no vector arithmetic.
  uint32_t a_off[NA + ODD], w_off[4];
#pragma unroll
  for (int j = 0; j < NA + ODD; ++j) {
    const int row = (j < NA ? wave * (8 * NA) + j * 8 : NA * 64 + wave * 8) + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    const int64_t last = M - 1 - m0;                  // rows past the end repeat the last row
    const uint32_t r = (uint32_t)(row < last ? row : last);
    a_off[j] = (r * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = wave * 32 + j * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    const int last = N - 1 - n0;
    const uint32_t r = (uint32_t)(row < last ? row : last);
    w_off[j] = (r * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
  const char* a_base = reinterpret_cast<const char*>(A + (size_t)m0 * K);
  const char* w_base = reinterpret_cast<const char*>(W + (size_t)n0 * K);
  const int KT = K / BK;
  auto dma_one = [&](int kt, int st, int d) {   // d = 0..NA-1: A rows; NA..NA+3: W rows; NA+4: A's last rows
    if (ODD && d == ND - 1 && wave >= 4) return;
    const size_t kb = (size_t)((kt < KT ? kt : KT - 1) * BK) * sizeof(bf16_t);
    const bool is_w = d >= NA && d < NA + 4;
    const int ja = d < NA ? d : NA;
    // opaque, or the compiler keeps the sums base + offset instead, 64 bits each: 18 registers that the tile needs
    asm volatile("" : "+v"(is_w ? w_off[d - NA] : a_off[ja]));
    if (is_w)
      __builtin_amdgcn_global_load_lds(OTAS_GPTR(w_base + kb + w_off[d - NA]),
                                       OTAS_LPTR(Ws + st * STAGE_W + (wave * 32 + (d - NA) * 8) * BK), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(
          OTAS_GPTR(a_base + kb + a_off[ja]),
          OTAS_LPTR(As + st * STAGE_A + (d < NA ? wave * (8 * NA) + d * 8 : NA * 64 + wave * 8) * BK), 16, 0, 0);
  };

  Acc<RB, CB> acc;
  acc.clear();

  // Fragments of a k-step (32 columns of K): lane (row = lane & 15, lane >> 4) holds 8 columns of a row.  W's blocks have
  // two registers each, for this k-step and the next; A's are read for the next k-step as soon as their row of MFMAs has
  // been issued.
  const int fr = lane & 15, fk = lane >> 4;
  const int frag_row = fr * BK, sw = (fr >> 1) & 7;
  bf16x8 af[RB], wf[2][CB];
  auto read_a = [&](int st, int ks, int i) {
    const int c = (((ks << 2) + fk) ^ sw) * 8;
    af[i] = *reinterpret_cast<const bf16x8*>(As + st * STAGE_A + (wm * WM + i * 16) * BK + frag_row + c);
  };
  auto read_w = [&](int st, int ks, int j) {
    const int c = (((ks << 2) + fk) ^ sw) * 8;
    wf[ks][j] = *reinterpret_cast<const bf16x8*>(Ws + st * STAGE_W + (wn * WN + j * 16) * BK + frag_row + c);
  };
  // Row blocks i0 .. i1 - 1 of k-step ks.  next: the fragments of k-step ks ^ 1 are read from stage st, in the order of
  // their use: W's behind the MFMAs of row i0, A's finished blocks behind the later ones.  load(t): what else to issue
  // behind MFMA t.
  auto rows = [&](int ks, int i0, int i1, int st, auto next, auto load) {
#pragma unroll
    for (int i = i0; i < i1; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        acc.mfma(i, j, wf[ks][j], af[i]);
        if constexpr (decltype(next)::value) {
          if (i == i0) read_w(st, ks ^ 1, j);
          else if (i == i0 + 1 && j <= i0) read_a(st, ks ^ 1, j);
          else if (i > i0 + 1 && j == 0) read_a(st, ks ^ 1, i - 1);
          if (i == i1 - 1 && j == CB - 1) read_a(st, ks ^ 1, i);
        }
        load((i - i0) * CB + j);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto no_load = [](int) {};

  // Two stages.  Per tile t (stage t & 1): k-step 0, during which the fragments of k-step 1 are read; the first HB row
  // blocks of k-step 1, which cover the last of those reads; then wait for this wave's loads of tile t+1, barrier -- after
  // it nobody reads stage t & 1 any more and tile t+1 is visible --, then the rest of k-step 1 while the loads of tile t+2
  // are issued into stage t & 1 and the first fragments of tile t+1 are read.
  // The last two tiles request nothing (LOAD), the last one reads no fragments ahead either (NEXT) and waits for no loads:
  // the first residual rows, requested beside the last-but-one tile's k-step 1, may still be on their way.
  bf16_t* bias_s = Ws + NS * STAGE_W;
  const bf16x8 bias_v = bias_fetch<BN>(bias, N, n0, tid);
  constexpr bool FIRST = EPI == EPI_RESIDUAL && RB <= 8;   // larger tiles leave no registers for them
  ResSlab<TN> first;
#pragma unroll
  for (int d = 0; d < ND; ++d) dma_one(0, 0, d);
#pragma unroll
  for (int d = 0; d < ND; ++d) dma_one(1, 1, d);
  // tile 0 landed (this wave's part), and the bias before it
  if (ODD && wave >= 4) OTAS_VMCNT(ND - 1);
  else OTAS_VMCNT(ND);
  bias_stage<BN>(bias_s, bias_v, tid);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < CB; ++j) read_w(0, 0, j);
#pragma unroll
  for (int i = 0; i < RB; ++i) read_a(0, 0, i);

  auto tile = [&](int kt, auto load, auto next) {
    constexpr bool LOAD = decltype(load)::value, NEXT = decltype(next)::value;
    const int st = kt & 1;
    rows(0, 0, RB, st, std::true_type(), no_load);
    rows(1, 0, HB, st, std::false_type(), no_load);
    // tile kt+1 landed, and the fragments of k-step 1 (read from stage st above, used below) are in
    // registers: after the barrier other waves start overwriting stage st
    if constexpr (NEXT) OTAS_WAIT_LOADS_AND_LDS();
    else OTAS_WAIT_LDS();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (FIRST && NEXT && !LOAD) first.load(res, M, N, m0 + wm * WM, n0 + wn * WN, lane);
    rows(1, HB, RB, st ^ 1, next, [&](int t) {
      if constexpr (LOAD) {
        constexpr int EVERY = (RB - HB) * CB >= 2 * ND ? 2 : 1;
        if (t % EVERY == EVERY - 1 && t / EVERY < ND) dma_one(kt + 2, st, t / EVERY);
      }
    });
  };
  for (int kt = 0; kt < KT - 2; ++kt) tile(kt, std::true_type(), std::true_type());
  tile(KT - 2, std::false_type(), std::true_type());
  tile(KT - 1, std::false_type(), std::false_type());   // its barrier: no wave reads a stage any more, the epilogue may write
  if constexpr (EPI == EPI_NONE || EPI == EPI_GELU) {
    bf16_t* slab = reinterpret_cast<bf16_t*>(smem) + wave * 32 * (WN + 8);
    if (stream) mfma_epilogue_bf16<EPI, RB, CB, true>(acc, slab, bias_s + wn * WN, Y, M, N, m0 + wm * WM, n0 + wn * WN, lane);
    else mfma_epilogue_bf16<EPI, RB, CB>(acc, slab, bias_s + wn * WN, Y, M, N, m0 + wm * WM, n0 + wn * WN, lane);
  } else
    mfma_epilogue<EPI, RB, CB, FIRST>(acc, reinterpret_cast<float*>(smem) + wave * 32 * (WN + 4), bias_s + wn * WN, res, Y,
                                      M, N, m0 + wm * WM, n0 + wn * WN, lane, first);
}

// Whether a bf16 output is written past the L2's replacement (non-temporal stores): the launch's panels stay in the L2s and less
// of the output is left to write back when it ends, but what reads the output next finds less of it there.  Measured
// inside passes of 1500 ... 68000 rows (MI355X; us per block, streamed less not streamed, ranges over the sizes):
//   QKV   D = 768, 1024, 1280: 16 - 26 MB -0.9 ... +0.6, 26 - 32 +0.1 ... +1.8, 32 - 128 -0.5 ... +7.7 (mean +3), 135 - 165
//         -2.6 ... +1.8, 168 - 256 -12 ... +3.2 (mean -5), above -10 ... +0.4
//   GELU  models of 170 MB of weights and more (12 layers at D = 768, 24 at 1024, 32 at 1280): 16 - 32 MB -2.6 ... +4.7 (mean -0.2;
//         at 768 +0.9 without merging, -0.3 with), 32 - 64 -4.2 ... +1.5 (mean -1.8), 65 - 157 -4.5 ... +9.2 (mean +2.6),
//         163 - 170 -8.9 ... +3.4, above -29 ... -6
//         models that stay in the last-level cache from pass to pass (113 MB: 8 layers at 768; 75 and 42 MB: 12 at 512 and 384; 57: 4
//         at 768): 16 - 64 MB -1.5 ... +8.7 (mean +3.7), 71 - 157 -13 ... +8, above 160 -24 ... -3
// So: outputs that the 256 MB last-level cache cannot hold beside the rest, and for models of more weights than half of it
// those behind GELU that are more than half of the L2s (32 MB) and up to a quarter of the last-level cache.  The 256-wide
// kernels are picked from about 16 MB on.
bool streams_output(int64_t M, int N, int epi, int64_t model_bytes) {
  constexpr int64_t MB = 1 << 20;
  const int64_t bytes = 2 * M * N;
  return bytes > 160 * MB ||
         (epi == EPI_GELU && model_bytes > 128 * MB && bytes > 16 * MB && bytes <= 64 * MB);
}

template <int RB>
static hipError_t linear_mfma256w8(const void* x, const void* w, const void* bias, const float* res, void* y, int64_t M,
                                   int N, int K, int epi, hipStream_t s, const PlanTail* pt, int64_t model_bytes) {
  constexpr int BM = 32 * RB;
  const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + 255) / 256;
  const size_t lds = ((size_t)2 * (BM + 256) * 64 + 256) * sizeof(bf16_t);   // the stages and the tile's bias
  dim3 grid((unsigned)(tiles_m * tiles_n + (pt ? pt->B : 0))), block(512);
#define OTAS_MFMA(E, ...)                                                                                         \
  do {                                                                                                            \
    auto kern = gemm_mfma256w8_kernel<E, RB, ##__VA_ARGS__>;                                                      \
    hipError_t e = set_max_dynamic_lds((const void*)kern, (int)lds);                                              \
    if (e != hipSuccess) return e;                                                                                \
    kern<<<grid, block, lds, s>>>((const bf16_t*)x, (const bf16_t*)w, (const bf16_t*)bias, res,                   \
                                  (typename OutType<bf16_t, E>::type*)y, M, N, K, tiles_m, tiles_n,               \
                                  streams_output(M, N, epi, model_bytes), pt ? *pt : PlanTail{});                               \
  } while (0)
  if (pt) {
    if (epi != EPI_RESIDUAL) return hipErrorInvalidValue;
    OTAS_MFMA(EPI_RESIDUAL, true);
  } else if (epi == EPI_NONE) OTAS_MFMA(EPI_NONE);
  else if (epi == EPI_GELU) OTAS_MFMA(EPI_GELU);
  else OTAS_MFMA(EPI_RESIDUAL);
#undef OTAS_MFMA
  return hipGetLastError();
}

// ------------------------------------------------------------------------------ 128 or 160 x 128, K step 64
// Block tile (32 RB) x 128 with RB = 4 or 5, 4 waves of (16 RB) x 64, two LDS stages of K step 64 (rows of 128 B = whole cache
// lines, 64 or 72 KB in all, two workgroups per CU).  Same per-tile protocol as gemm_mfma256w8_kernel.
template <int EPI, int RB, bool PLAN = false>
__global__ __launch_bounds__(256, 2) void gemm_mfma128k64_kernel(const bf16_t* __restrict__ A,
                                                                 const bf16_t* __restrict__ W,
                                                                 const bf16_t* __restrict__ bias, const float* res,
                                                                 typename OutType<bf16_t, EPI>::type* Y, int64_t M,
                                                                 int N, int K, int k_len, int tiles_m, int tiles_n,
                                                                 PlanTail pt) {
  constexpr int WM = 16 * RB, BM = 2 * WM, BN = 128, BK = 64, WN = 64, TN = 2;
  constexpr int CB = 2 * TN, HB = 2, ND = RB + 4;   // as in gemm_mfma256w8_kernel
  constexpr int STAGE_A = BM * BK, STAGE_W = BN * BK;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem);   // [2][BM][64]
  bf16_t* Ws = As + 2 * STAGE_A;                  // [2][128][64]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: LDS addresses of the DMA stay scalar
  const int wm = wave >> 1, wn = wave & 1;
  int tile_m, tile_n;
  OTAS_PLAN_TAIL_OR_TILE(256)
  tile_of_block(bid, tiles_m, tiles_n, tile_m, tile_n);
  const int64_t m0 = (int64_t)tile_m * BM;
  const int n0 = tile_n * BN;

  // wave w loads rows w*8*RB .. of the A tile and w*32 .. of the W tile, 8 rows (of 128 B) per instruction.
  // Global addresses: uniform base (tile origin + k) plus a constant per-lane 32-bit byte offset.
  uint32_t a_off[RB], w_off[4];
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    const int row = wave * (8 * RB) + j * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    const int64_t last = M - 1 - m0;                  // rows past the end repeat the last row
    const uint32_t r = (uint32_t)(row < last ? row : last);
    a_off[j] = (r * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = wave * 32 + j * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    const int last = N - 1 - n0;
    const uint32_t r = (uint32_t)(row < last ? row : last);
    w_off[j] = (r * (uint32_t)K + (uint32_t)c * 8u) * (uint32_t)sizeof(bf16_t);
  }
  // split-K launches: workgroup row blockIdx.y contracts over k_len columns from blockIdx.y * k_len and writes the
  // float partial result [M, N] number blockIdx.y
  const char* a_base = reinterpret_cast<const char*>(A + (size_t)m0 * K + (size_t)blockIdx.y * k_len);
  const char* w_base = reinterpret_cast<const char*>(W + (size_t)n0 * K + (size_t)blockIdx.y * k_len);
  if (EPI == EPI_PARTIAL) Y += (size_t)blockIdx.y * M * N;
  const int KT = k_len / BK;
  auto dma_one = [&](int kt, int st, int d) {   // d < 8: A and W rows in turn; then A's other rows
    const size_t kb = (size_t)((kt < KT ? kt : KT - 1) * BK) * sizeof(bf16_t);
    const bool is_w = d < 8 && (d & 1);
    const int j = d < 8 ? d >> 1 : d - 4;
    asm volatile("" : "+v"(is_w ? w_off[j] : a_off[j]));   // as in gemm_mfma256w8_kernel
    if (is_w)
      __builtin_amdgcn_global_load_lds(OTAS_GPTR(w_base + kb + w_off[j]),
                                       OTAS_LPTR(Ws + st * STAGE_W + (wave * 32 + j * 8) * BK), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(OTAS_GPTR(a_base + kb + a_off[j]),
                                       OTAS_LPTR(As + st * STAGE_A + (wave * (8 * RB) + j * 8) * BK), 16, 0, 0);
  };

  Acc<RB, CB> acc;
  acc.clear();

  const int fr = lane & 15, fk = lane >> 4;
  const int frag_row = fr * BK, sw = (fr >> 1) & 7;
  bf16x8 af[RB], wf[2][CB];
  auto read_a = [&](int st, int ks, int i) {
    const int c = (((ks << 2) + fk) ^ sw) * 8;
    af[i] = *reinterpret_cast<const bf16x8*>(As + st * STAGE_A + (wm * WM + i * 16) * BK + frag_row + c);
  };
  auto read_w = [&](int st, int ks, int j) {
    const int c = (((ks << 2) + fk) ^ sw) * 8;
    wf[ks][j] = *reinterpret_cast<const bf16x8*>(Ws + st * STAGE_W + (wn * WN + j * 16) * BK + frag_row + c);
  };
  auto rows = [&](int ks, int i0, int i1, int st, auto next, auto load) {
#pragma unroll
    for (int i = i0; i < i1; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        acc.mfma(i, j, wf[ks][j], af[i]);
        if constexpr (decltype(next)::value) {
          if (i == i0) read_w(st, ks ^ 1, j);
          else if (i == i0 + 1 && j <= i0) read_a(st, ks ^ 1, j);
          else if (i > i0 + 1 && j == 0) read_a(st, ks ^ 1, i - 1);
          if (i == i1 - 1 && j == CB - 1) read_a(st, ks ^ 1, i);
        }
        load((i - i0) * CB + j);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto no_load = [](int) {};

  bf16_t* bias_s = Ws + 2 * STAGE_W;
  bf16x8 bias_v;
  if (EPI != EPI_PARTIAL) bias_v = bias_fetch<BN>(bias, N, n0, tid);
  ResSlab<TN> first;
  if (EPI == EPI_RESIDUAL) first.load(res, M, N, m0 + wm * WM, n0 + wn * WN, lane);
#pragma unroll
  for (int d = 0; d < ND; ++d) dma_one(0, 0, d);
#pragma unroll
  for (int d = 0; d < ND; ++d) dma_one(1, 1, d);
  OTAS_VMCNT(ND);
  if (EPI != EPI_PARTIAL) bias_stage<BN>(bias_s, bias_v, tid);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < CB; ++j) read_w(0, 0, j);
#pragma unroll
  for (int i = 0; i < RB; ++i) read_a(0, 0, i);

  auto tile = [&](int kt, auto load, auto next) {   // as in gemm_mfma256w8_kernel
    constexpr bool LOAD = decltype(load)::value, NEXT = decltype(next)::value;
    const int st = kt & 1;
    rows(0, 0, RB, st, std::true_type(), no_load);
    rows(1, 0, HB, st, std::false_type(), no_load);
    OTAS_WAIT_LOADS_AND_LDS();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    rows(1, HB, RB, st ^ 1, next, [&](int t) {
      if constexpr (LOAD) { if (t < ND) dma_one(kt + 2, st, t); }
    });
  };
  static_assert((RB - HB) * CB >= ND, "a load behind each MFMA");
  for (int kt = 0; kt < KT - 2; ++kt) tile(kt, std::true_type(), std::true_type());
  tile(KT - 2, std::false_type(), std::true_type());
  tile(KT - 1, std::false_type(), std::false_type());
  if constexpr (EPI == EPI_NONE || EPI == EPI_GELU)
    mfma_epilogue_bf16<EPI, RB, CB>(acc, reinterpret_cast<bf16_t*>(smem) + wave * 32 * (WN + 8), bias_s + wn * WN, Y, M, N,
                                    m0 + wm * WM, n0 + wn * WN, lane);
  else
    mfma_epilogue<EPI, RB, CB, EPI == EPI_RESIDUAL>(acc, reinterpret_cast<float*>(smem) + wave * 32 * (WN + 4),
                                                    bias_s + wn * WN, res, Y, M, N, m0 + wm * WM, n0 + wn * WN, lane, first);
}

template <int RB>
static hipError_t linear_mfma128k64_rb(const void* x, const void* w, const void* bias, const float* res, void* y,
                                       int64_t M, int N, int K, int epi, hipStream_t s, int splits, const PlanTail* pt) {
  constexpr int BM = 32 * RB;
  const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + 127) / 128;
  const size_t lds = ((size_t)2 * (BM + 128) * 64 + 128) * sizeof(bf16_t);   // the stages and the tile's bias
  dim3 grid((unsigned)(tiles_m * tiles_n + (pt ? pt->B : 0)), (unsigned)splits), block(256);
  const int k_len = K / splits;
#define OTAS_MFMA(E, ...)                                                                                         \
  do {                                                                                                            \
    auto kern = gemm_mfma128k64_kernel<E, RB, ##__VA_ARGS__>;                                                        \
    hipError_t e = set_max_dynamic_lds((const void*)kern, (int)lds);                                              \
    if (e != hipSuccess) return e;                                                                                \
    kern<<<grid, block, lds, s>>>((const bf16_t*)x, (const bf16_t*)w, (const bf16_t*)bias, res,                   \
                                  (typename OutType<bf16_t, E>::type*)y, M, N, K, k_len, tiles_m, tiles_n,        \
                                  pt ? *pt : PlanTail{});                                                         \
  } while (0)
  if (pt) {
    if (epi != EPI_RESIDUAL || splits != 1) return hipErrorInvalidValue;
    OTAS_MFMA(EPI_RESIDUAL, true);
  } else if (epi == EPI_NONE) OTAS_MFMA(EPI_NONE);
  else if (epi == EPI_GELU) OTAS_MFMA(EPI_GELU);
  else if (epi == EPI_PARTIAL) OTAS_MFMA(EPI_PARTIAL);
  else OTAS_MFMA(EPI_RESIDUAL);
#undef OTAS_MFMA
  return hipGetLastError();
}

// 128 or 160 rows (the same bits): 160 where that takes the fullest CU a workgroup less.  Two workgroups of a CU share its path to
// L2, so that the second costs most of a round although it runs beside the first; a tile of 160 rows costs a tenth more.  Up to
// 768 columns of K: inside a pass, whose operands come from farther away, a long chain of k-tiles wants the second workgroup beside
// it (us in a pass of 64 / 24 queries with r = 16 / 10, 128 / 160 rows: 6464 x 768 x 3072 52.5 / 61.0, two partial products of 3300 x 768 x
// 3072 28.0 / 31.6; passes of 28 and 32 queries without merging 0.9 % shorter with 160 rows up to that line).
// Measured on MI355X (us, 128 / 160 rows, in brackets the workgroups of the fullest CU): 1406 x 3072 x 768 + GELU 14.1 / 13.7 (2 / 1),
// 2000 x 2304 x 768 12.6 / 12.3 (2 / 1), 3600 22.7 / 16.7 (3 / 2), 6000 x 768 x 768 + residual 17.3 / 15.2 (2 / 1), 6000 x 768 x 3072 42.2 /
// 40.6 (2 / 1, alone), six partial products of 900 x 768 x 3072 13.1 / 12.1 (2 / 1), 8000 x 2304 x 768 34.8 / 31.4 (5 / 4); with as many either
// way 10.9 / 11.7 (1300 x 2304 x 768) to 39.8 / 43.6.  192, 224 and 256 rows: one workgroup per CU, faster than both by 0.5 us at most.
int wide_rows(int64_t M, int N, int K, int splits) {
  if (K / splits > 768) return 128;
  const int64_t cols = (int64_t)((N + 127) / 128) * splits;
  return ((M + 127) / 128 * cols + 255) / 256 > ((M + 159) / 160 * cols + 255) / 256 ? 160 : 128;
}

static hipError_t linear_mfma128k64(const void* x, const void* w, const void* bias, const float* res, void* y,
                                    int64_t M, int N, int K, int epi, hipStream_t s, int splits = 1,
                                    const PlanTail* pt = nullptr) {
  return wide_rows(M, N, K, splits) == 160 ? linear_mfma128k64_rb<5>(x, w, bias, res, y, M, N, K, epi, s, splits, pt)
                                        : linear_mfma128k64_rb<4>(x, w, bias, res, y, M, N, K, epi, s, splits, pt);
}

// Runs one named kernel (gemm_kernel_id in kernels.h); hipErrorInvalidValue if it does not take the shape.
static hipError_t linear_mfma_kernel(int kernel, const void* x, const void* w, const void* bias, const float* res,
                                     void* y, int64_t M, int N, int K, int epi, hipStream_t s,
                                     const PlanTail* pt = nullptr, int64_t model_bytes = 0) {
  const bool k32 = K % 32 == 0 && K >= 64, k64 = K % 64 == 0 && K >= 128;
  switch (kernel) {
    case GK_128_K32: return k32 ? linear_mfma_k32<3, 2>(x, w, bias, res, y, M, N, K, epi, s, pt) : hipErrorInvalidValue;
    case GK_128_K64: return k64 ? linear_mfma128k64(x, w, bias, res, y, M, N, K, epi, s, 1, pt) : hipErrorInvalidValue;
    case GK_160X256: return k64 ? linear_mfma256w8<5>(x, w, bias, res, y, M, N, K, epi, s, pt, model_bytes) : hipErrorInvalidValue;
    case GK_192X256: return k64 ? linear_mfma256w8<6>(x, w, bias, res, y, M, N, K, epi, s, pt, model_bytes) : hipErrorInvalidValue;
    case GK_224X256: return k64 ? linear_mfma256w8<7>(x, w, bias, res, y, M, N, K, epi, s, pt, model_bytes) : hipErrorInvalidValue;
    case GK_256X256: return k64 ? linear_mfma256w8<8>(x, w, bias, res, y, M, N, K, epi, s, pt, model_bytes) : hipErrorInvalidValue;
    case GK_288X256: return k64 ? linear_mfma256w8<9>(x, w, bias, res, y, M, N, K, epi, s, pt, model_bytes) : hipErrorInvalidValue;
    case GK_320X256: return k64 ? linear_mfma256w8<10>(x, w, bias, res, y, M, N, K, epi, s, pt, model_bytes) : hipErrorInvalidValue;
    case GK_64X64: return k32 ? linear_mfma64(x, w, bias, res, y, M, N, K, epi, s, pt) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

// Kernel choice by a cost model.  A kernel with tile bm x bn and S workgroup slots on the chip (256 CUs x workgroups per
// CU) takes
//     (alpha[epilogue] + beta K) * G(tiles),   G = full rounds + p + (1 - p) * (last round's fill),
// i.e. whole rounds of S tiles, a partly filled last round costing p of a round plus its share.
// The constants come from two fits.  The first is to launches of every kernel repeated on their own, operands in the caches
// (a quarter of a round to two rounds of tiles, K = 768 ... 5120; 7 - 9 % rms).  Inside a pass, where operands come from
// other caches and power is shared with what ran before, the order of kernels shifts, so they were fitted again, with
// the first fit as a prior of 4 %, to what a whole pass gains or loses when one product runs in another kernel (MI355X; 336
// row counts from 246 to 66000 at D = 768, 1024, 1280, every kernel within 22 % of the best by the first fit).  Only
// differences between kernels are fitted: the absolute figures are those of neither kind of launch.  Over these the picks
// take 0.30 % longer than the best kernel of each shape in the same pass, 0.42 % by the first fit; on row counts left out
// of the fit 0.31 and 0.32 against 0.41 and 0.43 (two halves).  At widths of 128 to 512, not fitted to: 2.3 against 2.9 %.
// Kernels 7 and 3 are priced as what they were fitted as, 64 x 64 and 128 x 128 tiles; pick_small_tile and wide_rows then take a faster
// tile of theirs where there is one, which the model does not know of: 3600 x 2304 x 768, 16.7 us in 160 x 128 tiles on its own, runs 160 x 256.
// The choice depends on the shape only, so a shape always runs the same kernel.  The K-step-32 kernel is nowhere the
// fastest where K is a multiple of 64, and not among the candidates.
static double rounds_cost(double tiles, int slots, double p) {
  const double full = std::floor(tiles / slots), frac = tiles / slots - full;
  return full + (frac > 0 ? p + (1.0 - p) * frac : 0.0);
}

// The 64 x 64 kernel: the chains of k-tiles of a CU's workgroups, which share its path to L2 and so take as long as one
// after the other, the fullest CU's being the launch's.  The slope is that of launches on their own (us at 1, 2, 3, 4
// workgroups per CU: K = 768 4.8, 6.4, 9.6, 11.5; K = 3072 + residual 11.1, 20.9, 31.0, 40.8).  Past that it does not hold: inside a
// pass 95749 x 1024 x 256 + GELU takes 54 us longer than in 256 x 256 tiles, which the slope prices the same.
constexpr int kTile64Most = 4 * 256;
static double tile64_cost(int64_t M, int N, int k_len, int splits, double per_tile, double alpha) {
  const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64) * splits;
  return alpha + (0.0031 * k_len + per_tile) * (double)((tiles + 255) / 256);
}

static int pick_mfma_kernel(int64_t M, int N, int K, int epi) {
  if (K % 64 != 0 || K < 128) return ((M + 63) / 64) * ((N + 63) / 64) <= 450 ? GK_64X64 : GK_128_K32;
  struct Cand { int id, bm, bn, slots; double alpha[3], beta, p; };
  static const Cand cands[] = {
      {GK_128_K64, 128, 128, 512, {3.53, 4.72, 9.08}, 0.0146, 0.572},
      {GK_160X256, 160, 256, 256, {3.46, 5.42, 10.5}, 0.0190, 0.536},
      {GK_192X256, 192, 256, 256, {4.19, 6.88, 12.2}, 0.0211, 0.469},
      {GK_224X256, 224, 256, 256, {5.03, 8.07, 14.9}, 0.0240, 0.434},
      {GK_256X256, 256, 256, 256, {5.84, 9.37, 17.0}, 0.0262, 0.414},
      {GK_288X256, 288, 256, 256, {7.44, 11.5, 21.7}, 0.0284, 0.464},
      {GK_320X256, 320, 256, 256, {8.34, 13.0, 24.3}, 0.0305, 0.448},
  };
  const int e = epi == EPI_RESIDUAL ? 2 : epi == EPI_GELU ? 1 : 0;
  static const double alpha64[3] = {2.38, 2.59, 1.58};
  const bool few = ((M + 63) / 64) * ((N + 63) / 64) <= kTile64Most;
  double best = few ? tile64_cost(M, N, K, 1, e == 2 ? 0.975 : 0.0, alpha64[e]) : 1e30;
  int kernel = GK_64X64;
  for (const Cand& c : cands) {
    const double tiles = (double)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    const double cost = (c.alpha[e] + c.beta * K) * rounds_cost(tiles, c.slots, c.p);
    if (cost < best) { best = cost; kernel = c.id; }
  }
  return kernel;
}

// Split-K for few-tile, long-K products (the MLP's second linear once merging has shrunk the
// batch): with M * N / 128^2 tiles below the 512 workgroups the chip holds, one workgroup per
// tile walks the whole K alone and the launch is bound by that serial chain.  S workgroups per tile
// each contract over K / S and write a float partial result; a second kernel adds the partial
// results in split order (a fixed order: results are reproducible), the bias and the residual, and
// applies the LayerNorm that follows -- so the split costs S + 1 more float passes over the
// output than the one-kernel form followed by its LayerNorm.  S never exceeds max_split.
//
// S sets the order in which a row's sums are added, hence the last bits of a pass and, where two merge candidates tie
// within them, its merge decisions.  It is therefore a rule of its own that does not follow the kernels: the constants
// below stay when a kernel or pick_mfma_kernel's model changes.  They were fitted to launches inside the encoder, whose
// operands come from HBM (residual form: one row per tile shape; partial products: launches of 704 ... 7488 rows at
// N = 768, K = 3072 with S = 2 ... 12, 9 % rms), the passes are priced at the rate the reduce kernel reaches there.  S taken
// from pick_mfma_kernel's stand-alone model instead (1 or 2 where this gives 6 from 400 to 1400 rows of N = 768) measured
// the same within 0.3 % on passes of 7 ... 128 queries and 1 % faster on one query with r = 16 (522.5 against 527.9 us).
static double residual_in_pass_us(int64_t M, int N, int K) {
  struct Shape { int bm, bn, slots; double alpha, beta, p; };   // as in pick_mfma_kernel
  static const Shape shapes[] = {{128, 128, 768, 13.0, 0.0278, 0.27}, {128, 128, 512, 8.75, 0.0161, 0.58},
                                 {192, 256, 256, 11.9, 0.0215, 0.72}, {256, 256, 256, 12.7, 0.0252, 0.72},
                                 {320, 256, 256, 14.7, 0.0284, 0.74}};
  double best = 1e30;
  for (const Shape& c : shapes) {
    const double tiles = (double)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    best = std::min(best, (c.alpha + c.beta * K) * rounds_cost(tiles, c.slots, c.p));
  }
  return best;
}

int splitk_factor(int dtype, int64_t M, int N, int K, int max_split) {
  if (dtype == 0 || K < 2048 || K % 64 != 0 || N % 8 != 0 || M <= 0) return 1;
  const double pass_us = (double)M * N * 4.0 / 6.0e6;   // one float pass over the output at 6 TB/s
  double best = residual_in_pass_us(M, N, K) + 1.5 * pass_us;   // + the LayerNorm pass: float in, 16-bit out
  int S = 1;
  const double tiles = (double)((M + 127) / 128) * ((N + 127) / 128);
  static const int cand[] = {2, 3, 4, 6, 8};
  for (int c : cand) {
    if (c > max_split || K % (c * 64) != 0 || K / c < 128) continue;
    const double cost = (6.5 + 0.0153 * (K / c)) * rounds_cost(tiles * c, 512, 0.556) + (c + 2.5) * pass_us;
    if (cost < best) { best = cost; S = c; }
  }
  return S;
}

// Which tiles the partial products of a split run in: the same bits either way.
static bool splitk_tiles64(int64_t M, int N, int K, int S) {
  const double tiles = (double)((M + 127) / 128) * ((N + 127) / 128);
  return tile64_cost(M, N, K / S, S, 0.9, 2.4) < (6.5 + 0.0130 * (K / S)) * rounds_cost(tiles * S, 512, 0.556);
}

hipError_t launch_linear_splitk(const void* x, const void* w, float* part, int64_t M, int N, int K, int S,
                                hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (S < 1 || K % (S * 64) != 0 || K / S < 128 || N % 8 != 0) return hipErrorInvalidValue;
  return splitk_tiles64(M, N, K, S) ? linear_mfma64(x, w, nullptr, nullptr, part, M, N, K, EPI_PARTIAL, s, nullptr, S)
                                    : linear_mfma128k64(x, w, nullptr, nullptr, part, M, N, K, EPI_PARTIAL, s, S);
}

hipError_t launch_linear(int dtype, const void* x, const void* w, const void* bias, const float* res, void* y,
                         int64_t M, int N, int K, int epi, hipStream_t s, int64_t model_bytes) {
  if (M <= 0) return hipSuccess;
  if (dtype == 0) return linear_f32<float>(x, w, bias, res, y, M, N, K, epi, s);
  if (K % 32 == 0 && K >= 64 && N % 8 == 0)
    return linear_mfma_kernel(pick_mfma_kernel(M, N, K, epi), x, w, bias, res, y, M, N, K, epi, s, nullptr, model_bytes);
  return linear_f32<bf16_t>(x, w, bias, res, y, M, N, K, epi, s);
}

// Whether the projection's launch has workgroup slots to spare for B list workgroups: they take a slot each (a
// launch's dynamic LDS is the same for all its workgroups), so beside a launch that fills its last round they would
// cost a round of their own (measured: + 5 us on such launches, what the selection-only plan saves beside attention).
bool linear_plan_tail_fits(int dtype, const void* x, const void* w, int64_t M, int N, int K, int B) {
  if (dtype == 0 && M > 0 && B > 0) {
    const bool dma = f32_dma_takes(x, w, K);
    if (f32_small_tiles(M, N, dma)) return true;   // at most three tiles per CU, room for eight (B = 4000 beside them still gains: 506 -> 403 us)
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
    return dma && tiles % 512 != 0 && tiles % 512 + B <= 512;
  }
  if (M <= 0 || B <= 0 || !(K % 32 == 0 && K >= 64 && N % 8 == 0)) return false;
  int bm = 128, bn = 128, slots = 768;
  switch (pick_mfma_kernel(M, N, K, EPI_RESIDUAL)) {
    case GK_128_K64: bm = wide_rows(M, N, K, 1); slots = 512; break;
    case GK_160X256: bm = 160; bn = 256; slots = 256; break;
    case GK_192X256: bm = 192; bn = 256; slots = 256; break;
    case GK_224X256: bm = 224; bn = 256; slots = 256; break;
    case GK_288X256: bm = 288; bn = 256; slots = 256; break;
    case GK_256X256: bm = 256; bn = 256; slots = 256; break;
    case GK_320X256: bm = 320; bn = 256; slots = 256; break;
    case GK_64X64: {
      const SmallShape sh = small_shape(pick_small_tile_with_lists(M, N, K, B));
      bm = sh.bm; bn = sh.bn; slots = K % 64 == 0 ? sh.slots : 1024;
      break;
    }
    default: break;
  }
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  return lists_fit(tiles, slots, B);
}

hipError_t launch_linear_plan_tail(int dtype, const void* x, const void* w, const void* bias, const float* res, void* y,
                                   int64_t M, int N, int K, const PlanTail& tail, int max_n, hipStream_t s) {
  if (M <= 0 || tail.B <= 0 || max_n > kPlanThreads || plan_lists_lds_bytes(max_n) > kPlanListsLdsMax)
    return hipErrorInvalidValue;
  if (dtype == 0) return linear_f32<float>(x, w, bias, res, y, M, N, K, EPI_RESIDUAL, s, &tail);
  if (!(K % 32 == 0 && K >= 64 && N % 8 == 0)) return hipErrorInvalidValue;
  return linear_mfma_kernel(pick_mfma_kernel(M, N, K, EPI_RESIDUAL), x, w, bias, res, y, M, N, K, EPI_RESIDUAL, s, &tail);
}

int linear_kernel_choice(int dtype, int64_t M, int N, int K, int epi) {
  if (dtype == 0) return GK_FMA;
  if (K % 32 == 0 && K >= 64 && N % 8 == 0) return pick_mfma_kernel(M, N, K, epi);
  return GK_FMA;
}

hipError_t launch_linear_kernel(int kernel, int dtype, const void* x, const void* w, const void* bias,
                                const float* res, void* y, int64_t M, int N, int K, int epi, hipStream_t s) {
  if (kernel == GK_AUTO) return launch_linear(dtype, x, w, bias, res, y, M, N, K, epi, s);
  if (M <= 0) return hipSuccess;
  if (kernel == GK_FMA)
    return dtype == 0 ? linear_f32<float>(x, w, bias, res, y, M, N, K, epi, s)
                      : linear_f32<bf16_t>(x, w, bias, res, y, M, N, K, epi, s);
  if (dtype == 0 || N % 8 != 0) return hipErrorInvalidValue;
  return linear_mfma_kernel(kernel, x, w, bias, res, y, M, N, K, epi, s);
}

}  // namespace otas
#undef OTAS_PLAN_TAIL_OR_TILE
