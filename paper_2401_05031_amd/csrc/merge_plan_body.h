// The plan of the merging module (Sec. II-C) for one query, as device functions that a workgroup executes:
//   merge_plan_select  phases 0-2: head-mean metric, unit length, every A token's most similar B token
//                      (NT threads, a multiple of 64: kPlanThreads on its own, fewer beside attention)
//   merge_plan_lists   phases 3-5: the r best edges, list slots, scans, the lists (any multiple of 64 threads)
//   merge_plan_body    both, one after the other
// Used by merge_plan_kernel (one workgroup per query runs the whole plan), by the kernel that runs the selection
// beside attention in one launch, and by the GEMM kernels that run the list phases beside the projection.
#ifndef OTAS_MERGE_PLAN_BODY_H_
#define OTAS_MERGE_PLAN_BODY_H_

#include <cfloat>
#include <type_traits>

#include "common.h"

namespace otas {

constexpr int kPlanThreads = 1024;

// What the plan needs to know of its query: first packed row and length entering the merge, first row leaving it,
// tokens to remove, first entry of its edges in the trace.
struct PlanQuery { int i0, n, o0, r_eff, tr0; };
__device__ inline PlanQuery plan_query(const int32_t* in_off, const int32_t* out_off, const int32_t* reff,
                                       const int32_t* troff, int q) {
  return PlanQuery{in_off[q], in_off[q + 1] - in_off[q], out_off[q], reff[q], troff[q]};
}

// LDS layout of the plan kernel (4-byte words), n = query length, nA = ceil(n/2), nB = floor(n/2):
//   mh [rows][dm+4] normalised metric rows (rows = n for the whole plan) | best [nA4] | kept [nA4] | bcol [nA] | cnt [nB] |
//   keep_pos [n] | ent_pos [n] | wave_tot [32] | part_v [512] | part_c [512],   nA4 = nA rounded up to 4
// (the list phases on their own use the part from best on, without part_v / part_c; the selection on its own
// mh | part_v | part_c).
// Floats per metric row in LDS: the even and the odd columns each padded to a multiple of 4, plus 4.
__host__ __device__ static inline int plan_row_floats(int dm) { return 2 * (((dm >> 1) + 3) & ~3) + 4; }
// Bytes of LDS the selection on its own needs, in na x nb workgroups per query.
static inline size_t plan_select_lds_bytes(int max_n, int dm, int na, int nb) {
  const int bA = ((max_n + 1) / 2 + 31) / 32, bB = (max_n / 2 + 31) / 32;
  const int rows = ((bA + na - 1) / na + (bB + nb - 1) / nb) * 32;
  return 4 * ((size_t)(rows < max_n ? rows : max_n) * plan_row_floats(dm) + 2 * 512);
}
// Workgroups per query for the selection.  First as many as it takes to keep a workgroup's metric rows within lds_goal
// bytes (what the launch's other workgroups need anyway: a launch's LDS is the same for all), then, while the launch has
// no more than 128 of them (half the CUs), as many as its A and B tokens have blocks to deal: what a workgroup loads and
// compares shrinks with both numbers, at the cost of loading A tokens nb times and B tokens na times in all.
// ViT-B pass on MI355X with one workgroup per query and with this rule: ten queries of 577 / 197 tokens 1642 and 1551 us
// (above 554 tokens the plan could not run beside attention at all), one query of 197 tokens 551 and 545, 64 of them,
// where the rule gives two, the same.
struct PlanParts { int a, b; };
static inline PlanParts plan_parts(int B, int max_n, int dm, size_t lds_goal) {
  const int bA = ((max_n + 1) / 2 + 31) / 32, bB = (max_n / 2 + 31) / 32;
  PlanParts p = {1, 1};
  auto grow = [&] {   // one more halving of the larger share
    const int ra = (bA + p.a - 1) / p.a, rb = (bB + p.b - 1) / p.b;
    if (ra <= 1 && rb <= 1) return false;
    (ra > rb ? p.a : p.b) *= 2;
    return true;
  };
  while (plan_select_lds_bytes(max_n, dm, p.a, p.b) > lds_goal && grow()) {}
  while (2 * p.a * p.b * B <= 128 && grow()) {}
  if (p.a > bA) p.a = bA;
  if (p.b > bB) p.b = bB;
  return p;
}
// Bytes of LDS the list phases need for a query of up to max_n tokens, and that for the longest query there is.
static inline size_t plan_lists_lds_bytes(int max_n) {
  const size_t nA = (max_n + 1) / 2, nB = max_n / 2;
  return 4 * (3 * nA + nB + 2 * (size_t)max_n + 32 + 8);
}
constexpr size_t kPlanListsLdsMax = 4 * (3 * 512 + 512 + 2 * 1024 + 32 + 8);

// One workgroup of NT threads per query (pq; tid = thread index in the workgroup; lds: its dynamic LDS).
// src: the vectors the similarity is taken on; the metric of token i is the mean over H heads of src[(i0 + i) * row_stride + col_off + h * dm + c] (H = 1 for
// a caller-supplied metric, H heads of the attention keys inside the encoder), normalised to unit
// length with fp32 arithmetic.
// ROWS_IN_LDS = false: the metric rows of the query live in global memory (rows + i0 * ldm: the
// query's own rows of a [T][ldm] float buffer; written and read by this workgroup only, between its
// barriers) instead of LDS, for queries whose rows do not fit the 160 KB; same arithmetic, same order.
// TO_GLOBAL = false: the result (best[a] = similarity of A token a's best match, -inf for a protected leading
// token; bcol[a] = that B token) stays in LDS behind the metric rows, valid for every thread after the next barrier.
// TO_GLOBAL = true: it goes to g_best[i0 + a], g_bcol[i0 + a] (a < nA) for merge_plan_lists in a later launch.
// Queries with nothing to merge return at once.
// pt: the A and the B tokens are dealt in blocks of 32 to pt.na x pt.nb workgroups (A block k goes to those with
// pt.a = k % pt.na, B block k to those with pt.b = k % pt.nb); this one computes the rows of its blocks and the best match
// of its A tokens among its B tokens only, so that loading the keys and comparing them is shared between CUs; with
// pt.nb > 1 the list phases take the best of the pt.nb candidates (g_best [pt.nb][pt.stride]).  More than one workgroup
// needs TO_GLOBAL.  Every row and every similarity is computed by the same arithmetic in the same order whatever pt is.
struct PlanPart { int a, na, b, nb; int64_t stride; };
template <typename T, bool ROWS_IN_LDS, bool TO_GLOBAL, int NT = kPlanThreads>
__device__ __forceinline__ void merge_plan_select(
    const T* __restrict__ src, int64_t row_stride, int col_off, int H, int dm, const PlanQuery& pq, int n_lead,
    float* rows, float* lds, float* __restrict__ g_best, int32_t* __restrict__ g_bcol, const int tid,
    const PlanPart pt = PlanPart{0, 1, 0, 1, 0}) {
  const int i0 = pq.i0, n = pq.n;
  if (n <= 0 || pq.r_eff <= 0) return;
  const int half = dm >> 1, hp = (half + 3) & ~3;   // columns per parity, and their padded count
  const int nA = (n + 1) >> 1, nB = n >> 1, ldm = 2 * hp + 4;
  const int nAb = (nA + 31) >> 5, nBb = (nB + 31) >> 5;
  const int nAl = (nAb - pt.a + pt.na - 1) / pt.na;   // A blocks of this workgroup: pt.a, pt.a + pt.na, ...
  const int nBl = (nBb - pt.b + pt.nb - 1) / pt.nb;   // and B blocks
  if (nAl <= 0 || nBl <= 0) {
    // nothing to compare: no candidate for the A tokens (if any) of this workgroup
    if constexpr (TO_GLOBAL)
      for (int t = tid; t < nAl * 32; t += NT) {
        const int a = (pt.a + pt.na * (t >> 5)) * 32 + (t & 31);
        if (a < nA) { g_best[pt.b * pt.stride + i0 + a] = -INFINITY; g_bcol[pt.b * pt.stride + i0 + a] = 0x7fffffff; }
      }
    return;
  }
  // The rows this workgroup needs, numbered u = 0 .. n_need - 1: its B tokens, then its A tokens, block by block (only
  // a query's last block can be short, and it is the last of the workgroup that owns it).
  const int nBv = nBl * 32 - ((pt.b + pt.nb * (nBl - 1) == nBb - 1) ? nBb * 32 - nB : 0);
  const int nAv = nAl * 32 - ((pt.a + pt.na * (nAl - 1) == nAb - 1) ? nAb * 32 - nA : 0);
  const int n_need = nBv + nAv;
  auto token_of = [&](int u) {
    if (u < nBv) return 2 * ((pt.b + pt.nb * (u >> 5)) * 32 + (u & 31)) + 1;
    const int v = u - nBv;
    return 2 * ((pt.a + pt.na * (v >> 5)) * 32 + (v & 31));
  };
  // Metric rows in that order, ldm = dm + 4 floats apart (16 lanes
  // reading 16 bytes each from 16 consecutive rows then fall on all 64 banks once).  Inside a row the
  // columns are stored even ones first, then odd ones (each group zero-padded to a multiple of 4):
  // column c sits at (c & 1) * hp + c / 2, so
  // the two halves of a wave (which feed the even and the odd k of every fp32 MFMA) each read
  // consecutive floats.
  float* mh = ROWS_IN_LDS ? lds : rows + (size_t)i0 * ldm;
  float* best = ROWS_IN_LDS ? lds + (size_t)n * ldm : lds;   // TO_GLOBAL = false: one workgroup has all n rows
  int* bcol = (int*)(best + 2 * ((nA + 3) & ~3));   // behind kept of the list phases
  int* part_c = TO_GLOBAL ? (int*)(ROWS_IN_LDS ? lds + (size_t)n_need * ldm : lds)
                          : bcol + nA + nB + 2 * n + 32;   // behind cnt, keep_pos, ent_pos, wave_tot of the list phases
  float* part_v = reinterpret_cast<float*>(part_c + 512);

  // Phase 0: head-mean metric rows, heads summed in ascending order.  A thread takes 8 columns of a token when the
  // source is 16-bit and 16-byte aligned with dm % 8 == 0 (one 16-byte load per head, two 16-byte LDS stores: this phase is bound by
  // instruction issue on the one CU that runs the query), else 4 columns.
  const float inv_h = 1.0f / (float)H;
  if (sizeof(T) == 2 && (dm & 7) == 0 && (row_stride & 7) == 0 && (col_off & 7) == 0 &&
      (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
    const int c8n = dm >> 3;
    for (int t = tid; t < n_need * c8n; t += NT) {
      const int u = t / c8n, c = (t - u * c8n) * 8;
      const T* p = src + (size_t)(i0 + token_of(u)) * row_stride + col_off + c;
      float m[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) m[e] = 0.f;
      auto heads = [&](auto UH) {   // UH heads in flight together (loads past the last head repeat it)
        for (int h0 = 0; h0 < H; h0 += UH.value) {
          Oct<T> v[UH.value];
#pragma unroll
          for (int j = 0; j < UH.value; ++j) v[j] = *reinterpret_cast<const Oct<T>*>(p + (size_t)min(h0 + j, H - 1) * dm);
#pragma unroll
          for (int j = 0; j < UH.value; ++j)
            if (h0 + j < H) {
#pragma unroll
              for (int e = 0; e < 8; ++e) m[e] += to_float(v[j].x[e]);
            }
        }
      };
      if (H == 1) heads(std::integral_constant<int, 1>{});   // the caller's own metric
      // Any other number 12 at a time (48 registers).  Even groups of at most 16, picked by H, measured the same with 12
      // and with 16 heads (ViT-B batch of 64 1957 and 1960 us, ViT-L of 128 9492 and 9502) and cost the caller's own
      // metric 1.4 % (24.4 -> 24.8 us): 16 heads' second trip, eight of its loads repeats, is hidden.
      else heads(std::integral_constant<int, 12>{});
      float* r = mh + (size_t)u * ldm;
      const int ce = c >> 1;   // columns c, c+2, c+4, c+6 are even ones, the others odd ones
      *reinterpret_cast<floatx4*>(r + ce) = floatx4{m[0] * inv_h, m[2] * inv_h, m[4] * inv_h, m[6] * inv_h};
      *reinterpret_cast<floatx4*>(r + hp + ce) = floatx4{m[1] * inv_h, m[3] * inv_h, m[5] * inv_h, m[7] * inv_h};
    }
  } else {
    const int c4n = dm >> 2;
    for (int t = tid; t < n_need * c4n; t += NT) {
      const int u = t / c4n, c = (t - u * c4n) * 4;
      const T* p = src + (size_t)(i0 + token_of(u)) * row_stride + col_off + c;
      float m0 = 0.f, m1 = 0.f, m2 = 0.f, m3 = 0.f;
#pragma unroll 4
      for (int h = 0; h < H; ++h) {
        const Quad<T> v = *reinterpret_cast<const Quad<T>*>(p);
        m0 += to_float(v.x[0]); m1 += to_float(v.x[1]); m2 += to_float(v.x[2]); m3 += to_float(v.x[3]);
        p += dm;
      }
      float* r = mh + (size_t)u * ldm;
      const int ce = c >> 1;   // columns c, c+2 are even ones, c+1, c+3 odd ones
      r[ce] = m0 * inv_h;
      r[ce + 1] = m2 * inv_h;
      r[hp + ce] = m1 * inv_h;
      r[hp + ce + 1] = m3 * inv_h;
    }
  }
  if (hp != half)   // the padding columns take part in the contraction: zero
    for (int t = tid; t < n_need * 2 * (hp - half); t += NT) {
      const int u = t / (2 * (hp - half)), c = t - u * (2 * (hp - half));
      mh[(size_t)u * ldm + (c & 1) * hp + half + (c >> 1)] = 0.f;
    }
  __syncthreads();
  // Phase 1: unit length.  16 consecutive lanes share a row of 2 hp floats (the zero padding adds nothing): lane j
  // sums the squares of the 16-byte pieces j, j + 16, ... in ascending order, the sixteen partial sums are added by
  // a fixed butterfly, and every lane scales its own pieces.
  {
    const int q4 = (2 * hp) >> 2;   // 16-byte pieces per row
    for (int u0 = 0; u0 < n_need; u0 += NT / 16) {
      const int u = u0 + (tid >> 4), j = tid & 15;
      float* r = mh + (size_t)min(u, n_need - 1) * ldm;
      float ss = 0.f;
      for (int m = j; m < q4; m += 16) {
        const floatx4 v = *reinterpret_cast<const floatx4*>(r + 4 * m);
        ss = fmaf(v[0], v[0], ss); ss = fmaf(v[1], v[1], ss); ss = fmaf(v[2], v[2], ss); ss = fmaf(v[3], v[3], ss);
      }
      ss = dpp_sum<kDppXor2>(dpp_sum<kDppXor1>(ss));
      ss = dpp_sum<kDppHalfMirror>(ss);   // the lanes of a quad agree by now: the mirrored lane holds the other quad's sum
      ss = dpp_sum<dpp_ror(8)>(ss);
      const float rn = 1.0f / fmaxf(sqrtf(ss), 1e-12f);
      if (u < n_need)
        for (int m = j; m < q4; m += 16) {
          floatx4 v = *reinterpret_cast<const floatx4*>(r + 4 * m);
          v[0] *= rn; v[1] *= rn; v[2] *= rn; v[3] *= rn;
          *reinterpret_cast<floatx4*>(r + 4 * m) = v;
        }
    }
  }
  __syncthreads();

  // Phase 2: every A token picks its most similar B token.  The similarity matrix is a dense
  // contraction over the metric width, done on the matrix cores in true fp32
  // (v_mfma_f32_32x32x2_f32), transposed: B tokens are the first operand (rows), A tokens the second
  // (columns), so a lane owns ONE A token and holds 16 of a 32-token B block's similarities in its
  // accumulator (rows 8 (e / 4) + 4 (lane >> 5) + (e & 3)): its arg-max is a scan of its own registers
  // in ascending B order plus one exchange with lane ^ 32.  Wave w owns the workgroup's A block w % nAl and every
  // G-th of its B blocks; the G partial results per A token are combined through LDS.  Ties go to the
  // lowest B position at every step.
  // With few blocks for the waves (a small batch's workgroup has one of either kind) they are cut into tiles of 16 x 16, so that one
  // wave's chain of 32 MFMAs of 64 clocks becomes one of 16 of 32 clocks in each of four waves.  Either instruction adds the
  // products of its columns one after the other, in ascending order, so the similarities are the same bits.  16 x 16 tiles
  // take twice the operand reads, so only where there is a wave for each (four blocks in eight waves: otas_token_merge of one query of
  // 197 tokens 14.7 -> 15.1 us).  ViT-B passes of 1 / 4 / 8 / 16 queries of 197 tokens with r = 16 451 / 563 / 690 / 922 -> 443 / 557 / 687 / 918
  // us, of 101 with r = 8 419 / 485 / 553 / 687 -> 409 / 480 / 548 / 679; ViT-L, four of 197 with r = 8, 1378 -> 1362.
  constexpr int NWV = NT / 64;
  const bool fine = NT < kPlanThreads && 4 * nAl * nBl <= NWV;
  const int nAs = (nAv + 15) >> 4, nBs = (nBv + 15) >> 4;
  const int G = max(1, NWV / (fine ? nAs : nAl)), part_rows = fine ? nAs * 16 : nAl * 32;
  if (fine) {
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fk = lane >> 4;   // accumulator: A token fr, B tokens 4 fk .. + 3 of the tile
    const int al = w % nAs, grp = w / nAs;      // nAs <= NWV
    if (grp < G) {
      // lane group fk feeds column 4 u + fk to MFMA u: every second float of the even or the odd columns
      const float* pa = mh + (size_t)(nBv + min(al * 16 + fr, nAv - 1)) * ldm + (fk & 1) * hp + (fk >> 1);
      float bv = -FLT_MAX;   // as below
      int bc = 0;
      for (int bl = grp; bl < nBs; bl += G) {
        const float* pb = mh + (size_t)min(bl * 16 + fr, nBv - 1) * ldm + (fk & 1) * hp + (fk >> 1);
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < hp; k0 += 16) {   // 8 MFMAs per batch, their operand reads issued first (hp % 4 == 0)
          float ra[8], rb[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int k = k0 + 2 * (u & ~1) < hp ? k0 + 2 * u : 0;
            ra[u] = pa[k];
            rb[u] = pb[k];
          }
#pragma unroll
          for (int u = 0; u < 8; u += 2)
            if (k0 + 2 * u < hp) {
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rb[u], ra[u], acc, 0, 0, 0);
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rb[u + 1], ra[u + 1], acc, 0, 0, 0);
            }
        }
        const int b0 = (pt.b + pt.nb * (bl >> 1)) * 32 + 16 * (bl & 1) + 4 * fk;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (b0 + e < nB && acc[e] > bv) { bv = acc[e]; bc = b0 + e; }
      }
      auto take = [&](float ov, int oc) { if (ov > bv || (ov == bv && oc < bc)) { bv = ov; bc = oc; } };
      take(__shfl_xor(bv, 16, kWave), __shfl_xor(bc, 16, kWave));
      take(wave_halves(bv).hi, __float_as_int(wave_halves(__int_as_float(bc)).hi));   // the first 16 lanes decide
      if (fk == 0) {
        part_v[grp * part_rows + al * 16 + fr] = bv;
        part_c[grp * part_rows + al * 16 + fr] = bc;
      }
    }
  } else {
    const int lane = tid & 63, w = tid >> 6;
    const int fr = lane & 31, fk = lane >> 5;
    // nAl <= NWV: one (A block, B group) per wave, groups beyond G idle; more A blocks than waves: one group, the
    // waves take the blocks in turn
    const bool wide = nAl > NWV;
    const int grp = wide ? 0 : w / nAl;
    for (int al = wide ? w : w % nAl; al < nAl && grp < G; al += wide ? NWV : nAl) {
      const float* pa = mh + (size_t)(nBv + min(al * 32 + fr, nAv - 1)) * ldm + fk * hp;
      // An A token that compares with no B token (NaN in its metric, or in all of theirs) goes to B token 0, behind every
      // other and before a protected one: the list phases index with its choice.
      float bv = -FLT_MAX;
      int bc = 0;
      for (int bl = grp; bl < nBl; bl += G) {
        const float* pb = mh + (size_t)min(bl * 32 + fr, nBv - 1) * ldm + fk * hp;
        floatx16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
        // MFMA u contracts over columns 2u (lanes 0..31) and 2u + 1 (lanes 32..63): with the even /
        // odd column split a lane's operands of four consecutive MFMAs are one 16-byte read
        for (int k0 = 0; k0 < hp; k0 += 8) {   // 8 MFMAs per batch, their operand reads issued first
          const floatx4 ra0 = *reinterpret_cast<const floatx4*>(pa + k0);
          const floatx4 rb0 = *reinterpret_cast<const floatx4*>(pb + k0);
          floatx4 ra1 = ra0, rb1 = rb0;
          if (k0 + 4 < hp) {
            ra1 = *reinterpret_cast<const floatx4*>(pa + k0 + 4);
            rb1 = *reinterpret_cast<const floatx4*>(pb + k0 + 4);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(rb0[u], ra0[u], acc, 0, 0, 0);
          if (k0 + 4 < hp) {
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(rb1[u], ra1[u], acc, 0, 0, 0);
          }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int b = (pt.b + pt.nb * bl) * 32 + 8 * (e >> 2) + 4 * fk + (e & 3);
          if (b < nB && acc[e] > bv) { bv = acc[e]; bc = b; }
        }
      }
      const float ov = wave_halves(bv).hi;   // the lower half's lanes (fk == 0) decide
      const int oc = __float_as_int(wave_halves(__int_as_float(bc)).hi);
      if (ov > bv || (ov == bv && oc < bc)) { bv = ov; bc = oc; }
      if (fk == 0) {
        part_v[grp * part_rows + al * 32 + fr] = bv;
        part_c[grp * part_rows + al * 32 + fr] = bc;
      }
    }
  }
  __syncthreads();
  for (int t = tid; t < nAv; t += NT) {
    const int a = (pt.a + pt.na * (t >> 5)) * 32 + (t & 31);
    float bv = part_v[t];
    int bc = part_c[t];
    for (int g = 1; g < G; ++g) {
      const float v = part_v[g * part_rows + t];
      const int c = part_c[g * part_rows + t];
      if (v > bv || (v == bv && c < bc)) { bv = v; bc = c; }
    }
    const float v = (2 * a < n_lead) ? -INFINITY : bv;   // protected leading token: never a merge source
    if constexpr (TO_GLOBAL) {
      g_best[pt.b * pt.stride + i0 + a] = v;
      g_bcol[pt.b * pt.stride + i0 + a] = bc;
    } else {
      best[a] = v;
      bcol[a] = bc;
    }
  }
  // (TO_GLOBAL = false: best and bcol are visible after the barrier that merge_plan_lists begins with)
}

// The list phases for a query by a workgroup of NT threads (a multiple of 64, at most 1024).  small: LDS for
// best [nA4] | kept [nA4] | bcol [nA] | cnt [nB] | keep_pos [n] | ent_pos [n] | wave_tot [32] (4-byte words), 16-byte aligned.
// FROM_GLOBAL = false: best / bcol are already there (merge_plan_select in the same workgroup);
// true: they are read from g_best / g_bcol [nb][stride], entry i0 + a: the best of nb candidates, ties to the lowest B
// token.  Integer work only, apart from comparisons of the
// similarities: the result does not depend on NT.
template <int NT, bool FROM_GLOBAL>
__device__ __forceinline__ void merge_plan_lists(
    float* small, const float* __restrict__ g_best, const int32_t* __restrict__ g_bcol, int nb, int64_t stride,
    const PlanQuery& pq, int32_t* __restrict__ src_list, int32_t* __restrict__ row_ptr, int32_t* __restrict__ trace_src,
    int32_t* __restrict__ trace_dst, const int tid) {
  const int i0 = pq.i0, n = pq.n, o0 = pq.o0, r_eff = pq.r_eff;
  if (n <= 0) return;
  if (r_eff <= 0) {  // nothing merges: every output row is its own single source
    for (int i = tid; i < n; i += NT) {
      row_ptr[o0 + i] = i0 + i;
      src_list[i0 + i] = i0 + i;
    }
    return;
  }
  const int nA = (n + 1) >> 1, nB = n >> 1, nA4 = (nA + 3) & ~3;
  float* best = small;
  int* kept = (int*)(best + nA4);   // destination of a kept edge (from its slot's count on: + slot << 16), -1: survives
  int* bcol = kept + nA4;
  int* cnt = bcol + nA;
  int* keep_pos = cnt + nB;      // [n] exclusive scan of "row survives"
  int* ent_pos = keep_pos + n;   // [n] exclusive scan of list lengths
  int* wave_tot = ent_pos + n;   // [16]
  int* rank = keep_pos;          // until phase 4
  int* edge = (int*)best;        // from the end of the ranking on: the kept edges by rank, destination << 16 | source
  if constexpr (FROM_GLOBAL) {
    // All candidates of an A token are requested before the first is compared: written on other CUs a launch earlier, each
    // is a round trip beyond the XCD's L2, and one after the other they were the longest part of the lists.
    constexpr int NC = 4;
    for (int a = tid; a < nA; a += NT) {
      float v = -INFINITY;
      int c = 0x7fffffff;
      for (int p0 = 0; p0 < nb; p0 += NC) {
        float u[NC];
        int d[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {   // past the last candidate: that one again
          const int64_t at = min(p0 + j, nb - 1) * stride + i0 + a;
          u[j] = g_best[at];
          d[j] = g_bcol[at];
        }
#pragma unroll
        for (int j = 0; j < NC; ++j)
          if (u[j] > v || (u[j] == v && d[j] < c)) { v = u[j]; c = d[j]; }
      }
      best[a] = v;
      bcol[a] = c;
    }
  }
  if (tid < nA4 - nA) best[nA + tid] = -INFINITY;   // ranks behind every token it could be compared with
  for (int a = tid; a < nA; a += NT) rank[a] = 0;
  for (int b = tid; b < nB; b += NT) cnt[b] = 0;
  __syncthreads();

  // Phase 3: keep the r_eff best edges.  rank = number of A tokens that come before this one in
  // (similarity descending, position ascending) order: a count over all A tokens.  A
  // thread takes one A token and one part of the tokens it is compared with (the same for its whole wave: they are
  // read four at a time, every lane the same address), the parts are added by LDS atomics on integers.  The phase is
  // bound by the number of LDS reads a wave waits for: with eight lanes per A token, each reading every eighth token on
  // its own, a ViT-B pass over ten queries of 577 / 197 tokens took 1700 us, one query of 197 tokens 559; now 1642, 551.
  const int nAp = (nA + 63) & ~63;                 // whole waves
  const int parts = max(1, NT / nAp), part = __builtin_amdgcn_readfirstlane(tid / nAp);   // the same for a whole wave
  const int chunk = ((nA + parts - 1) / parts + 3) & ~3;
  const int k_beg = part * chunk, k_end = min(nA4, k_beg + chunk);
  if (part < parts)
    for (int a = tid - part * nAp; a < nA; a += NT) {   // a second round only when nAp > NT: one part then
      const float v = best[a];
      // this wave's A tokens are a0 .. a0 + 63: ties only have to be looked at among those
      const int a0 = __builtin_amdgcn_readfirstlane(a) & ~63;
      const int k_lo = min(max(a0, k_beg), k_end), k_hi = min(max(a0 + 64, k_beg), k_end);
      int c = 0;
#pragma unroll 4
      for (int k = k_beg; k < k_lo; k += 4) {
        const floatx4 u = *reinterpret_cast<const floatx4*>(best + k);
#pragma unroll
        for (int j = 0; j < 4; ++j) c += u[j] >= v ? 1 : 0;
      }
#pragma unroll 4
      for (int k = k_lo; k < k_hi; k += 4) {
        const floatx4 u = *reinterpret_cast<const floatx4*>(best + k);
#pragma unroll
        for (int j = 0; j < 4; ++j) c += (u[j] > v || (u[j] == v && k + j < a)) ? 1 : 0;
      }
#pragma unroll 4
      for (int k = k_hi; k < k_end; k += 4) {
        const floatx4 u = *reinterpret_cast<const floatx4*>(best + k);
#pragma unroll
        for (int j = 0; j < 4; ++j) c += u[j] > v ? 1 : 0;
      }
      if (parts > 1) atomicAdd(&rank[a], c);
      else rank[a] = c;
    }
  __syncthreads();
  for (int a = tid; a < nA; a += NT) {
    const int k = rank[a], dst = bcol[a];
    const bool keep = k < r_eff;
    if (!keep) kept[a] = -1;
    else {
      edge[k] = dst << 16 | a;
      if (trace_src) {
        trace_src[pq.tr0 + k] = 2 * a;
        trace_dst[pq.tr0 + k] = 2 * dst + 1;
      }
    }
  }
  if (tid < (-r_eff & 3)) edge[r_eff + tid] = 0x7fffffff;   // counts as nobody's neighbour below; r_eff <= nA
  __syncthreads();
  // slot = number of kept edges with the same destination and a lower source position (the order of a destination's
  // source list): counted among the r_eff kept edges, a few dozen of the hundreds of A tokens.
  for (int i = tid; i < r_eff; i += NT) {
    const int me = edge[i], a = me & 0xffff, dst = me >> 16, lo = dst << 16;
    int c = 0;
#pragma unroll 4
    for (int k = 0; k < r_eff; k += 4) {
      const int4 u = *reinterpret_cast<const int4*>(edge + k);
      c += ((unsigned)(u.x - lo) < (unsigned)a) + ((unsigned)(u.y - lo) < (unsigned)a) +
           ((unsigned)(u.z - lo) < (unsigned)a) + ((unsigned)(u.w - lo) < (unsigned)a);
    }
    kept[a] = dst | c << 16;
    atomicAdd(&cnt[dst], 1);   // an integer count: the result does not depend on the order
  }
  __syncthreads();

  // Phase 4: positions.  keep(i) = 1 unless i is a merged A token; entries(i) = keep(i) * (1 +
  // number of sources merged into i).  Exclusive scans of both over i = 0..n-1, in the two halves of a word (both totals
  // are at most n <= 1024): every thread takes ceil(n / NT) consecutive positions (one when n <= NT), wave scan of the
  // thread sums by shuffles, then the wave totals.
  {
    const int C = (n + NT - 1) / NT;
    const int lane = tid & 63, w = tid >> 6;
    auto counts_of = [&](int i) {   // entries << 16 | keep
      if (i & 1) return (1 + cnt[i >> 1]) << 16 | 1;
      return kept[i >> 1] >= 0 ? 0 : 1 << 16 | 1;
    };
    int sum = 0;
    for (int c = 0; c < C; ++c) {
      const int i = tid * C + c;
      if (i < n) sum += counts_of(i);
    }
    int scan = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(scan, o, kWave);
      if (lane >= o) scan += t;
    }
    if (lane == 63) wave_tot[w] = scan;
    __syncthreads();
    int pos = scan - sum;
    for (int j = 0; j < w; ++j) pos += wave_tot[j];
    for (int c = 0; c < C; ++c) {
      const int i = tid * C + c;
      if (i < n) {
        keep_pos[i] = pos & 0xffff;
        ent_pos[i] = pos >> 16;
        pos += counts_of(i);
      }
    }
  }
  __syncthreads();

  // Phase 5: write the lists: every surviving row opens its list with itself, every merged A token
  // enters its destination's list at its slot.
  for (int i = tid; i < n; i += NT) {
    const bool odd = i & 1;
    if (!odd && kept[i >> 1] >= 0) {
      const int k = kept[i >> 1], d = 2 * (k & 0xffff) + 1;
      src_list[i0 + ent_pos[d] + 1 + (k >> 16)] = i0 + i;
    } else {
      const int e = i0 + ent_pos[i];
      row_ptr[o0 + keep_pos[i]] = e;
      src_list[e] = i0 + i;
    }
  }
}

// The whole plan of a query by one workgroup of NT threads (a multiple of 64; tid = thread index; lds: its dynamic LDS).
template <typename T, bool ROWS_IN_LDS, int NT = kPlanThreads>
__device__ __forceinline__ void merge_plan_body(
    const T* __restrict__ src, int64_t row_stride, int col_off, int H, int dm, const PlanQuery& pq, int n_lead,
    int32_t* __restrict__ src_list, int32_t* __restrict__ row_ptr, int32_t* __restrict__ trace_src,
    int32_t* __restrict__ trace_dst, float* rows, float* lds, const int tid) {
  merge_plan_select<T, ROWS_IN_LDS, false, NT>(src, row_stride, col_off, H, dm, pq, n_lead, rows, lds, nullptr, nullptr,
                                               tid);
  float* small = ROWS_IN_LDS ? lds + (size_t)max(pq.n, 0) * plan_row_floats(dm) : lds;
  merge_plan_lists<NT, false>(small, nullptr, nullptr, 1, 0, pq, src_list, row_ptr, trace_src, trace_dst, tid);
}

}  // namespace otas
#endif  // OTAS_MERGE_PLAN_BODY_H_
