// select.hip - the top-k selection of the forward (Eq. top-k), fused with the
// landmark-key score pass so that the M x N score matrix is never stored.
//
//   1-2. the sampled scores and pivots (sample.hpp; in the forward's one-expert
//      path beside the routing logits, pivots_logits_kernel): the scores of
//      every landmark against ns evenly spaced keys, as order-preserving keys
//      (the same tile arithmetic as the score pass, so the same values); per
//      landmark row, the pivot = the r-th largest sampled key. r is chosen on
//      the host so that at least k and far fewer than `cap` tokens of the row
//      score >= pivot, except with negligible probability (r = k exactly when
//      the sample is the whole row).
//   3. the score pass lists every token scoring >= pivot (bits of its
//      unscaled dot, token index), in token order, in one region per (row,
//      key chunk); the finish scales the dots as every score is scaled.
//   4. finalize_kernel: with k <= count <= cap the list holds the row's whole
//      top-k, since every token left out scores below the pivot, which the
//      k-th listed score reaches. The row's regions are packed into LDS, the
//      k-th largest key is found exactly, and an ordered scan writes the
//      tokens above it and the first ones equal to it, as many as the set still
//      needs; the list is already in ascending token order. A row whose count
//      is out of range goes to a fallback list. Where the routing came first,
//      rows of experts without queries are only counted, not stored or
//      selected: nothing reads their sets.
//   5. fallback rows: the row is scored in full with the score pass's products
//      (score_row in the forward's placement launch; scores_rows_kernel with the
//      staged gather) and the exact top-k selects from it.
// The sets equal those of the exact top-k over the stored score rows.
#include "cdna4.hpp"
#include "flash.hpp"
#include "kernels.hpp"
#include "check.hpp"
#include "finalize.hpp"
#include "sample.hpp"
#include "worklist.hpp"

#include <type_traits>

namespace mita {

// waves per workgroup of pivots16_body without the logits (fp32: its registers)
template <typename T> constexpr int PIVOT16_WAVES = sizeof(T) == 2 ? 16 : 8;

// One workgroup per (16 landmarks, head) slot (ROWS 0: pivots16_body) or (ROWS
// landmarks, head) slot, with the sets if the sample is the whole row (SETS);
// slots spread over the XCDs in contiguous ranges (xcd_slot): a head's landmark
// blocks share an XCD, so its sampled key rows are fetched into one L2 instead
// of one per block.
template <typename T, int D, int ROWS, bool SETS>
__global__ __launch_bounds__(ROWS ? 64 * ROWS : 64 * PIVOT16_WAVES<T>) void sample_pivot_kernel(
    const T *__restrict__ q_lm, const T *__restrict__ k, uint32_t *__restrict__ plo, uint32_t *__restrict__ fail_cnt,
    int N, int M, int r, float scale, int nbx, int nslots, int32_t *__restrict__ idx) {
  static_assert(ROWS != 0 || !SETS, "sets come from rows of keys");
  __shared__ __align__(16) std::conditional_t<ROWS != 0, uint32_t[ROWS ? ROWS : 1][SP_PITCH], PivotLds> sh;
  const int f = xcd_slot((int)blockIdx.x, (int)gridDim.x / NXCD);
  if (f >= nslots) return;  // the whole workgroup
  if constexpr (ROWS != 0)
    sample_pivot_body<T, D, SETS, ROWS>(sh, f % nbx, f / nbx, q_lm, k, plo, fail_cnt, N, M, SETS ? N : SEL_NS, r, scale,
                                        idx, r);
  else
    pivots16_body<T, D, PIVOT16_WAVES<T>>(sh, f % nbx, f / nbx, q_lm, k, plo, fail_cnt, N, M, r, scale);
}

template <typename T, int D, int CAP, bool MERGE>
__global__ __launch_bounds__(256) void finalize_kernel(const uint2 *__restrict__ cand,
                                                       const uint32_t *__restrict__ ccnt, int32_t *__restrict__ idx,
                                                       uint32_t *__restrict__ fail_cnt,
                                                       int32_t *__restrict__ fail_list, int k, int cap, int nch,
                                                       const float2 *__restrict__ part_ml,
                                                       const float *__restrict__ part_o, T *__restrict__ v_lm, int M,
                                                       float scale, LiveRows live) {
  __shared__ FinalizeLds<T, D, CAP, MERGE> sh;
  finalize_row<T, D, CAP, MERGE>(sh, blockIdx.x, cand, ccnt, idx, fail_cnt, fail_list, k, cap, nch, part_ml, part_o,
                                 v_lm, M, scale, live);
}

// The same with one wave per row (lists of at most SEL_NS, at most 64 chunks).
template <typename T, int D, bool MERGE>
__global__ __launch_bounds__(256) void finalize_wave_kernel(const uint2 *__restrict__ cand,
                                                            const uint32_t *__restrict__ ccnt,
                                                            int32_t *__restrict__ idx, uint32_t *__restrict__ fail_cnt,
                                                            int32_t *__restrict__ fail_list, int k, int cap, int nch,
                                                            const float2 *__restrict__ part_ml,
                                                            const float *__restrict__ part_o, T *__restrict__ v_lm,
                                                            int M, float scale, int64_t nrows, LiveRows live) {
  __shared__ FinalizeWaveLds sh[4];
  const int w = (int)threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= nrows) return;  // the whole wave
  finalize_row_wave<T, D, MERGE>(sh[w], row, cand, ccnt, idx, fail_cnt, fail_list, k, cap, nch, part_ml, part_o,
                                 v_lm, M, scale, live);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T, int D>
static hipError_t sample_pivot_t(const mita_cfg_t &c, const void *q_lm, const void *k, const SelectBufs &sb,
                                 hipStream_t st) {
  constexpr int MANY = sizeof(T) == 2 ? 16 : 8;  // rows per workgroup (fp32 fragments need eight waves' registers)
#define MITA_PIVOTS(ROWS, PER, SETS)                                                                                \
  {                                                                                                                 \
    const int nbx = (c.M + PER - 1) / PER, nslots = nbx * (int)BH(c);                                               \
    hipLaunchKernelGGL((sample_pivot_kernel<T, D, ROWS, SETS>), dim3((unsigned)(NXCD * ((nslots + NXCD - 1) / NXCD))), \
                       dim3(64 * (ROWS ? ROWS : PIVOT16_WAVES<T>)), 0, st, (const T *)q_lm, (const T *)k, sb.plo, sb.fail_cnt, c.N, \
                       c.M, sb.rank, eff_scale(c), nbx, nslots, sb.idx);                                            \
  }
  if (!sb.idx) {
    if (few_pivots(c))
      MITA_PIVOTS(SP_ROWS, SP_ROWS, false)
    else
      MITA_PIVOTS(0, 16, false)
  } else if (few_rows(c)) {
    MITA_PIVOTS(SP_ROWS, SP_ROWS, true)
  } else {
    MITA_PIVOTS(MANY, MANY, true)
  }
#undef MITA_PIVOTS
  return launched("sample_pivot_kernel", st);
}

hipError_t launch_select_pivots(const mita_cfg_t &c, const void *q_lm, const void *k, const SelectBufs &sb,
                                hipStream_t st) {
  // sets from the whole row, or pivots of SEL_NS samples
  if (sb.idx ? sb.ns != c.N || sb.ns > SEL_NS || sb.rank != c.k : sb.ns != SEL_NS) return hipErrorInvalidValue;
  if (c.dtype == MITA_F32)
    return c.d == 64 ? sample_pivot_t<float, 64>(c, q_lm, k, sb, st) : sample_pivot_t<float, 128>(c, q_lm, k, sb, st);
  return c.d == 64 ? sample_pivot_t<bf16_t, 64>(c, q_lm, k, sb, st) : sample_pivot_t<bf16_t, 128>(c, q_lm, k, sb, st);
}

// The finalize kernel alone (a workgroup or a wave per landmark row).
hipError_t launch_select_finalize(const mita_cfg_t &c, const SelectBufs &sb, int32_t *idx, const void *partial,
                                  void *v_lm, hipStream_t st) {
  const unsigned rows = (unsigned)(BH(c) * c.M);
  const int nch = score_chunks(c);
  const float2 *ml = (const float2 *)partial;
  const float *po = v_lm ? (const float *)((const char *)partial + align_up((size_t)BH(c) * nch * c.M * sizeof(float2)))
                         : nullptr;
#define MITA_FINALIZE(TT, DD, CAP, MG)                                                                          \
  hipLaunchKernelGGL((finalize_kernel<TT, DD, CAP, MG>), dim3(rows), dim3(256), 0, st, sb.cand, sb.ccnt, idx,   \
                     sb.fail_cnt, sb.fail_list, c.k, sb.cap, nch, ml, po, (TT *)v_lm, c.M, eff_scale(c), live)
#define MITA_FINALIZE_WAVE(TT, DD, MG)                                                                          \
  hipLaunchKernelGGL((finalize_wave_kernel<TT, DD, MG>), dim3((rows + 3) / 4), dim3(256), 0, st, sb.cand, sb.ccnt, \
                     idx, sb.fail_cnt, sb.fail_list, c.k, sb.cap, nch, ml, po, (TT *)v_lm, c.M, eff_scale(c),      \
                     (int64_t)rows, live)
  const LiveRows live{sb.live, sb.live_groups};
  // Lists of at most SEL_NS entries over at most 64 chunks: one wave per row,
  // unless there are so few rows that a workgroup per row is resident at once and
  // its shorter chain counts (us with a wave and with a workgroup, d = 64: 4096
  // tokens 11.8 and 10.2 at 256 rows, 14.6 and 12.0 at 1536, 14.8 and 16.3 at 2048;
  // 8192 tokens 15.4 and 9.9, 17.5 and 12.8, 17.8 and 17.3; 1100 tokens 9.3 and 9.6
  // at 1024 rows, 9.6 and 11.0 at 1536).
  const bool wave = sb.cap <= SEL_NS && nch <= 64 && rows > (nch >= 8 ? 1536u : 1024u);
#define MITA_FINALIZE_CAP(TT, DD, MG)     \
  if (wave)                               \
    MITA_FINALIZE_WAVE(TT, DD, MG);       \
  else if (sb.cap <= 1024)                \
    MITA_FINALIZE(TT, DD, 1024, MG);      \
  else if (sb.cap <= 2048)                \
    MITA_FINALIZE(TT, DD, 2048, MG);      \
  else if (sb.cap <= 4096)                \
    MITA_FINALIZE(TT, DD, 4096, MG);      \
  else                                    \
    MITA_FINALIZE(TT, DD, SEL_CAP, MG);
  if (!v_lm) {
    MITA_FINALIZE_CAP(float, 64, false)
  } else if (c.dtype == MITA_F32) {
    if (c.d == 64) {
      MITA_FINALIZE_CAP(float, 64, true)
    } else {
      MITA_FINALIZE_CAP(float, 128, true)
    }
  } else {
    if (c.d == 64) {
      MITA_FINALIZE_CAP(bf16_t, 64, true)
    } else {
      MITA_FINALIZE_CAP(bf16_t, 128, true)
    }
  }
#undef MITA_FINALIZE_CAP
#undef MITA_FINALIZE_WAVE
#undef MITA_FINALIZE
  return launched(wave ? "finalize_wave_kernel" : "finalize_kernel", st);
}

hipError_t launch_select_finish(const mita_cfg_t &c, const void *q_lm, const void *k, const SelectBufs &sb, float *S,
                                int32_t *idx, const void *partial, void *v_lm, hipStream_t st) {
  if (sb.idx) return hipSuccess;  // the pivot launch wrote the sets; nothing is listed
  hipError_t e = launch_select_finalize(c, sb, idx, partial, v_lm, st);
  if (e != hipSuccess) return e;
  if ((e = launch_scores_rows(c, q_lm, k, S, sb.fail_cnt, sb.fail_list, st)) != hipSuccess) return e;
  return launch_topk(c, S, idx, st, sb.fail_cnt, sb.fail_list);
}

}  // namespace mita
