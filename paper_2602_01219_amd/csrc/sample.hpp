// sample.hpp - the sampled scores and pivots of the fused top-k selection
// (Eq. top-k): each landmark row is scored against ns evenly spaced keys with
// the score pass's tile arithmetic, and its pivot is taken from those
// samples; used by the pivot launch and by the launch that runs it together
// with the routing logits.
#pragma once
#include <type_traits>

#include "cdna4.hpp"
#include "flash.hpp"
#include "check.hpp"
#include "scores.hpp"

namespace mita {

// Token index of sample j of ns: the middle of the j-th of ns equal parts of
// [0, N). Distinct and below N for ns <= N; equal to j when ns == N.
__device__ __forceinline__ int sample_pos(int j, int N, int ns) {
  return (int)(((2 * (int64_t)j + 1) * N) / (2 * (int64_t)ns));
}

// Bin of a 256-bin histogram (hist[0..255], counted from the top bin down)
// holding the need-th item, for one wave: returns the bin, *above = items in
// higher bins. need must be in [1, total].
__device__ __forceinline__ int wave_find_bin(const uint32_t *hist, uint32_t need, uint32_t *above) {
  const int lane = threadIdx.x & 63;
  uint32_t c[4], sum = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    c[q] = hist[255 - 4 * lane - q];
    sum += c[q];
  }
  const uint32_t incl = wave_inclusive_scan(sum);
  const uint32_t excl = incl - sum;
  int bin = -1;
  uint32_t ab = 0;
  if (excl < need && need <= incl) {
    uint32_t acc = excl;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (bin < 0) {
        if (acc + c[q] >= need)
          bin = 255 - 4 * lane - q;
        else
          acc += c[q];
      }
    }
    ab = acc;
  }
  const uint64_t m = __ballot(bin >= 0);
  const int src = __ffsll((unsigned long long)m) - 1;
  *above = (uint32_t)__shfl((int)ab, src);
  return __shfl(bin, src);
}

// ---------------------------------------------------------------------------
// Pivot of one landmark row from its at most 64 P keys, held by one wave, P per
// lane (in any order; 0 marks an empty slot: no score has key 0). The pivot is the exact r-th largest
// sampled key, found in two steps:
//  1. a 256-bin LDS histogram over the VALUE range [fmin, fmax] of the row's
//     samples (bin = floor((x - fmin) * 255.5 / (fmax - fmin)), a
//     non-decreasing function of the key, so every key in a higher bin is
//     larger than every key in a lower one) gives the bin holding the r-th
//     largest and the number of samples above it. Linear bins keep the
//     counts per bin small for bell-shaped scores (bins by key bits would put
//     a third of the samples into the one bin of a binade, and its LDS
//     atomics would serialise);
//  2. that bin's keys (at most 64 of them) are compacted into one register
//     per lane and an MSB-first bisection over the 32 key bits, counting by
//     ballots, finds the exact rank among them.
// Rows whose samples span a non-finite range or crowd more than 64 into the
// bin (clustered scores) take the bisection over all samples instead.
// Uses words 0..383 of the LDS row at `lds`.
// ---------------------------------------------------------------------------
// need-th largest of the keys x, one per lane (0 = none); 1 <= need <= count
// of nonzero keys. Bit b of the result is set iff at least `need` keys reach
// the result's higher bits with b set.
__device__ __forceinline__ uint32_t wave_kth_key(uint32_t x, uint32_t need) {
  uint32_t t = 0;
#pragma unroll
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t c = t | (1u << bit);
    if ((uint32_t)__popcll(__ballot(x >= c)) >= need) t = c;
  }
  return t;
}
// The same over P keys per lane.
template <int P>
__device__ __forceinline__ uint32_t wave_kth_key(const uint32_t (&x)[P], uint32_t need) {
  uint32_t t = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t c = t | (1u << bit);
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) n += (uint32_t)__popcll(__ballot(x[i] >= c));
    if (n >= need) t = c;
  }
  return t;
}

template <int P>
__device__ __forceinline__ uint32_t pivot_of(const uint32_t (&v)[P], uint32_t *lds, int r) {
  const int lane = threadIdx.x & 63;
  uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    if (v[i]) mn = min(mn, v[i]);
    mx = max(mx, v[i]);
  }
  const uint32_t kmin = wave_min_u32(mn), kmax = wave_max_u32(mx);
  if (kmin == kmax) return kmin;  // all samples equal
  const float fmin = key_to_float(kmin), span = key_to_float(kmax) - fmin;
  const float inv = 255.5f / span;
  if (!(span < INFINITY) || !(inv < INFINITY)) return wave_kth_key(v, (uint32_t)r);
  // (x - fmin) <= span after rounding, so (x - fmin) * inv < 256: bins 0..255;
  // empty slots go to words 256 + lane (distinct, never read as counts)
  uint32_t bin[P];
#pragma unroll
  for (int q = 0; q < 4; ++q) lds[lane + 64 * q] = 0u;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const uint32_t b = min((uint32_t)((key_to_float(v[i]) - fmin) * inv), 255u);
    bin[i] = v[i] ? b : 256u + (uint32_t)lane;
    atomicAdd(lds + bin[i], 1u);
  }
  uint32_t above;
  const uint32_t b = (uint32_t)wave_find_bin(lds, (uint32_t)r, &above);
  const uint32_t cnt = lds[b];
  if (cnt > 64u) return wave_kth_key(v, (uint32_t)r);
  uint32_t *slot = lds + 320;
  uint32_t base = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const uint64_t m = __ballot(bin[i] == b);
    if (bin[i] == b) slot[base + lanes_below(m)] = v[i];
    base += (uint32_t)__popcll(m);
  }
  return wave_kth_key((uint32_t)lane < cnt ? slot[lane] : 0u, (uint32_t)r - above);
}

// ---------------------------------------------------------------------------
// Sampled scores and pivots. Workgroup = ROWS waves for ROWS landmark rows of
// one head (4, 8 or 16): wave w scores the MFMA column block of 16 landmarks that
// holds them against every ROWS-th 64-key tile of the samples (the A fragments
// loaded straight from the sampled key rows, the next tile's in flight; tile
// arithmetic as in the score pass, so the same values) and keeps the ROWS
// rows' keys = score_key(fl(dot) * scale) in LDS; then wave w takes the pivot
// of row w, its histogram and compaction slots in the first 384 words of its
// row's keys once they are in registers (the wave's LDS accesses are in order).
// Several workgroups score each column block: the products are cheap, and a row
// per wave is the shortest chain. Where rows are many (few_rows), ROWS = 16 waves
// and rows read the keys once per block. Workgroup (0, 0) also zeroes the fallback
// counter.
// ---------------------------------------------------------------------------
constexpr int SP_ROWS = 4;            // landmark rows per workgroup
constexpr int SP_PITCH = SEL_NS + 4;  // keys per LDS row: rows start 4 banks apart
constexpr int SP_BYTES = SP_ROWS * SP_PITCH * 4;

// Workgroup (bx, by) of the sample grid (landmarks ROWS bx .. of head by; ROWS waves,
// a row each); keys: ROWS LDS rows of SP_PITCH words.
// SETS (the sample is the whole row, ns == N, and r == kk): the rows' top-kk
// sets are written too, in ascending token order: every key above the pivot
// and, in token order, as many keys equal to it as the set still needs (the
// order of the top-k: larger score first, lower index first among equal
// scores).
template <typename T, int D, bool SETS, int ROWS = SP_ROWS>
__device__ __forceinline__ void sample_pivot_body(uint32_t (*keys)[SP_PITCH], int bx, int by,
                                                  const T *__restrict__ q_lm, const T *__restrict__ k,
                                                  uint32_t *__restrict__ plo, uint32_t *__restrict__ fail_cnt, int N,
                                                  int M, int ns, int r, float scale, int32_t *__restrict__ idx,
                                                  int kk) {
  const int64_t bh = by;
  const int lm0 = bx * ROWS, lmb = lm0 & ~15;  // the rows; their column block
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, p = lane & 15;
  if (bx == 0 && by == 0 && threadIdx.x == 0) *fail_cnt = 0;
  Frag<T> qf[D / 32];
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    if (lmb + p < M)
      qf[ks].load(q_lm + (bh * M + lmb + p) * D + ks * 32 + g * 8);
    else
      qf[ks].zero();
  }
  const T *kb_ = k + bh * (int64_t)N * D;
  // a tile's A fragments, all loads issued before the first is used
  auto load = [&](Frag<T> (&a)[4][D / 32], int j0) {
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const int j = j0 + kb * 16 + p;  // A row p of block kb: sample j
      const int64_t pos = j < ns ? sample_pos(j, N, ns) : 0;
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) a[kb][ks].load(kb_ + pos * D + ks * 32 + g * 8);
    }
  };
  const int row = p - (lm0 - lmb);  // this column's row of the four, if it is one
  auto use = [&](const Frag<T> (&a)[4][D / 32], int j0) {
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) acc = mma(a[kb][ks], qf[ks], acc);
      // lane (g, p) holds samples j0 + 16 kb + 4 g + (0..3) of column p
      const int jb = j0 + kb * 16 + 4 * g;
      if (row >= 0 && row < ROWS) {
        uint32_t key[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) key[q] = jb + q < ns ? score_key(acc[q] * scale) : 0u;
        *reinterpret_cast<uint4 *>(&keys[row][jb]) = make_uint4(key[0], key[1], key[2], key[3]);
      }
    }
  };
  constexpr bool AHEAD = sizeof(T) == 2 && D == 64 && ROWS <= 8;  // (registers for two tiles' fragments)
  Frag<T> a[AHEAD ? 2 : 1][4][D / 32];
  const int j1 = min(ns, SEL_NS);
  if (AHEAD) {
    if (w * TK < j1) load(a[0], w * TK);
#pragma unroll
    for (int i = 0; i < SEL_NS / (ROWS * TK); ++i) {
      const int j0 = (ROWS * i + w) * TK;
      if (j0 + ROWS * TK < j1) load(a[(i + 1) & 1], j0 + ROWS * TK);
      if (j0 < j1) use(a[i & 1], j0);
    }
  } else {
    for (int j0 = w * TK; j0 < j1; j0 += ROWS * TK) {
      load(a[0], j0);
      use(a[0], j0);
    }
  }
  // slots past ns stay 0 (below every key) for the selection
  for (int j = ns + (int)threadIdx.x; j < SEL_NS; j += 64 * ROWS)
#pragma unroll
    for (int q = 0; q < ROWS; ++q) keys[q][j] = 0u;
  __syncthreads();
  // uniform for the wave; no workgroup barriers below
  if (lm0 + w >= M) return;
  // lane l holds keys 4 l + 256 i + (0..3); rows of at most 256 or 512 samples
  // take fewer registers and steps
  auto row_pivot = [&](auto per_c) {
    constexpr int P = decltype(per_c)::value;
    uint32_t v[P];
#pragma unroll
    for (int i = 0; i < P / 4; ++i) {
      const uint4 x = *reinterpret_cast<const uint4 *>(&keys[w][256 * i + 4 * lane]);
      v[4 * i] = x.x;
      v[4 * i + 1] = x.y;
      v[4 * i + 2] = x.z;
      v[4 * i + 3] = x.w;
    }
    const uint32_t lo = pivot_of(v, &keys[w][0], r);
    if (lane == 0) plo[bh * M + lm0 + w] = lo;
    if (!SETS) return;
    // the row's keys back in LDS (pivot_of used its first words)
#pragma unroll
    for (int i = 0; i < P / 4; ++i)
      *reinterpret_cast<uint4 *>(&keys[w][256 * i + 4 * lane]) = make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    uint32_t gt = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) gt += v[i] > lo ? 1u : 0u;
    const uint32_t need_eq = (uint32_t)kk - wave_sum_u32(gt);  // >= 1: lo is the kk-th largest
    int32_t *out = idx + (bh * M + lm0 + w) * (int64_t)kk;
    uint32_t taken = 0, eq_seen = 0;
    for (int j0 = 0; j0 < ns; j0 += 64) {
      const int j = j0 + lane;
      const uint32_t key = j < ns ? keys[w][j] : 0u;  // 0 lies below every key
      const uint64_t be = __ballot(key == lo);
      const bool take = key > lo || (key == lo && eq_seen + lanes_below(be) < need_eq);
      const uint64_t bt = __ballot(take);
      if (take) out[taken + lanes_below(bt)] = j;
      taken += (uint32_t)__popcll(bt);
      eq_seen += (uint32_t)__popcll(be);
    }
  };
  if (ns <= 256)
    row_pivot(std::integral_constant<int, 4>{});
  else if (ns <= 512)
    row_pivot(std::integral_constant<int, 8>{});
  else
    row_pivot(std::integral_constant<int, 16>{});
}

// ---------------------------------------------------------------------------
// The pivots alone, from SEL_NS samples of N > SEL_NS keys. Workgroup = NW waves
// for one MFMA column block of 16 landmark rows; wave w scores every NW-th
// 64-key tile, and the samples stay in registers as floats in key order (NaN
// as -inf, -0 as +0): lane (g, p) of a wave holds 256 / NW of row p. The exact r-th
// largest of each row, by the steps of pivot_of over all 16 rows at once:
// range, 256-bin histogram over it, the bin of rank r, that bin's few samples
// ranked. Rows whose range is not finite or whose bin holds more than 64
// samples bisect the 32 key bits over all samples instead.
// The sampled keys are read once per 16 rows and the samples cross LDS only as
// histogram counts: 22 KB per workgroup, so that the routing logits fit beside
// it (16 rows of keys took 66 KB; with four rows per workgroup, at 256 heads of
// 2048 tokens, M = 128, the launch with the logits took 159 us, 81 this way).
// What bounds a block is its chain: a round trip per tile of keys, a wave's tiles
// one after another, then some twenty instructions per sample and lane. So more
// waves where nothing else fills the CUs: without the logits sixteen (fp32
// eight), 14 us at up to 256 blocks of d = 64 and 30 at 1024, 17.5 and 36 with
// four.
// ---------------------------------------------------------------------------
struct PivotLds {
  uint32_t hist[16][260];  // counts per bin; rows start 4 banks apart
  uint32_t slot[16][64];   // the keys of a row's bin
  uint32_t red[16][2][16];  // the waves' key ranges per row
  uint32_t n[16];          // keys in slot
  uint32_t bin[16], above[16];
  uint32_t bad;            // some row bisects
};

__device__ __forceinline__ float canonical_score(float x) { return x != x ? -INFINITY : x + 0.f; }

template <typename T, int D, int NW = 4>
__device__ __forceinline__ void pivots16_body(PivotLds &sh, int bx, int by, const T *__restrict__ q_lm,
                                              const T *__restrict__ k, uint32_t *__restrict__ plo,
                                              uint32_t *__restrict__ fail_cnt, int N, int M, int r, float scale) {
  constexpr int NT = SEL_NS / (NW * TK);  // tiles per wave
  constexpr int RPW = 16 / NW;            // rows ranked per wave
  static_assert(NT * NW * TK == SEL_NS && RPW * NW == 16 && NW >= 4, "whole tiles and rows");
  const int64_t bh = by;
  const int lm0 = bx * 16;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, p = lane & 15;
  if (bx == 0 && by == 0 && tid == 0) *fail_cnt = 0;
  for (int i = tid; i < 16 * 260; i += 64 * NW) (&sh.hist[0][0])[i] = 0u;
  if (tid < 16) sh.n[tid] = 0u;
  if (tid == 0) sh.bad = 0u;
  Frag<T> qf[D / 32];
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    if (lm0 + p < M)
      qf[ks].load(q_lm + (bh * M + lm0 + p) * D + ks * 32 + g * 8);
    else
      qf[ks].zero();
  }
  const T *kb_ = k + bh * (int64_t)N * D;
  float x[NT][4][4];
  // a tile's loads are issued before the first is used, where registers allow
  // with the next tile's in flight
  constexpr bool AHEAD = sizeof(T) * D == 128;
  Frag<T> a[AHEAD ? 2 : 1][4][D / 32];
  auto load = [&](Frag<T>(&f)[4][D / 32], int t) {
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const int64_t pos = sample_pos((NW * t + w) * TK + kb * 16 + p, N, SEL_NS);
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) f[kb][ks].load(kb_ + pos * D + ks * 32 + g * 8);
    }
  };
  if (AHEAD) load(a[0], 0);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (!AHEAD)
      load(a[0], t);
    else if (t + 1 < NT)
      load(a[(t + 1) & 1], t + 1);
    // (else the loads sink to their uses, one wait each; with one tile per wave the
    // many waves cover those, and the registers held would halve them)
    if (NT > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) acc = mma(a[AHEAD ? t & 1 : 0][kb][ks], qf[ks], acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) x[t][kb][q] = canonical_score(acc[q] * scale);
    }
  }
  // every sample once: f(x)
  auto each = [&](auto f) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int q = 0; q < 4; ++q) f(x[t][kb][q]);
  };
  // the rows' ranges: lanes, lane groups, waves
  float lo = INFINITY, hi = -INFINITY;
  each([&](float v) {
    lo = fminf(lo, v);
    hi = fmaxf(hi, v);
  });
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    lo = fminf(lo, __shfl_xor(lo, o));
    hi = fmaxf(hi, __shfl_xor(hi, o));
  }
  if (g == 0) {
    sh.red[w][0][p] = __float_as_uint(lo);
    sh.red[w][1][p] = __float_as_uint(hi);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    lo = fminf(lo, __uint_as_float(sh.red[i][0][p]));
    hi = fmaxf(hi, __uint_as_float(sh.red[i][1][p]));
  }
  const float span = hi - lo, inv = 255.5f / span;
  // one value only (span 0) needs no bins; a range or scale that is not finite bisects
  const bool same = hi == lo, ok = !same && span < INFINITY && inv < INFINITY;
  auto bin_of = [&](float v) { return min((uint32_t)((v - lo) * inv), 255u); };
  if (ok) each([&](float v) { atomicAdd(&sh.hist[p][bin_of(v)], 1u); });
  if (w == 0 && g == 0 && !same && !ok) sh.bad = 1u;
  __syncthreads();
  if (w < 4) {
    // wave w's lane group g: the bin of row 4 w + g that holds rank r, lane p
    // summing bins 255 - 16 p down to 240 - 16 p
    const int row = 4 * w + g;
    uint32_t c[16], sum = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      c[i] = sh.hist[row][255 - 16 * p - i];
      sum += c[i];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 16);
      if (p >= o) incl += y;
    }
    uint32_t ab = incl - sum;
    if (ab < (uint32_t)r && (uint32_t)r <= incl) {  // one lane of the row (none if it has no bins)
      int b = 0;
      uint32_t cb = 0;
      bool found = false;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const bool here = !found && ab + c[i] >= (uint32_t)r;
        b = here ? 255 - 16 * p - i : b;
        cb = here ? c[i] : cb;
        found = found || here;
        ab += found ? 0u : c[i];
      }
      sh.bin[row] = (uint32_t)b;
      sh.above[row] = ab;
      if (cb > 64u) sh.bad = 1u;
    }
  }
  __syncthreads();
  if (sh.bad == 0u) {  // uniform
    const uint32_t mybin = sh.bin[p];
    if (ok)
      each([&](float v) {
        if (bin_of(v) == mybin) sh.slot[p][atomicAdd(&sh.n[p], 1u) & 63u] = ordered_key(v);
      });
    __syncthreads();
    // wave w ranks the slots of its RPW rows
    for (int i = 0; i < RPW; ++i) {
      const int row = RPW * w + i;
      if (lm0 + row >= M) break;  // uniform for the wave
      const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.n[row]);
      // (a row of one value: no slots)
      uint32_t key = ordered_key(__shfl(lo, row));
      if (n > 0u) {
        const uint32_t mine = (uint32_t)lane < n ? sh.slot[row][lane] : 0u;
        uint32_t rank = 0;
        for (uint32_t j = 0; j < n; ++j) {
          const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)j);
          rank += other > mine || (other == mine && j < (uint32_t)lane) ? 1u : 0u;
        }
        const uint64_t m = __ballot((uint32_t)lane < n && rank == (uint32_t)r - 1u - sh.above[row]);
        key = (uint32_t)__shfl((int)mine, __ffsll((unsigned long long)m) - 1);
      }
      if (lane == 0) plo[bh * M + lm0 + row] = key;
    }
    return;
  }
  // bisection over all samples, every row: bit b of the result is set iff at
  // least r samples reach the result's higher bits with b set (counts of step
  // `bit` in hist row bit / 2, words 128 (bit & 1) + row of a fresh buffer)
  __syncthreads();
  for (int i = tid; i < 16 * 260; i += 64 * NW) (&sh.hist[0][0])[i] = 0u;
  __syncthreads();
  uint32_t t = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t c = t | (1u << bit);
    uint32_t n = 0;
    each([&](float v) { n += ordered_key(v) >= c ? 1u : 0u; });
    n += (uint32_t)__shfl_xor((int)n, 16);
    n += (uint32_t)__shfl_xor((int)n, 32);
    uint32_t *cell = &sh.hist[bit >> 1][128 * (bit & 1) + p];
    if (g == 0) atomicAdd(cell, n);
    __syncthreads();
    if (*cell >= (uint32_t)r) t = c;
  }
  if (w == 0 && g == 0 && lm0 + p < M) plo[bh * M + lm0 + p] = t;
}

}  // namespace mita
