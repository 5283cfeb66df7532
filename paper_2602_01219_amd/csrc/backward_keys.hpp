// backward_keys.hpp - the keys' gradients of the bf16 backward pass on DMA
// tiles: a workgroup owns a block of keys and streams the queries that attend
// them.
#pragma once
#include <type_traits>

#include "cdna4.hpp"
#include "check.hpp"
#include "flash.hpp"
#include "worklist.hpp"

namespace mita {

// Arguments of the key-owned kernels (bf16 and fp32). Queries are numbered by
// item: position in the routing's grouping (perm), or token without routing.
struct KvArgs {
  const void *q, *k, *v, *dO, *q_lm, *v_lm;
  const int32_t *idx, *perm, *offsets;  // perm, offsets: NULL without routing
  const float *q_lse, *q_D;   // [BH, N] per item
  const void *dv_lm16;        // LMV keys: [BH, M, d] bf16 gradient of the landmark values
  const float *lse_lm, *D_lm; // LMV keys: [BH, M] the landmark rows' log-sum-exp and dV~ . V~
  // LMV keys: the routed keys' staged per-expert rows (inverse index
  // inv_start / inv_slot, NULL without routing) are summed in, and dk, dv
  // written in bf16
  const int32_t *inv_start, *inv_slot;
  void *dk_out, *dv_out;
  float *stage;               // ROUTED: [BH, M, k, 2, d] a slot's dK row, then its dV row
  float *part_k, *part_v;     // SHARED: [BH, chunks, M, d] sums over one query chunk
  // LMV keys: the landmark queries' gradient, dq_lm [BH, M, d] += the sum of
  // its nred partial sums dq_part [BH, nred, M, d] (blocks x >= ntotal)
  float *dq_lm;
  const float *dq_part;
  int nred;
  int N, M, topk;
  int nblk;                   // key blocks per expert (ROUTED) or landmark blocks (SHARED)
  int ntotal;                 // blocks with work (the grid is rounded up to a multiple of 8)
  int qchunk;                 // SHARED: queries per block (a multiple of 64)
  float scale;
};

// Orders one wave's LDS accesses before and after it (LDS serves a wave's
// accesses in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Key blocks: an expert's routed keys (its queries), landmark keys (a chunk of
// all queries), or tokens as the keys of the landmark values (the landmark
// rows as queries).
constexpr int KV_ROUTED = 0, KV_SHARED = 1, KV_LMV = 2;

// ---------------------------------------------------------------------------
// Wave w of NW owns NG 16-key column groups of the block's 16 NG NW keys;
// their K and V rows stay in registers as MFMA B fragments, dK^T and dV^T as
// accumulators. The queries come in stages of TS rows of Q and dO (LDS DMA,
// row-major with the 16-byte swizzle) with their log-sum-exps and D = dO . o,
// double buffered: the next stage is in flight while the current one's 32-row
// tiles are used, one barrier per stage. The two buffers are LDS objects of
// their own and each is named by a constant: in one array the compiler cannot
// tell the stage in flight from the one being read, and waits for it first (at
// 12 heads of 13818 tokens, M = 16, k = 56 the routed pass took 307 us, 241 with
// two). Per group and 32-query tile (lane
// (g, p): queries 16 qb + 4 g + r of key p):
//   S = Q K^T, dP = dO V^T; P = exp2(S scale log2 e - lse_q),
//   dZ = P (dP - D_q) (both rounded to bf16 for the MFMA);
//   dV^T += dO^T P, dK^T += Q^T dZ, with dO^T and Q^T read by transposing
//   LDS reads of the tiles (the P and dZ fragments are already the B
//   operand, in the key order of the transposing reads).
//
// What bounds it: the typical expert holds 10 to 130 queries, so a routed
// block's work is a few tiles behind a chain of dependent loads (the expert's
// offsets; its items, keys and log-sum-exps; the rows). The log-sum-exps and D
// are kept per item, contiguous for an expert, so that they are loaded beside
// the items and not behind them. A block
// of an expert without queries does nothing: its staged rows are not written
// and the inverse index leaves its slots out.
// ---------------------------------------------------------------------------
template <int D, int NG, int NW> struct KvTile {
  static constexpr int KB = 16 * NG * NW;           // keys per workgroup
  static constexpr int TS = D == 64 && NW == 4 ? 64 : 32;  // query rows per stage (16 KB; 8 KB for two waves)
  static constexpr int RB = 2 * D;                  // bytes per Q / dO row
  static constexpr int SB = 2 * TS * RB;            // bytes per stage (Q, then dO)
  // the landmark-value finish: TG tokens at a time per wave, 2 D floats each
  static constexpr int TG = D == 64 ? 16 : 8;
  static constexpr int FP = 2 * D + 4;              // floats per row: rows start 4 banks apart
  static constexpr int FB = NW / 2 * TG * FP * 4;   // the finish: half of the waves in each buffer
  template <int KM> static constexpr int bytes() { return KM == KV_LMV && FB > SB ? FB : SB; }
};

// LMV keys: the inverse index of the block's tokens, loaded while the landmark
// rows are streamed.
constexpr int KV_SLOTS = 1024;  // slots kept (a block's mean is 512 at M k = 4 N)
struct KvSlots {
  int32_t start[128 + 1];
  int32_t slot[KV_SLOTS];
};

// The staged per-expert rows of TG tokens (block tokens t0 .. t0 + TG - 1)
// added to their rows of `acc` (TG rows of FP floats in LDS: dK, then dV), by
// one wave. A slot's row is 2 D consecutive floats, read by D / 2 lanes, 16
// bytes each; at d = 64 the wave's halves take eight tokens each. The slots of
// consecutive tokens are consecutive in the index, so a half streams one list,
// U rows in flight, whatever the tokens' own counts (between 0 and over 100; a
// lane per token with its own loop waited for the longest list of the wave:
// 35 us of the 41 a block of 64 tokens took at 16384 tokens, M = 128, k = 512).
// KEPT: all of the block's slots are in ks.
template <int D, int FP, int TG, bool KEPT>
__device__ __forceinline__ void add_staged_rows(float *acc, const float *__restrict__ stage, const KvSlots &ks,
                                                const int32_t *__restrict__ slot, int t0) {
  constexpr int LPS = D / 2;           // lanes per slot row
  constexpr int TH = TG / (64 / LPS);  // tokens per part of the wave
  constexpr int U = 16;
  const int lane = threadIdx.x & 63, l = lane % LPS, part = lane / LPS;
  int s[TH + 1];  // the tokens' starts
#pragma unroll
  for (int i = 0; i <= TH; ++i) s[i] = ks.start[t0 + TH * part + i];
  const int base = ks.start[0], end = s[TH];
  float *row0 = acc + TH * part * FP + 4 * l;
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  int cur = -1;  // the token `sum` belongs to
  auto flush = [&]() {
    if (cur >= 0) {
      float4 *dst = reinterpret_cast<float4 *>(row0 + cur * FP);
      float4 x = *dst;
      x.x += sum.x; x.y += sum.y; x.z += sum.z; x.w += sum.w;
      *dst = x;
    }
  };
  for (int i = s[0]; i < end; i += U) {
    // (no branches: positions past the end repeat the last slot, unused)
    int sl[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = min(i + u, end - 1);
      sl[u] = KEPT ? ks.slot[at - base] : slot[at];
    }
    float4 y[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      y[u] = *reinterpret_cast<const float4 *>(stage + (int64_t)sl[u] * (2 * D) + 4 * l);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i + u >= end) break;
      int t = 0;
#pragma unroll
      for (int j = 1; j < TH; ++j) t += i + u >= s[j] ? 1 : 0;
      if (t != cur) {
        flush();
        cur = t;
        sum = y[u];
      } else {
        sum.x += y[u].x; sum.y += y[u].y; sum.z += y[u].z; sum.w += y[u].w;
      }
    }
  }
  flush();
}

// Block x of the (bh, x) grid.
template <int D, int KM, int NG, int NW>
__device__ __forceinline__ void kv16_body(const KvArgs &a, char *lds0, char *lds1, float *lse_s, float *nD_s,
                                          KvSlots *ks, int x) {
  using KT = KvTile<D, NG, NW>;
  constexpr int TS = KT::TS, RB = KT::RB, TQ = 32;
  using DT = DmaTile<D, TS, NW>;
  constexpr int PW = DT::PW;
  const int64_t bh = blockIdx.y;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 4, p = lane & 15;
  const int N = a.N, M = a.M, K = a.topk;
  int e = 0, kb0, nkeys, q0, nq;
  if (KM == KV_ROUTED) {
    e = x / a.nblk;
    kb0 = (x % a.nblk) * KT::KB;
    nkeys = min(KT::KB, K - kb0);
    q0 = a.offsets[bh * (M + 1) + e];
    nq = a.offsets[bh * (M + 1) + e + 1] - q0;
    if (nq == 0) return;  // uniform: no staged rows (the inverse index has none)
  } else if (KM == KV_SHARED) {
    kb0 = (x % a.nblk) * KT::KB;
    nkeys = min(KT::KB, M - kb0);
    q0 = (x / a.nblk) * a.qchunk;
    nq = min(a.qchunk, N - q0);
  } else {
    kb0 = x * KT::KB;
    nkeys = min(KT::KB, N - kb0);
    q0 = 0;
    nq = M;
  }
  constexpr bool LMV = KM == KV_LMV;
  // the streamed queries: tokens (q, dO), or for LMV keys the landmark rows
  // (q_lm and the landmark values' gradient)
  const int QN = LMV ? M : N;
  const char *qg = (const char *)(LMV ? a.q_lm : a.q) + bh * (int64_t)QN * RB;
  const char *dOg = (const char *)(LMV ? a.dv_lm16 : a.dO) + bh * (int64_t)QN * RB;
  const float *lse_g = (LMV ? a.lse_lm : a.q_lse) + bh * QN + q0;
  const float *D_g = (LMV ? a.D_lm : a.q_D) + bh * QN + q0;
  const int32_t *perm = !LMV && a.perm ? a.perm + bh * N + q0 : nullptr;

  // this lane's row of each of its wave's DMA instructions, and the row's
  // swizzled chunk (stages start at multiples of 32 rows: the same in each)
  DmaLane<D, TS, NW> dl;
  dl.init(w, lane);
  // of the stage to be issued next: the rows' tokens, and (lane = row) the
  // log-sum-exp (wave 0) or D (the last wave)
  int pm[PW];
  float ld;
  static_assert(NW > 1, "one wave loads the log-sum-exps, another D");
  auto load_rows = [&](int c0) {
    const int n = min(TS, nq - c0);
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      // rows past the last query repeat the stage's first
      const int i = c0 + ((int)dl.row[j] < n ? (int)dl.row[j] : 0);
      pm[j] = perm ? perm[i] : q0 + i;
    }
    if (w == 0 || w == NW - 1) ld = (w == 0 ? lse_g : D_g)[c0 + min(lane, n - 1)];
  };
  auto issue = [&](int c0, auto b_c) {
    constexpr int b = decltype(b_c)::value;
    const int n = min(TS, nq - c0), rows = (n + TQ - 1) / TQ * TQ;
    char *st = b ? lds1 : lds0;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int ins = w * PW + j;
      if (ins * DT::RPI < rows) {  // uniform
        const uint32_t go = (uint32_t)pm[j] * RB + dl.chunk[j];
        __builtin_amdgcn_global_load_lds(qg + go, (lds_void_t *)(st + ins * 1024), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(dOg + go, (lds_void_t *)(st + TS * RB + ins * 1024), 16, 0, 0);
      }
    }
    // rows past the last query have no weight: exp2(s - inf) = 0
    if (w == 0) lse_s[64 * b + lane] = lane < n ? ld : INFINITY;
    if (w == NW - 1) nD_s[64 * b + lane] = -ld;
  };

  load_rows(0);
  // the keys' rows (loaded behind the first items, used after the first stage)
  const bool tok_keys = KM != KV_SHARED;  // keys are token rows of k, v
  const bf16_t *kbase = tok_keys ? (const bf16_t *)a.k + bh * (int64_t)N * D : (const bf16_t *)a.q_lm + bh * (int64_t)M * D;
  const bf16_t *vbase = tok_keys ? (const bf16_t *)a.v + bh * (int64_t)N * D : (const bf16_t *)a.v_lm + bh * (int64_t)M * D;
  int krow[NG];
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    const int key = 16 * (NG * w + c) + p;
    krow[c] = key < nkeys ? (KM == KV_ROUTED ? a.idx[(bh * M + e) * (int64_t)K + kb0 + key] : kb0 + key) : 0;
  }
  issue(0, std::integral_constant<int, 0>{});
  if (TS < nq) load_rows(TS);
  Frag<bf16_t> kf[NG][D / 32], vf[NG][D / 32];
#pragma unroll
  for (int c = 0; c < NG; ++c)
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) {
      if (16 * (NG * w + c) + p < nkeys) {
        kf[c][ks].load(kbase + (int64_t)krow[c] * D + 32 * ks + 8 * g);
        vf[c][ks].load(vbase + (int64_t)krow[c] * D + 32 * ks + 8 * g);
      } else {
        kf[c][ks].zero();
        vf[c][ks].zero();
      }
    }
  f32x4 dka[NG][D / 16], dva[NG][D / 16];
#pragma unroll
  for (int c = 0; c < NG; ++c)
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      dka[c][db] = f32x4{0.f, 0.f, 0.f, 0.f};
      dva[c][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  Att16Addr<D> ad;
  ad.init();
  const float sl2 = a.scale * LOG2E;
  const bool busy = 16 * NG * w < nkeys;  // does the wave own keys?

  // one query tile at LDS rows qbase / dbase, its log-sum-exps and -D at lp / nDp
  auto tile = [&](const char *qbase, const char *dbase, const float *lp, const float *nDp) {
    f32x4 s[NG][2], dp[NG][2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        s[c][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
        dp[c][qb] = *reinterpret_cast<const f32x4 *>(nDp + 16 * qb + 4 * g);  // dP - D from the MFMAs
      }
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        Frag<bf16_t> A, B;
        A.v = *reinterpret_cast<const uint4 *>(qbase + ad.k[ks] + qb * 16 * RB);
        B.v = *reinterpret_cast<const uint4 *>(dbase + ad.k[ks] + qb * 16 * RB);
#pragma unroll
        for (int c = 0; c < NG; ++c) {
          s[c][qb] = mma(A, kf[c][ks], s[c][qb]);
          dp[c][qb] = mma(B, vf[c][ks], dp[c][qb]);
        }
      }
    }
    // the rows' log-sum-exps (queries 16 qb + 4 g + r of the tile)
    f32x4 lq[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) lq[qb] = *reinterpret_cast<const f32x4 *>(lp + 16 * qb + 4 * g);
    Frag<bf16_t> pf[NG], zf[NG];
#pragma unroll
    for (int c = 0; c < NG; ++c) {
      float pp[8], zz[8];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(s[c][qb][r], sl2, -lq[qb][r]));
          pp[4 * qb + r] = pr;
          zz[4 * qb + r] = pr * dp[c][qb][r];
        }
      pf[c].from_f32(pp);
      zf[c].from_f32(zz);
    }
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      uint2 hq[2], hd[2];
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        hq[h2] = __builtin_bit_cast(
            uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(qbase + ad.v[db] + h2 * 16 * RB)));
        hd[h2] = __builtin_bit_cast(
            uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(dbase + ad.v[db] + h2 * 16 * RB)));
      }
      Frag<bf16_t> AQ, AD;
      AQ.v = make_uint4(hq[0].x, hq[0].y, hq[1].x, hq[1].y);
      AD.v = make_uint4(hd[0].x, hd[0].y, hd[1].x, hd[1].y);
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        dva[c][db] = mma(AD, pf[c], dva[c][db]);
        dka[c][db] = mma(AQ, zf[c], dka[c][db]);
      }
    }
  };

  if (LMV && a.inv_start) {  // the tokens' starts (tokens past N: empty)
    static_assert(KM != KV_LMV || (KT::KB <= 128 && KT::KB < 64 * NW), "one start per thread");
    const int i = (int)threadIdx.x;
    if (i <= KT::KB) ks->start[i] = a.inv_start[bh * (N + 1) + min(kb0 + i, N)];
  }
  wait_loads();
  __syncthreads();
  constexpr int SPT = KV_SLOTS / (64 * NW);  // slots per thread
  int sl[SPT], nsl = 0;
  if (LMV && a.inv_start) {  // their slots, stored behind the first stage
    const int s0 = ks->start[0];
    nsl = min(KV_SLOTS, ks->start[KT::KB] - s0);
    const int32_t *sg = a.inv_slot + bh * (int64_t)M * K + s0;
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
      const int i = (int)threadIdx.x + 64 * NW * j;
      sl[j] = i < nsl ? sg[i] : 0;
    }
  }
  auto step = [&](int c0, auto b_c) {
    constexpr int b = decltype(b_c)::value;
    if (c0 + TS < nq) {
      issue(c0 + TS, std::integral_constant<int, b ^ 1>{});
      if (c0 + 2 * TS < nq) load_rows(c0 + 2 * TS);
    }
    // the next stage's DMA is issued before this one's arithmetic
    __builtin_amdgcn_sched_barrier(0);
    if (busy) {
      const int n = min(TS, nq - c0);
      const char *qb = b ? lds1 : lds0, *db = qb + TS * RB;
      const float *lp = lse_s + 64 * b, *nDp = nD_s + 64 * b;
      for (int t = 0; t < n; t += TQ) tile(qb + t * RB, db + t * RB, lp + t, nDp + t);
    }
    if (LMV && c0 == 0 && a.inv_start) {
#pragma unroll
      for (int j = 0; j < SPT; ++j) {
        const int i = (int)threadIdx.x + 64 * NW * j;
        if (i < nsl) ks->slot[i] = sl[j];
      }
    }
    wait_loads();
    __syncthreads();
  };
  for (int c0 = 0; c0 < nq; c0 += 2 * TS) {
    step(c0, std::integral_constant<int, 0>{});
    if (c0 + TS < nq) step(c0 + TS, std::integral_constant<int, 1>{});
  }

  if (LMV) {
    // the wave's tokens, TG at a time, through its part of the (now free)
    // stage buffers: the landmark-value sums, then the staged per-expert rows
    // on top, then dk and dv rows in bf16
    constexpr int TG = KT::TG, FP = KT::FP;
    float *acc = reinterpret_cast<float *>(w < NW / 2 ? lds0 : lds1) + w % (NW / 2) * TG * FP;
    const int64_t per_head = (int64_t)M * K;
#pragma unroll
    for (int c = 0; c < NG; ++c)
#pragma unroll
      for (int h = 0; h < 16 / TG; ++h) {
        const int key0 = 16 * (NG * w + c) + TG * h;
        if (key0 >= nkeys) continue;  // uniform for the wave
        if (p / TG == h) {
#pragma unroll
          for (int db = 0; db < D / 16; ++db) {
            float *dst = acc + (p % TG) * FP + 16 * db + 4 * g;
            *reinterpret_cast<float4 *>(dst) = make_float4(dka[c][db][0] * a.scale, dka[c][db][1] * a.scale,
                                                           dka[c][db][2] * a.scale, dka[c][db][3] * a.scale);
            *reinterpret_cast<float4 *>(dst + D) = make_float4(dva[c][db][0], dva[c][db][1], dva[c][db][2], dva[c][db][3]);
          }
        }
        wave_sync();
        if (a.inv_start) {
          const float *stage = a.stage + bh * per_head * (2 * D);
          const int32_t *slot = a.inv_slot + bh * per_head;
          if (ks->start[KT::KB] - ks->start[0] <= KV_SLOTS)  // uniform
            add_staged_rows<D, FP, TG, true>(acc, stage, *ks, slot, key0);
          else
            add_staged_rows<D, FP, TG, false>(acc, stage, *ks, slot, key0);
        }
        wave_sync();
        constexpr int LPR = D / 2;  // lanes per row: 4 floats each, dK then dV
        const int l = lane % LPR;
        bf16_t *out = l < LPR / 2 ? (bf16_t *)a.dk_out : (bf16_t *)a.dv_out;
#pragma unroll
        for (int r = lane / LPR; r < TG; r += 64 / LPR) {
          const float4 f = *reinterpret_cast<const float4 *>(acc + r * FP + 4 * l);
          if (key0 + r < nkeys)
            *reinterpret_cast<uint2 *>(out + (bh * N + kb0 + key0 + r) * D + 4 * (l % (LPR / 2))) =
                make_uint2(pack_bf16x2(f.x, f.y), pack_bf16x2(f.z, f.w));
        }
        wave_sync();
      }
    return;
  }
  // dK^T, dV^T: dims 16 db + 4 g + r of key p of group c
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    const int key = 16 * (NG * w + c) + p;
    if (key >= nkeys) continue;
    float *ko, *vo;
    if (KM == KV_ROUTED) {
      ko = a.stage + ((bh * M + e) * (int64_t)K + kb0 + key) * (2 * D) + 4 * g;
      vo = ko + D;
    } else {
      const int nch = a.ntotal / a.nblk;
      const int64_t at = ((bh * nch + x / a.nblk) * M + kb0 + key) * D + 4 * g;
      ko = a.part_k + at;
      vo = a.part_v + at;
    }
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      *reinterpret_cast<float4 *>(ko + 16 * db) = make_float4(dka[c][db][0] * a.scale, dka[c][db][1] * a.scale,
                                                              dka[c][db][2] * a.scale, dka[c][db][3] * a.scale);
      *reinterpret_cast<float4 *>(vo + 16 * db) = make_float4(dva[c][db][0], dva[c][db][1], dva[c][db][2], dva[c][db][3]);
    }
  }
}

// The landmark queries' gradient: dq_lm += the sum of its partial sums, one
// thread per 4 floats, blocks y of ny per head.
template <int D>
__device__ __forceinline__ void reduce_dq_lm(const KvArgs &a, int y, int ny, int nt) {
  const int64_t bh = blockIdx.y;
  const int n4 = a.M * D / 4;
  float4 *dst = reinterpret_cast<float4 *>(a.dq_lm) + bh * n4;
  const float4 *src = reinterpret_cast<const float4 *>(a.dq_part) + bh * a.nred * (int64_t)n4;
  for (int i = y * nt + (int)threadIdx.x; i < n4; i += ny * nt) {
    float4 s = dst[i];
#pragma unroll 8
    for (int c = 0; c < a.nred; ++c) {
      const float4 x = src[(int64_t)c * n4 + i];
      s.x += x.x; s.y += x.y; s.z += x.z; s.w += x.w;
    }
    dst[i] = s;
  }
}

// The block, spread over the XCDs as the attention work list is, so that the
// key blocks of one expert (the same queries) share an L2.
__device__ __forceinline__ int kv_block(int b, int nb) {
  const int C = (nb + NXCD - 1) / NXCD;
  return (b % NXCD) * C + b / NXCD;
}

// Three waves per SIMD: the accumulators and key fragments of two groups at
// d = 64 take 96 registers, a tile's scores and fragments about as many.
template <int D, int KM, int NG, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3))) void bwd_kv16_kernel(KvArgs a) {
  __shared__ __align__(16) char lds0[KvTile<D, NG, NW>::template bytes<KM>()];
  __shared__ __align__(16) char lds1[KvTile<D, NG, NW>::template bytes<KM>()];
  __shared__ __align__(16) float lse_s[2 * 64], nD_s[2 * 64];
  __shared__ std::conditional_t<KM == KV_LMV, KvSlots, char> ks_mem;
  KvSlots *ks = reinterpret_cast<KvSlots *>(&ks_mem);  // (LMV only)
  int nb = (int)gridDim.x, bx = (int)blockIdx.x;
  if (KM == KV_LMV) {
    // the last gridDim.x - nb blocks of a head reduce the landmark queries' gradient
    nb = (a.ntotal + NXCD - 1) / NXCD * NXCD;
    if (bx >= nb) {
      reduce_dq_lm<D>(a, bx - nb, (int)gridDim.x - nb, 64 * NW);
      return;
    }
  }
  const int x = kv_block(bx, nb);
  if (x >= a.ntotal) return;  // uniform
  kv16_body<D, KM, NG, NW>(a, lds0, lds1, lse_s, nD_s, ks, x);
}

}  // namespace mita
