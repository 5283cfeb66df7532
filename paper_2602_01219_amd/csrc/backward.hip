// backward.hip - gradients of the MiTA forward with respect to q, k, v, the
// top-k sets and the routing held fixed (they are piecewise constant in the
// inputs): the attention of Eq. mita, the landmark values of Eq.
// landmark-value (itself an attention of the landmark queries over all keys)
// and the pooling of the landmark queries.
//
// bf16 takes the DMA-tiled kernels: bwd_att16_kernel (dQ, and the landmark
// queries' gradient) below and the key passes of backward_keys.hpp. fp32, and
// the dQ of bf16 row lists too long for LDS, take bwd_kernel in one of two modes:
//   ATT: a workgroup takes one tile of the forward's work list (64 queries
//        of one expert); its keys are the shared landmarks (keys q_lm,
//        values v_lm) and the expert's k routed rows. A first pass over the
//        keys forms each query's log-sum-exp (kept for the key side), a
//        second one dQ, in registers (a query's keys are all seen here),
//        written once.
//   LMV: a workgroup takes 64 landmarks (as queries) and one chunk of the
//        N keys; the upstream gradient is that of the landmark values, the
//        log-sum-exp of each landmark row comes from the score pass. dQ (the
//        landmark queries' gradient) is a partial sum over the chunk and is
//        added atomically.
// Per key tile of 32 keys, with P = softmax weights and dO the upstream
// gradient of the queries' outputs:
//   S^T = K Q^T, dP^T = V dO^T                      (keys x queries)
//   P = exp2(S^T * scale * log2 e - lse), dZ = P (dP - D), D = dO . o
//   dQ += dZ K,  dK += dZ^T Q,  dV += P^T dO        (scale applied at the end)
// All products run on MFMA (16x16 tiles over 32-long reduction steps) from
// LDS copies laid out so that most operands are read as 8 consecutive
// elements: Q and dO row-major (in the fp32 passes that need their columns those
// are read element by element), the key tile row-major and transposed, P and dZ
// as [key][query] and dZ as [query][key].
// The keys' gradients of the MiTA attention come from key-owned kernels
// (bwd_kv_kernel in fp32), where a workgroup owns a block of keys and streams
// the queries that attend them, so that dK and dV stay in registers: a routed
// key block of one expert sees that expert's queries (the per-expert sums are
// staged and then summed per token through an inverse index of the top-k sets);
// a block of shared keys sees a chunk of all queries and writes its partial
// sums, which bwd_prep_kernel adds up. fp32 atomic adds retire at a few hundred
// G/s on the whole chip, and many chunks adding to the same rows at less, so a
// design that adds every tile's key gradients atomically is bound by them.
// The order of a token's slots in the inverse index, and with it the order of
// its staged rows, varies from run to run (as do the atomic adds of the fp32
// landmark-value backward), so dq, dk, dv are reproducible only to rounding (a
// few ulp), not bit for bit.
#include "backward_keys.hpp"
#include "cdna4.hpp"
#include "check.hpp"
#include "flash.hpp"
#include "kernels.hpp"
#include "worklist.hpp"

namespace mita {

constexpr int BWD_TQ = 64;  // queries per workgroup
constexpr int BWD_TK = 32;  // keys per tile
constexpr int BWD_CHUNK = 512;  // keys per workgroup of the landmark-value backward

template <typename T, int D> struct BwdLds {
  static constexpr int PAD = 16 / (int)sizeof(T);
  static constexpr int QS = D + PAD;        // [query][d]
  static constexpr int KS = D + PAD;        // [key][d]
  static constexpr int KTS = BWD_TK + PAD;  // [d][key]
  static constexpr int PS = BWD_TQ + PAD;   // [key][query]
  static constexpr int ZS = BWD_TK + PAD;   // [query][key]
  static constexpr int NQ = BWD_TQ * QS, NK = BWD_TK * KS, NKT = D * KTS, NP = BWD_TK * PS, NZ = BWD_TQ * ZS;
};

// 8 elements base[(r0 + i) * stride + col], i < 8 (a column of a row-major tile).
__device__ __forceinline__ Frag<float> load_col(const float *base, int stride, int r0, int col) {
  Frag<float> f;
  f.a = make_float4(base[r0 * stride + col], base[(r0 + 1) * stride + col], base[(r0 + 2) * stride + col],
                    base[(r0 + 3) * stride + col]);
  f.b = make_float4(base[(r0 + 4) * stride + col], base[(r0 + 5) * stride + col], base[(r0 + 6) * stride + col],
                    base[(r0 + 7) * stride + col]);
  return f;
}

// 16 bytes of T at p as VE floats.
template <typename T> __device__ __forceinline__ void load16_f32(const T *p, float *x) {
  unpack16(*reinterpret_cast<const uint4 *>(p), x, p);
}

// Arguments of bwd_kernel (both modes).
struct BwdArgs {
  const void *q, *k, *v, *o, *dO;  // [BH, N, d] (io type)
  const void *q_lm, *v_lm;         // [BH, M, d] (io type)
  const int32_t *idx, *perm, *offsets, *tile_start;
  const float *lse_lm;     // [BH, M] landmark rows' log-sum-exp, log2 units (LMV)
  const float *dv_lm;      // [BH, M, d] gradient of the landmark values (LMV input)
  float *dq;               // [BH, N, d] ATT: the queries' direct gradient (written)
  float *dk, *dv;          // [BH, N, d] accumulators (atomic adds)
  float *dq_lm, *dv_lm_out;  // [BH, M, d] accumulators (atomic adds)
  float *q_lse, *q_D;      // [BH, N] ATT: each query's log-sum-exp (log2 units) and dO . o (written), by item
                           // (position in perm; token without routing)
  const void *dv_lm16;     // [BH, M, d] bf16 copy of dv_lm (the DMA-tiled landmark-value pass)
  const float *D_lm;       // [BH, M] dv_lm . v_lm (the DMA-tiled landmark-value pass)
  float *dq_part;          // [BH, chunks, M, d] the DMA-tiled landmark-value pass's sums per key chunk
  int N, M, topk, chunk;
  float scale;
};

constexpr int BWD_ATT = 0, BWD_LMV = 1;

template <typename T, int D, int MODE, bool SHARED, bool ROUTED>
__global__ __launch_bounds__(256) void bwd_kernel(BwdArgs a) {
  using L = BwdLds<T, D>;
  constexpr int VE = 16 / (int)sizeof(T);
  // the key-side tiles ([key][query] P and dZ) serve the LMV mode's dK and dV
  // only (fp32)
  constexpr bool KEYS = MODE == BWD_LMV;
  __shared__ __align__(16) T Qs[L::NQ];
  __shared__ __align__(16) T dOs[L::NQ];
  __shared__ __align__(16) T Ks[L::NK];
  __shared__ __align__(16) T Vs[L::NK];
  __shared__ __align__(16) T KT[L::NKT];
  __shared__ __align__(16) T Pkq[KEYS ? L::NP : 1];
  __shared__ __align__(16) T Zkq[KEYS ? L::NP : 1];
  __shared__ __align__(16) T Zqk[L::NZ];
  __shared__ float Dq[BWD_TQ];
  __shared__ int32_t qrow[BWD_TQ];  // each query's row in its tensor (token or landmark), -1 if none
  int64_t bh = blockIdx.y;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, g = lane >> 4, p = lane & 15;
  const int N = a.N, M = a.M, K = a.topk;
  const T *q = (const T *)a.q, *kk = (const T *)a.k, *vv = (const T *)a.v;
  const T *q_lm = (const T *)a.q_lm, *v_lm = (const T *)a.v_lm;

  // ---------------------------------------------------------------- queries
  int e = 0, q_begin = 0, q_end = 0, c0 = 0, c1 = 0;
  if (MODE == BWD_ATT) {
    if (!attend_queries<ROUTED>(a.tile_start, a.offsets, bh, N, M, e, q_begin, q_end)) return;  // uniform
  } else {
    const int nlb = (M + BWD_TQ - 1) / BWD_TQ;
    const int lb = (int)blockIdx.x % nlb, ch = (int)blockIdx.x / nlb;
    q_begin = lb * BWD_TQ;
    q_end = min(M, q_begin + BWD_TQ);
    c0 = ch * a.chunk;
    c1 = min(N, c0 + a.chunk);
    if (c0 >= N) return;
  }
  if (tid < BWD_TQ) {
    const int qi = q_begin + tid;
    int r = -1;
    if (qi < q_end) r = MODE == BWD_ATT ? (ROUTED ? a.perm[bh * N + qi] : qi) : qi;
    qrow[tid] = r;
  }
  __syncthreads();
  // Q and dO rows (zero for missing queries), their transposes, and D = dO . o
  {
    const T *qsrc = MODE == BWD_ATT ? q + bh * (int64_t)N * D : q_lm + bh * (int64_t)M * D;
    for (int c = tid; c < BWD_TQ * (D / VE); c += 256) {
      const int row = c / (D / VE), cc = c % (D / VE);
      const int r = qrow[row];
      uint4 xq = make_uint4(0, 0, 0, 0), xd = make_uint4(0, 0, 0, 0);
      if (r >= 0) {
        xq = *reinterpret_cast<const uint4 *>(qsrc + (int64_t)r * D + cc * VE);
        if (MODE == BWD_ATT) {
          xd = *reinterpret_cast<const uint4 *>((const T *)a.dO + (bh * N + r) * D + cc * VE);
        } else {
          float f[VE];
          const float *src = a.dv_lm + (bh * M + r) * D + cc * VE;
#pragma unroll
          for (int i = 0; i < VE; ++i) f[i] = src[i];
          T t[VE];
#pragma unroll
          for (int i = 0; i < VE; ++i) t[i] = from_f32<T>(f[i]);
          xd = *reinterpret_cast<const uint4 *>(t);
        }
      }
      *reinterpret_cast<uint4 *>(Qs + row * L::QS + cc * VE) = xq;
      *reinterpret_cast<uint4 *>(dOs + row * L::QS + cc * VE) = xd;
    }
    // D: four threads per query, D / 4 dimensions each, in fp32 (the upstream
    // gradient of the landmark values in its own fp32)
    const int row = tid >> 2, part = tid & 3;
    const int r = qrow[row];
    float dsum = 0.f;
    if (r >= 0) {
#pragma unroll
      for (int c = 0; c < D / 4; c += VE) {
        const int dim = part * (D / 4) + c;
        float ov[VE], dv[VE];
        if (MODE == BWD_ATT) {
          load16_f32((const T *)a.o + (bh * N + r) * D + dim, ov);
          load16_f32((const T *)a.dO + (bh * N + r) * D + dim, dv);
        } else {
          load16_f32(v_lm + (bh * M + r) * D + dim, ov);
#pragma unroll
          for (int i = 0; i < VE; ++i) dv[i] = a.dv_lm[(bh * M + r) * D + dim + i];
        }
#pragma unroll
        for (int i = 0; i < VE; ++i) dsum = __builtin_fmaf(ov[i], dv[i], dsum);
      }
    }
    dsum += __shfl_xor(dsum, 1);
    dsum += __shfl_xor(dsum, 2);
    if (part == 0) Dq[row] = dsum;
  }
  __syncthreads();

  // ---------------------------------------------------------------- keys
  // tiles: [0, nA) shared (landmark rows), [nA, nA + nB) routed / chunk rows
  const int nA = MODE == BWD_ATT && SHARED ? (M + BWD_TK - 1) / BWD_TK : 0;
  const int nkB = MODE == BWD_ATT ? (ROUTED ? K : 0) : c1 - c0;
  const int nB = (nkB + BWD_TK - 1) / BWD_TK;
  const int ntile = nA + nB;
  const int32_t *gidx = MODE == BWD_ATT && ROUTED ? a.idx + (bh * M + e) * (int64_t)K : nullptr;
  // row of key j of tile i in its tensor; rows >= nr are padding
  auto key_row = [&](int i, int j, bool &shared_key, int &nr) -> int {
    shared_key = i < nA;
    if (shared_key) {
      nr = min(BWD_TK, M - i * BWD_TK);
      return i * BWD_TK + j;
    }
    const int b0 = (i - nA) * BWD_TK;
    nr = min(BWD_TK, nkB - b0);
    if (MODE == BWD_ATT) return j < nr ? gidx[b0 + j] : 0;
    return c0 + b0 + j;
  };
  // stage key tile i: K rows (and V rows and K^T when full)
  auto stage = [&](int i, bool with_v) {
    for (int c = tid; c < BWD_TK * (D / VE); c += 256) {
      const int j = c / (D / VE), cc = c % (D / VE);
      bool sk;
      int nr;
      const int r = key_row(i, j, sk, nr);
      uint4 xk = make_uint4(0, 0, 0, 0), xv = make_uint4(0, 0, 0, 0);
      if (j < nr) {
        const T *kb = sk ? q_lm + bh * (int64_t)M * D : kk + bh * (int64_t)N * D;
        const T *vb = sk ? v_lm + bh * (int64_t)M * D : vv + bh * (int64_t)N * D;
        xk = *reinterpret_cast<const uint4 *>(kb + (int64_t)r * D + cc * VE);
        if (with_v) xv = *reinterpret_cast<const uint4 *>(vb + (int64_t)r * D + cc * VE);
      }
      *reinterpret_cast<uint4 *>(Ks + j * L::KS + cc * VE) = xk;
      if (with_v) {
        *reinterpret_cast<uint4 *>(Vs + j * L::KS + cc * VE) = xv;
        const T *tk = reinterpret_cast<const T *>(&xk);
#pragma unroll
        for (int u = 0; u < VE; ++u) KT[(cc * VE + u) * L::KTS + j] = tk[u];
      }
    }
  };
  const float sl2 = a.scale * LOG2E;
  const int myq = 16 * w + p;  // this lane's query (column of the S^T blocks)
  const bool qok = qrow[myq] >= 0;
  // S^T blocks of the wave's 16 queries against the tile's 32 keys
  auto scores = [&](f32x4 (&s)[2]) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      s[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        Frag<T> A, B;
        A.load(Ks + (16 * kb + p) * L::KS + 32 * ks + 8 * g);
        B.load(Qs + myq * L::QS + 32 * ks + 8 * g);
        s[kb] = mma(A, B, s[kb]);
      }
    }
  };

  // ---------------------------------------------------------------- pass 1: lse
  float lse;
  if (MODE == BWD_ATT) {
    float m = -INFINITY, l = 0.f;
    for (int i = 0; i < ntile; ++i) {
      __syncthreads();
      stage(i, false);
      __syncthreads();
      bool sk;
      int nr;
      key_row(i, 0, sk, nr);
      f32x4 s[2];
      scores(s);
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = 16 * kb + 4 * g + r < nr ? fmaxf(mx, s[kb][r] * sl2) : mx;
      const float mn = fmaxf(m, mx);
      float add = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          add += 16 * kb + 4 * g + r < nr ? __builtin_amdgcn_exp2f(s[kb][r] * sl2 - mn) : 0.f;
      l = (mn == -INFINITY ? 0.f : l * __builtin_amdgcn_exp2f(m - mn)) + add;
      m = mn;
    }
    // merge the four lane groups of the query's column
    const float mc = max_lane_groups(m);
    float lc = m == -INFINITY ? 0.f : l * __builtin_amdgcn_exp2f(m - mc);
    lc += __shfl_xor(lc, 16);
    lc += __shfl_xor(lc, 32);
    lse = mc + __log2f(lc);
    if (g == 0 && qok) {
      a.q_lse[bh * N + q_begin + myq] = lse;
      a.q_D[bh * N + q_begin + myq] = Dq[myq];
    }
  } else {
    lse = qok ? a.lse_lm[bh * M + q_begin + myq] : 0.f;
  }
  const float dq_row = Dq[myq];

  // ---------------------------------------------------------------- pass 2: gradients
  f32x4 dqa[D / 16];
#pragma unroll
  for (int db = 0; db < D / 16; ++db) dqa[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int NBLK = D / 16;  // dK / dV blocks per wave (D / 4 over the workgroup)
  for (int i = 0; i < ntile; ++i) {
    __syncthreads();
    stage(i, true);
    __syncthreads();
    bool sk;
    int nr;
    key_row(i, 0, sk, nr);
    f32x4 s[2], dp[2];
    scores(s);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      dp[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        Frag<T> A, B;
        A.load(Vs + (16 * kb + p) * L::KS + 32 * ks + 8 * g);
        B.load(dOs + myq * L::QS + 32 * ks + 8 * g);
        dp[kb] = mma(A, B, dp[kb]);
      }
    }
    // P and dZ of (key 16 kb + 4 g + r, query myq)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float pz[4], zz[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = 16 * kb + 4 * g + r;
        const bool ok = qok && key < nr;
        const float pr = ok ? __builtin_amdgcn_exp2f(s[kb][r] * sl2 - lse) : 0.f;
        pz[r] = pr;
        zz[r] = pr * (dp[kb][r] - dq_row);
        if constexpr (KEYS) {
          Pkq[key * L::PS + myq] = from_f32<T>(pz[r]);
          Zkq[key * L::PS + myq] = from_f32<T>(zz[r]);
        }
      }
      T z4[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) z4[r] = from_f32<T>(zz[r]);
      T *dst = Zqk + myq * L::ZS + 16 * kb + 4 * g;
      if (sizeof(T) == 2)
        *reinterpret_cast<uint2 *>(dst) = *reinterpret_cast<const uint2 *>(z4);
      else
        *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(z4);
    }
    __syncthreads();
    // dQ (queries 16 w + 4 g + r, dims 16 db + p) += dZ K over the tile's 32 keys
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      Frag<T> A, B;
      A.load(Zqk + myq * L::ZS + 8 * g);
      B.load(KT + (16 * db + p) * L::KTS + 8 * g);
      dqa[db] = mma(A, B, dqa[db]);
    }
    // LMV: dK = dZ^T Q and dV = P^T dO over the 64 queries (two 32-long
    // steps), block b = w * NBLK + j of D / 4: first half dK, second half dV
    // (in ATT mode the keys' gradients come from bwd_kv_kernel)
    if constexpr (KEYS)
#pragma unroll
    for (int j = 0; j < NBLK; ++j) {
      const int b = w * NBLK + j;
      const bool isv = b >= D / 8;
      const int rem = isv ? b - D / 8 : b;
      const int kb = rem / (D / 16), db = rem % (D / 16);
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) {
        Frag<T> A, B;
        A.load((isv ? Pkq : Zkq) + (16 * kb + p) * L::PS + 32 * qs + 8 * g);
        B = load_col(isv ? dOs : Qs, L::QS, 32 * qs + 8 * g, 16 * db + p);
        acc = mma(A, B, acc);
      }
      // rows: key 16 kb + 4 g + r of the tile; column: dim 16 db + p
      const float f = isv ? 1.f : a.scale;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = 16 * kb + 4 * g + r;
        if (key >= nr) continue;
        bool sk2;
        int nr2;
        const int row = key_row(i, key, sk2, nr2);
        float *dst;
        if (sk)
          dst = (isv ? a.dv_lm_out : a.dq_lm) + (bh * M + row) * D;
        else
          dst = (isv ? a.dv : a.dk) + (bh * N + row) * D;
        unsafeAtomicAdd(dst + 16 * db + p, acc[r] * f);
      }
    }
  }

  // ---------------------------------------------------------------- dQ out
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int qq = 16 * w + 4 * g + r;
    const int row = qrow[qq];
    if (row < 0) continue;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      const float val = dqa[db][r] * a.scale;
      if (MODE == BWD_ATT)
        a.dq[(bh * N + row) * D + 16 * db + p] = val;
      else
        unsafeAtomicAdd(a.dq_lm + (bh * M + row) * D + 16 * db + p, val);
    }
  }
}

// ---------------------------------------------------------------------------
// The dQ pass for bf16 with the key row list in LDS, on the forward
// attention's tile machinery (attend16_kernel): each wave owns NG 16-query
// column groups of the workgroup's 64 queries and every key; 32-key tiles by
// LDS DMA, double buffered, one barrier per tile, K and V row-major with the
// 16-byte swizzle, K^T read by ds_read_b64_tr_b16 for dQ. Per group and key
// tile (lane (g, p): keys 16 kb + 4 g + r of query p):
//   P = exp2(S^T scale log2 e - ref), S^T = K Q^T, dP^T = V dO^T,
//   dZ = P (dP - D) (rounded to bf16 for the MFMA), dQ^T += K^T dZ^T,
//   l += P (fp32);
// then dQ * scale / l, the log-sum-exp ref + log2 l and D = dO . o (fp32, over
// the lane's 16 dimensions and then the four lane groups) are written per
// query. S and P take the unscaled bf16 queries and an fp32 multiply by
// scale log2 e, as the key-owned kernel does.
// One sweep over the keys, as in the forward: ref is the column maximum of
// the first tile, and the weights, their sum and dQ stay unnormalised (the
// rounding of dZ to bf16 is relative, so the common factor does not matter).
// They overflow only when a later score exceeds the first tile's maximum by
// about 2^7 (log2 units); if some query's sums are then not finite, the
// workgroup sweeps the keys again for the log-sum-exps (K tiles only) and
// runs the pass with ref = lse, l = 1. At 16384 tokens, M = 128, k = 512,
// 24 heads the pass takes 154 us against 202 us with the two sweeps
// always.
// The landmark mode (LMV) has its log-sum-exps from the score pass and writes
// the key chunk's partial sums to dq_part (summed by the landmark-value key
// pass's spare blocks).
// ---------------------------------------------------------------------------
constexpr int BWD16_TK = 32;
constexpr int BWD16_LMV_CHUNK = 2048;  // most keys per workgroup of the landmark queries' gradient
template <int D> constexpr int BWD16_GROUPS = D == 64 ? 2 : 1;
// query groups per wave of the dQ pass: at d = 128 two waves per SIMD instead of
// four, but half the LDS reads per MFMA (16 heads of 4096 tokens, M = 64,
// k = 256: 80 -> 60 us; the landmark mode has too few workgroups to gain). Over one
// to 64 heads of 196 to 16384 tokens, M = 16 to 1000, k = 16 to 7500 it takes 0.71
// to 1.0 of one group's time, also where experts have few queries (384 heads of
// 196, M = 16: 79 against 103) and lists are long; up to 1.05 of it where there is
// less than one workgroup per CU (one head of 4096, M = 16, k = 1000: 52.3, 50.5).
constexpr int BWD16_DQ_GROUPS = 2;
template <int D> constexpr size_t bwd16_tiles_lds() { return 4 * (size_t)DmaTile<D, BWD16_TK>::BYTES; }

template <int D, bool SHARED, bool ROUTED, int NG, bool LMV = false>
__global__ __launch_bounds__(256 / NG) __attribute__((amdgpu_waves_per_eu(D == 128 && NG == 2 ? 2 : 4))) void bwd_att16_kernel(BwdArgs a) {
  constexpr int NW = 4 / NG;  // waves per workgroup
  constexpr int NT = 64 * NW;
  constexpr int TK = BWD16_TK;
  static_assert(NG * NW * 16 == BWD_TQ, "64 queries per workgroup");
  using DT = DmaTile<D, TK, NW>;
  constexpr int RB = 2 * D;  // bytes per K / V row
  __shared__ __align__(16) char tiles0[2 * DT::BYTES];
  __shared__ __align__(16) char tiles1[2 * DT::BYTES];
  auto Ks = [&](int b) { return reinterpret_cast<bf16_t *>(b ? tiles1 : tiles0); };
  auto Vt = [&](int b) { return reinterpret_cast<bf16_t *>((b ? tiles1 : tiles0) + DT::BYTES); };
  extern __shared__ uint32_t sidx[];  // byte offsets of the M + k key rows
  int64_t bh = blockIdx.y;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 4, p = lane & 15;
  const int N = a.N, M = a.M, K = a.topk;
  int e = 0, q_begin, q_end, c0 = 0, nck = 0;
  if (LMV) {
    // landmark block lb (the queries) against key chunk ch
    const int nlb = (M + BWD_TQ - 1) / BWD_TQ;
    const int lb = (int)blockIdx.x % nlb, ch = (int)blockIdx.x / nlb;
    q_begin = lb * BWD_TQ;
    q_end = min(M, q_begin + BWD_TQ);
    c0 = ch * a.chunk;
    if (c0 >= N) return;  // uniform
    nck = min(N - c0, a.chunk);
  } else if (!attend_queries<ROUTED>(a.tile_start, a.offsets, bh, N, M, e, q_begin, q_end)) {
    return;  // uniform
  }
  // LMV: the chunk's keys take the place of the routed ones
  const int nrt = LMV ? nck : (ROUTED ? K : 0);
  const int nA = SHARED && !LMV ? M / TK : 0, pA = SHARED && !LMV ? M % TK : 0;
  const int nB = nrt / TK, pB = nrt % TK;
  const int nfull = nA + nB;
  const bf16_t *sh_k = (const bf16_t *)a.q_lm + bh * (int64_t)M * D;
  const bf16_t *sh_v = (const bf16_t *)a.v_lm + bh * (int64_t)M * D;
  const bf16_t *rkb = (const bf16_t *)a.k + bh * (int64_t)N * D;
  const bf16_t *rvb = (const bf16_t *)a.v + bh * (int64_t)N * D;
  const int nsh = SHARED && !LMV ? M : 0;
  for (int i = threadIdx.x; i < nsh; i += NT) sidx[i] = (uint32_t)i * RB;
  if (LMV) {
    for (int i = threadIdx.x; i < nck; i += NT) sidx[i] = (uint32_t)(c0 + i) * RB;
  } else if (ROUTED) {
    const int32_t *gidx = a.idx + (bh * M + e) * (int64_t)K;
    for (int i = threadIdx.x; i < K; i += NT) sidx[nsh + i] = (uint32_t)gidx[i] * RB;
  }
  __syncthreads();
  const uint32_t *rows = sidx;
  auto tile_base = [&](int i, const bf16_t *&kb, const bf16_t *&vb, int &off) {
    const bool sh = i < nA;
    kb = sh ? sh_k : rkb;
    vb = sh ? sh_v : rvb;
    off = sh ? i * TK : nsh + (i - nA) * TK;
  };

  // this wave's groups: group c holds queries q_begin + 16 (NG w + c) + p
  // (LMV: landmark rows of q_lm, their upstream gradient in bf16, D given)
  const bf16_t *qg = LMV ? (const bf16_t *)a.q_lm : (const bf16_t *)a.q;
  const bf16_t *dOg = LMV ? (const bf16_t *)a.dv_lm16 : (const bf16_t *)a.dO, *og = (const bf16_t *)a.o;
  const int QN = LMV ? M : N;  // rows per head of the query tensors
  int tok[NG];
  bool qvalid[NG];
  Frag<bf16_t> qf[NG][D / 32], df[NG][D / 32];
  float Dq[NG];
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    const int qi = q_begin + 16 * (NG * w + c) + p;
    qvalid[c] = qi < q_end;
    tok[c] = qvalid[c] ? (ROUTED && !LMV ? a.perm[bh * N + qi] : qi) : 0;
    float dpart = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) {
      const int64_t at = (bh * QN + tok[c]) * D + ks * 32 + g * 8;
      if (LMV) {
        if (qvalid[c]) {
          qf[c][ks].load(qg + at);
          df[c][ks].load(dOg + at);
        } else {
          qf[c][ks].zero();
          df[c][ks].zero();
        }
      } else if (qvalid[c]) {
        qf[c][ks].load(qg + at);
        df[c][ks].load(dOg + at);
        float ov[8], dv[8];
        load16_f32(og + at, ov);
        unpack16(df[c][ks].v, dv, (const bf16_t *)nullptr);
#pragma unroll
        for (int i = 0; i < 8; ++i) dpart = __builtin_fmaf(ov[i], dv[i], dpart);
      } else {
        qf[c][ks].zero();
        df[c][ks].zero();
      }
    }
    // D = dO . o of query p: the four lane groups' parts, in a fixed order
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(dpart), __float_as_uint(dpart), false, false);
    const float pair = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(pair), __float_as_uint(pair), false, false);
    Dq[c] = __uint_as_float(y[0]) + __uint_as_float(y[1]);
    if (LMV) Dq[c] = qvalid[c] ? a.D_lm[bh * M + tok[c]] : 0.f;
  }
  int nbusy = 0;
#pragma unroll
  for (int c = 0; c < NG; ++c) nbusy += q_begin + 16 * (NG * w + c) < q_end ? 1 : 0;
  DmaLane<D, TK, NW> dl;
  dl.init(w, lane);
  Att16Addr<D> ad;
  ad.init();
  const float sl2 = a.scale * LOG2E;
  const bf16_t *kb, *vb;
  int off;
  wait_loads();
  __syncthreads();

  // S^T of the tile for the first NGB groups, from zero
  auto scores = [&](f32x4 (&acc)[NG][2], const bf16_t *Kl, auto ngb_c) {
    constexpr int NGB = decltype(ngb_c)::value;
    const char *kbase = reinterpret_cast<const char *>(Kl);
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
#pragma unroll
      for (int c = 0; c < NGB; ++c) acc[c][kb2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        Frag<bf16_t> A;
        A.v = *reinterpret_cast<const uint4 *>(kbase + ad.k[ks] + kb2 * 16 * RB);
#pragma unroll
        for (int c = 0; c < NGB; ++c) acc[c][kb2] = mma(A, qf[c][ks], acc[c][kb2]);
      }
    }
  };
  // One sweep over the key tiles (DMA pipeline as in attend16_kernel);
  // body(Kc, Vc, nvalid, masked_c) runs each tile's arithmetic,
  // first(Kc, nvalid, masked_c) comes before it on the first tile.
  auto sweep = [&](auto with_v_c, auto first, auto body) {
    constexpr bool WV = decltype(with_v_c)::value;
    auto issue = [&](int j, bf16_t *Kn, bf16_t *Vn) {
      if (j < nfull) {
        tile_base(j, kb, vb, off);
        dma_tile_lane<D, TK, NW, WV>(Kn, Vn, kb, vb, rows + off, dl);
      }
    };
    auto step = [&](int i, int b) {
      issue(i + 1, Ks(b ^ 1), Vt(b ^ 1));
      __builtin_amdgcn_sched_barrier(0);
      body(Ks(b), Vt(b), TK, std::false_type{});
      wait_loads();
      __syncthreads();
    };
    if (nfull > 0) {
      issue(0, Ks(0), Vt(0));
      wait_loads();
      __syncthreads();
      first(Ks(0), TK, std::false_type{});
      int i = 0;
      for (; i + 1 < nfull; i += 2) {
        step(i, 0);
        step(i + 1, 1);
      }
      if (i < nfull) step(i, 0);
    }
    for (int part = 0; part < 2; ++part) {
      const int nr = part == 0 ? pA : pB;
      if (nr == 0) continue;  // uniform
      if (part == 0)
        dma_tile<D, false, TK, NW, WV>(Ks(0), Vt(0), sh_k, sh_v, rows + nA * TK, nr);
      else
        dma_tile<D, false, TK, NW, WV>(Ks(0), Vt(0), rkb, rvb, rows + nsh + nB * TK, nr);
      wait_loads();
      __syncthreads();
      if (nfull == 0 && (part == 0 || pA == 0)) first(Ks(0), nr, std::true_type{});
      body(Ks(0), Vt(0), nr, std::true_type{});
      __syncthreads();
    }
  };
  // the sum over the four lane groups of a column, in a fixed order
  auto column_sum = [](float x) {
    const auto a4 = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float pair = __uint_as_float(a4[0]) + __uint_as_float(a4[1]);
    const auto b4 = __builtin_amdgcn_permlane32_swap(__float_as_uint(pair), __float_as_uint(pair), false, false);
    return __uint_as_float(b4[0]) + __uint_as_float(b4[1]);
  };

  // the log-sum-exps alone (after an overflow)
  float lm[NG], ll[NG];
  auto pass1 = [&](auto ngb_c) {
    constexpr int NGB = decltype(ngb_c)::value;
    sweep(std::false_type{}, [](const bf16_t *, int, auto) {}, [&](const bf16_t *Kc, const bf16_t *, int nv, auto masked_c) {
      constexpr bool MK = decltype(masked_c)::value;
      if (NGB == 0) return;
      f32x4 acc[NG][2];
      scores(acc, Kc, ngb_c);
#pragma unroll
      for (int c = 0; c < NGB; ++c) {
        float mx = -INFINITY;
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            mx = (!MK || 16 * kb2 + 4 * g + r < nv) ? fmaxf(mx, acc[c][kb2][r]) : mx;
        const float mn = fmaxf(lm[c], mx * sl2);
        float add = 0.f;
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            add += (!MK || 16 * kb2 + 4 * g + r < nv) ? __builtin_amdgcn_exp2f(__builtin_fmaf(acc[c][kb2][r], sl2, -mn))
                                                      : 0.f;
        ll[c] = (mn == -INFINITY ? 0.f : ll[c] * __builtin_amdgcn_exp2f(lm[c] - mn)) + add;
        lm[c] = mn;
      }
    });
  };
  // ref: the weights' reference (log2 units), ll: the lane's sum of the
  // weights; LMV: the landmark row's log-sum-exp from the score pass
  float ref[NG];
#pragma unroll
  for (int c = 0; c < NG; ++c) ref[c] = LMV && qvalid[c] ? a.lse_lm[bh * M + tok[c]] : 0.f;
  f32x4 dqa[NG][D / 16];
  bool redo = false;  // uniform for the workgroup
  auto pass2 = [&](auto ngb_c) {
    constexpr int NGB = decltype(ngb_c)::value;
    auto first = [&](const bf16_t *Kc, int nv, auto masked_c) {
      constexpr bool MK = decltype(masked_c)::value;
      if (LMV || NGB == 0 || redo) return;
      f32x4 acc[NG][2];
      scores(acc, Kc, ngb_c);
#pragma unroll
      for (int c = 0; c < NGB; ++c) ref[c] = max_lane_groups(att16_lane_max<MK>(acc[c], nv)) * sl2;
    };
    sweep(std::true_type{}, first, [&](const bf16_t *Kc, const bf16_t *Vc, int nv, auto masked_c) {
      constexpr bool MK = decltype(masked_c)::value;
      if (NGB == 0) return;
      f32x4 acc[NG][2], dp[NG][2];
      scores(acc, Kc, ngb_c);
      const char *vbase = reinterpret_cast<const char *>(Vc);
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2) {
#pragma unroll
        for (int c = 0; c < NGB; ++c) dp[c][kb2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
          Frag<bf16_t> A;
          A.v = *reinterpret_cast<const uint4 *>(vbase + ad.k[ks] + kb2 * 16 * RB);
#pragma unroll
          for (int c = 0; c < NGB; ++c) dp[c][kb2] = mma(A, df[c][ks], dp[c][kb2]);
        }
      }
      Frag<bf16_t> z[NG];
#pragma unroll
      for (int c = 0; c < NGB; ++c) {
        float zz[8];
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[c][kb2][r], sl2, -ref[c]));
            if (MK && 16 * kb2 + 4 * g + r >= nv) pr = 0.f;
            if (!LMV) ll[c] += pr;
            zz[4 * kb2 + r] = pr * (dp[c][kb2][r] - Dq[c]);
          }
        z[c].from_f32(zz);
      }
      // dQ^T += K^T dZ^T: the K^T operand by transposing reads of the K tile
      const char *kbase = reinterpret_cast<const char *>(Kc);
#pragma unroll
      for (int db = 0; db < D / 16; ++db) {
        uint2 half[2];
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
          half[h2] = __builtin_bit_cast(
              uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(kbase + ad.v[db] + h2 * 16 * RB)));
        Frag<bf16_t> A;
        A.v = make_uint4(half[0].x, half[0].y, half[1].x, half[1].y);
#pragma unroll
        for (int c = 0; c < NGB; ++c) dqa[c][db] = mma(A, z[c], dqa[c][db]);
      }
    });
  };
  auto run = [&](auto pass) {
    if (NG == 2 && nbusy == 2)
      pass(std::integral_constant<int, NG>{});
    else if (nbusy >= 1)
      pass(std::integral_constant<int, 1>{});
    else
      pass(std::integral_constant<int, 0>{});
  };
  __shared__ uint32_t overflow;
  if (!LMV && threadIdx.x == 0) overflow = 0u;
  float lsum[NG];
  while (true) {
    if (!LMV && redo) {
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        lm[c] = -INFINITY;
        ll[c] = 0.f;
      }
      run(pass1);
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        const float mc = max_lane_groups(lm[c]);
        ref[c] = mc + __log2f(column_sum(lm[c] == -INFINITY ? 0.f : ll[c] * __builtin_amdgcn_exp2f(lm[c] - mc)));
      }
    }
#pragma unroll
    for (int c = 0; c < NG; ++c) {
      ll[c] = 0.f;
#pragma unroll
      for (int db = 0; db < D / 16; ++db) dqa[c][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    run(pass2);
    if (LMV) break;
#pragma unroll
    for (int c = 0; c < NG; ++c) lsum[c] = redo ? 1.f : column_sum(ll[c]);
    if (redo) break;
    bool ok = true;
#pragma unroll
    for (int c = 0; c < NG; ++c) {
      // (a sum beyond 2^100 would also take scale / l into the subnormals)
      bool fin = lsum[c] < 0x1p100f;
#pragma unroll
      for (int db = 0; db < D / 16; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) fin = fin && __builtin_isfinite(dqa[c][db][r]);
      ok = ok && (fin || c >= nbusy);
    }
    if (__ballot(!ok) && lane == 0) atomicOr(&overflow, 1u);
    __syncthreads();
    if (overflow == 0u) break;  // uniform
    redo = true;
  }

  // ------------------------------------------------------------ outputs
  if (LMV) {  // the chunk's part of the landmark queries' gradient
    const int nlb = (M + BWD_TQ - 1) / BWD_TQ, nch = (int)gridDim.x / nlb, ch = (int)blockIdx.x / nlb;
#pragma unroll
    for (int c = 0; c < NG; ++c) {
      if (!qvalid[c]) continue;
      float *drow = a.dq_part + ((bh * nch + ch) * M + tok[c]) * D;
#pragma unroll
      for (int db = 0; db < D / 16; ++db)
        *reinterpret_cast<float4 *>(drow + db * 16 + 4 * g) =
            make_float4(dqa[c][db][0] * a.scale, dqa[c][db][1] * a.scale, dqa[c][db][2] * a.scale,
                        dqa[c][db][3] * a.scale);
    }
    return;
  }
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    if (!qvalid[c]) continue;
    const float f = a.scale / lsum[c];
    float *drow = a.dq + (bh * N + tok[c]) * D;
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
      *reinterpret_cast<float4 *>(drow + db * 16 + 4 * g) =
          make_float4(dqa[c][db][0] * f, dqa[c][db][1] * f, dqa[c][db][2] * f, dqa[c][db][3] * f);
    if (g == 0) {
      const int64_t item = bh * N + q_begin + 16 * (NG * w + c) + p;
      a.q_lse[item] = ref[c] + __log2f(lsum[c]);
      a.q_D[item] = Dq[c];
    }
  }
}

// ---------------------------------------------------------------------------
// Key-owned backward of the MiTA attention: a workgroup owns KB = 64 keys
// (wave w the 16 keys 16 w ..), whose K and V fragments stay in registers,
// and streams the queries that attend them in tiles of 64, with each query's
// log-sum-exp and D = dO . o from the dQ pass. Per query tile:
//   S^T = K Q^T, dP^T = V dO^T (keys x queries, one wave's 16 keys),
//   P = exp2(S^T scale log2 e - lse), dZ = P (dP - D),
//   dK += dZ^T Q, dV += P^T dO (reduction over the tile's 64 queries; P and
//   dZ go through a per-wave LDS area to take the operand layout).
//   ROUTED: block x = (expert e, key block b); keys idx[e][64 b ..], queries
//           the expert's group (perm[offsets[e] ..]); the expert's sums are
//           written to the staging rows [e][64 b ..] (plain stores).
//   SHARED: block x = (landmark block, chunk of qchunk queries); keys q_lm /
//           v_lm rows; the chunk's sums are written to part_k, part_v (their
//           sum over the chunks is taken by bwd_prep_kernel).
// Blocks are spread over the XCDs as the attention work list is, so the key
// blocks of one expert (same queries) share an L2.
// ---------------------------------------------------------------------------
constexpr int BWD_KB = 64;

template <int D> struct KvLds {
  static constexpr int PAD = 4;
  static constexpr int QS = D + PAD, WS = BWD_TQ + PAD;
  static constexpr int NQ = BWD_TQ * QS, NW = 4 * 16 * WS;
};

template <int D, bool ROUTED>
__global__ __launch_bounds__(256) void bwd_kv_kernel(KvArgs a) {
  using T = float;
  using L = KvLds<D>;
  constexpr int VE = 16 / (int)sizeof(T);
  __shared__ __align__(16) T Qs[L::NQ];
  __shared__ __align__(16) T dOs[L::NQ];
  __shared__ __align__(16) T Pw[L::NW];
  __shared__ __align__(16) T Zw[L::NW];
  __shared__ float lse_s[BWD_TQ], D_s[BWD_TQ];
  __shared__ int32_t qtok[BWD_TQ];
  const int64_t bh = blockIdx.y;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, g = lane >> 4, p = lane & 15;
  const int N = a.N, M = a.M, K = a.topk;
  const T *q = (const T *)a.q, *dO = (const T *)a.dO;
  // the block, spread over the XCDs
  const int nb = (int)gridDim.x;
  const int C = (nb + NXCD - 1) / NXCD;
  const int x = ((int)blockIdx.x % NXCD) * C + (int)blockIdx.x / NXCD;
  if (x >= a.ntotal) return;  // uniform
  int e = 0, kb0, nkeys, q0, nq;
  if (ROUTED) {
    e = x / a.nblk;
    kb0 = (x % a.nblk) * BWD_KB;
    nkeys = min(BWD_KB, K - kb0);
    q0 = a.offsets[bh * (M + 1) + e];
    nq = a.offsets[bh * (M + 1) + e + 1] - q0;
  } else {
    kb0 = (x % a.nblk) * BWD_KB;
    nkeys = min(BWD_KB, M - kb0);
    q0 = (x / a.nblk) * a.qchunk;
    nq = min(a.qchunk, N - q0);
  }
  if (nq == 0) return;  // uniform: no staged rows (the inverse index has none)
  // this wave's 16 keys: K and V fragments (row p of the wave's block)
  const int mykey = 16 * w + p;
  const bool kvalid = mykey < nkeys;
  int krow = 0;
  if (kvalid) krow = ROUTED ? a.idx[(bh * M + e) * (int64_t)K + kb0 + mykey] : kb0 + mykey;
  const T *kbase = ROUTED ? (const T *)a.k + bh * (int64_t)N * D : (const T *)a.q_lm + bh * (int64_t)M * D;
  const T *vbase = ROUTED ? (const T *)a.v + bh * (int64_t)N * D : (const T *)a.v_lm + bh * (int64_t)M * D;
  Frag<T> kf[D / 32], vf[D / 32];
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    if (kvalid) {
      kf[ks].load(kbase + (int64_t)krow * D + 32 * ks + 8 * g);
      vf[ks].load(vbase + (int64_t)krow * D + 32 * ks + 8 * g);
    } else {
      kf[ks].zero();
      vf[ks].zero();
    }
  }
  const float sl2 = a.scale * LOG2E;
  f32x4 dk[D / 16], dv[D / 16];
#pragma unroll
  for (int db = 0; db < D / 16; ++db) {
    dk[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    dv[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  T *pw = Pw + w * 16 * L::WS, *zw = Zw + w * 16 * L::WS;
  for (int t0 = 0; t0 < nq; t0 += BWD_TQ) {
    __syncthreads();
    if (tid < BWD_TQ) {
      int tok = -1;
      const int64_t item = bh * N + q0 + t0 + tid;
      const bool in = t0 + tid < nq;
      if (in) tok = a.perm ? a.perm[item] : q0 + t0 + tid;
      qtok[tid] = tok;
      lse_s[tid] = in ? a.q_lse[item] : 0.f;
      D_s[tid] = in ? a.q_D[item] : 0.f;
    }
    __syncthreads();
    for (int c = tid; c < BWD_TQ * (D / VE); c += 256) {
      const int row = c / (D / VE), cc = c % (D / VE);
      const int tok = qtok[row];
      uint4 xq = make_uint4(0, 0, 0, 0), xd = make_uint4(0, 0, 0, 0);
      if (tok >= 0) {
        xq = *reinterpret_cast<const uint4 *>(q + (bh * N + tok) * D + cc * VE);
        xd = *reinterpret_cast<const uint4 *>(dO + (bh * N + tok) * D + cc * VE);
      }
      *reinterpret_cast<uint4 *>(Qs + row * L::QS + cc * VE) = xq;
      *reinterpret_cast<uint4 *>(dOs + row * L::QS + cc * VE) = xd;
    }
    __syncthreads();
    // P and dZ of (key 16 w + 4 g + r, query 16 qb + p) into the wave's LDS area
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) {
      f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f}, dp = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        Frag<T> B;
        B.load(Qs + (16 * qb + p) * L::QS + 32 * ks + 8 * g);
        s = mma(kf[ks], B, s);
        B.load(dOs + (16 * qb + p) * L::QS + 32 * ks + 8 * g);
        dp = mma(vf[ks], B, dp);
      }
      const int qq = 16 * qb + p;
      const bool qok = qtok[qq] >= 0;
      const float lq = lse_s[qq], dq = D_s[qq];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = 16 * w + 4 * g + r;
        const bool ok = qok && key < nkeys;
        const float pr = ok ? __builtin_amdgcn_exp2f(s[r] * sl2 - lq) : 0.f;
        pw[(4 * g + r) * L::WS + qq] = pr;
        zw[(4 * g + r) * L::WS + qq] = pr * (dp[r] - dq);
      }
    }
    __syncthreads();
    // dK += dZ^T Q, dV += P^T dO: rows = the wave's 16 keys, columns = dims
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) {
        Frag<T> A, B;
        A.load(zw + p * L::WS + 32 * qs + 8 * g);
        B = load_col(Qs, L::QS, 32 * qs + 8 * g, 16 * db + p);
        dk[db] = mma(A, B, dk[db]);
        A.load(pw + p * L::WS + 32 * qs + 8 * g);
        B = load_col(dOs, L::QS, 32 * qs + 8 * g, 16 * db + p);
        dv[db] = mma(A, B, dv[db]);
      }
    }
  }
  // rows: key 16 w + 4 g + r of the block; column: dim 16 db + p
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int key = 16 * w + 4 * g + r;
    if (key >= nkeys) continue;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      if (ROUTED) {
        const int64_t at = ((bh * M + e) * (int64_t)K + kb0 + key) * (2 * D) + 16 * db + p;
        a.stage[at] = dk[db][r] * a.scale;
        a.stage[at + D] = dv[db][r];
      } else {
        const int nch = a.ntotal / a.nblk;
        const int64_t at = ((bh * nch + x / a.nblk) * M + kb0 + key) * D + 16 * db + p;
        a.part_k[at] = dk[db][r] * a.scale;
        a.part_v[at] = dv[db][r];
      }
    }
  }
}

// What the landmark-value backward needs of each landmark row, one wave per
// row (lane = 4 dims of the row and, of the chunks, every (256 / D)-th; the
// parts are then summed across lanes):
//  - dv_lm and dq_lm = the sums of the shared keys' partial sums over the
//    query chunks;
//  - for the DMA-tiled kernels (dv16 given) dv_lm in bf16 (the MFMA operand)
//    and D = dV~ . V~ (fp32) instead of dv_lm;
//  - the row's log-sum-exp (log2 units) from the score pass's per-chunk (max,
//    sum) partials, every 64th per lane.
__device__ __forceinline__ void lse_combine(float &m, float &l, float2 x) {
  const float mn = fmaxf(m, x.x);
  if (mn == -INFINITY) return;  // (nothing but empty partials so far)
  l = l * __builtin_amdgcn_exp2f(m - mn) + x.y * __builtin_amdgcn_exp2f(x.x - mn);
  m = mn;
}
template <typename T, int D>
__global__ __launch_bounds__(256) void bwd_prep_kernel(const float *__restrict__ part_k,
                                                       const float *__restrict__ part_v, int nchunk,
                                                       const T *__restrict__ v_lm, float *__restrict__ dq_lm,
                                                       float *__restrict__ dv_lm, bf16_t *__restrict__ dv16,
                                                       float *__restrict__ D_lm, const float2 *__restrict__ part_ml,
                                                       float *__restrict__ lse, int64_t rows, int M, int nch) {
  constexpr int L = D / 4, P = 64 / L;  // lanes per row copy, parts of the chunks
  const int lane = threadIdx.x & 63, c = 4 * (lane % L);
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;  // the whole wave
  const int64_t bh = row / M;
  const int lm = (int)(row - bh * M);
  float4 fk = make_float4(0.f, 0.f, 0.f, 0.f), fv = fk;
  const int64_t at0 = (bh * nchunk * M + lm) * D + c;
#pragma unroll 4
  for (int ch = lane / L; ch < nchunk; ch += P) {
    const float4 x = *reinterpret_cast<const float4 *>(part_k + at0 + (int64_t)ch * M * D);
    const float4 y = *reinterpret_cast<const float4 *>(part_v + at0 + (int64_t)ch * M * D);
    fk.x += x.x; fk.y += x.y; fk.z += x.z; fk.w += x.w;
    fv.x += y.x; fv.y += y.y; fv.z += y.z; fv.w += y.w;
  }
  float m = -INFINITY, l = 0.f;
  const float2 *ml = part_ml + bh * nch * M + lm;
  for (int i = lane; i < nch; i += 64) lse_combine(m, l, ml[(int64_t)i * M]);
#pragma unroll
  for (int o = L; o < 64; o <<= 1) {
    fk.x += __shfl_xor(fk.x, o); fk.y += __shfl_xor(fk.y, o); fk.z += __shfl_xor(fk.z, o); fk.w += __shfl_xor(fk.w, o);
    fv.x += __shfl_xor(fv.x, o); fv.y += __shfl_xor(fv.y, o); fv.z += __shfl_xor(fv.z, o); fv.w += __shfl_xor(fv.w, o);
  }
  float dsum = 0.f;
  if (dv16) {
    const T *vp = v_lm + row * D + c;
    const float f[4] = {fv.x, fv.y, fv.z, fv.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) dsum = __builtin_fmaf(to_f32<T>(vp[i]), f[i], dsum);
  }
#pragma unroll
  for (int o = 1; o < L; o <<= 1) dsum += __shfl_xor(dsum, o);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float2 other = make_float2(__shfl_xor(m, o), __shfl_xor(l, o));
    lse_combine(m, l, other);
  }
  if (lane < L) {
    *reinterpret_cast<float4 *>(dq_lm + row * D + c) = fk;
    if (dv16)
      *reinterpret_cast<uint2 *>(dv16 + row * D + c) = make_uint2(pack_bf16x2(fv.x, fv.y), pack_bf16x2(fv.z, fv.w));
    else
      *reinterpret_cast<float4 *>(dv_lm + row * D + c) = fv;
  }
  if (lane == 0) {
    if (dv16) D_lm[row] = dsum;
    lse[row] = m + __log2f(l);
  }
}

// Inverse index of the top-k sets: for each token, the slots e * k + j with
// idx[e][j] = token, listed by start [BH, N + 1] and slot [BH, M * k] (a
// counting sort). One workgroup per (head, range of T tokens), its counters
// in LDS: it reads all of its head's sets, counting the slots of its own
// tokens and those of the tokens below its range (the range's base), scans
// its counts from that base, and places its slots on a second read. The
// order of a token's slots is that of the LDS atomics. Entries outside
// [0, N), and those of experts without queries (no staged rows; about 40% of
// the experts on clustered inputs), are left out of the index.
constexpr int INV_THREADS = 1024, INV_WAVES = INV_THREADS / 64;
constexpr int INV_TMAX = 15360;  // tokens per workgroup: 60 KiB of counters (+ 384 B)

// Is expert i among the head's experts with queries (bit i of live)? The
// expert of entry e is e / k: the estimate by rk = floor(2^32 / k) is the
// quotient or one less (e < 2^31).
__device__ __forceinline__ bool inv_live(const uint32_t *live, uint32_t e, uint32_t k, uint32_t rk) {
  uint32_t i = __umulhi(e, rk);
  if (e - i * k >= k) ++i;
  return (live[i >> 5] >> (i & 31)) & 1u;
}

// f(e, tok) for the head's per_head entries, strided over the workgroup, 16
// per thread and call (e[i] the entry, tok[i] its token; -1 pads a short
// batch and stands for the entries of experts without queries): up to
// sixteen 16-byte loads in flight where the rows allow them (k a multiple of
// four: the four entries of a load are one expert's), and the callee's LDS
// atomics of a batch issued before their results are used.
template <class F>
__device__ __forceinline__ void inv_entries(const int32_t *__restrict__ ih, int per_head, uint32_t k, uint32_t rk,
                                            const uint32_t *live, F &&f) {
  int e[16], t[16];
  int i = threadIdx.x;
  if ((k & 3) == 0 && ((uintptr_t)ih & 15) == 0) {
    const int4 *v = reinterpret_cast<const int4 *>(ih);
    const int n4 = per_head >> 2;
    // eight loads in flight (with sixteen the registers of the live test spill)
    for (; i + 7 * INV_THREADS < n4; i += 8 * INV_THREADS) {
      int4 x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = v[i + u * INV_THREADS];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e0 = 4 * (i + (4 * b + u) * INV_THREADS);
          const int4 y = x[4 * b + u];
          const bool ok = inv_live(live, (uint32_t)e0, k, rk);
          e[4 * u] = e0, e[4 * u + 1] = e0 + 1, e[4 * u + 2] = e0 + 2, e[4 * u + 3] = e0 + 3;
          t[4 * u] = ok ? y.x : -1, t[4 * u + 1] = ok ? y.y : -1, t[4 * u + 2] = ok ? y.z : -1,
                t[4 * u + 3] = ok ? y.w : -1;
        }
        f(e, t);
      }
    }
    for (; i + 3 * INV_THREADS < n4; i += 4 * INV_THREADS) {
      int4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = v[i + u * INV_THREADS];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e0 = 4 * (i + u * INV_THREADS);
        const bool ok = inv_live(live, (uint32_t)e0, k, rk);
        e[4 * u] = e0, e[4 * u + 1] = e0 + 1, e[4 * u + 2] = e0 + 2, e[4 * u + 3] = e0 + 3;
        t[4 * u] = ok ? x[u].x : -1, t[4 * u + 1] = ok ? x[u].y : -1, t[4 * u + 2] = ok ? x[u].z : -1,
              t[4 * u + 3] = ok ? x[u].w : -1;
      }
      f(e, t);
    }
#pragma unroll
    for (int q = 4; q < 16; ++q) e[q] = 0, t[q] = -1;
    for (; i < n4; i += INV_THREADS) {
      const int4 x = v[i];
      const bool ok = inv_live(live, 4 * (uint32_t)i, k, rk);
      e[0] = 4 * i, e[1] = 4 * i + 1, e[2] = 4 * i + 2, e[3] = 4 * i + 3;
      t[0] = ok ? x.x : -1, t[1] = ok ? x.y : -1, t[2] = ok ? x.z : -1, t[3] = ok ? x.w : -1;
      f(e, t);
    }
    return;
  }
  for (; i < per_head; i += 16 * INV_THREADS) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      e[q] = i + q * INV_THREADS;
      t[q] = e[q] < per_head ? ih[e[q]] : -1;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (e[q] < per_head && !inv_live(live, (uint32_t)e[q], k, rk)) t[q] = -1;
    f(e, t);
  }
}

// Grid: NXCD * ceil(nwork / NXCD) workgroups of INV_THREADS, nwork = BH *
// parts, parts = ceil(N / T); dynamic LDS (T + 2 * INV_WAVES + 64) * 4 bytes.
__global__ __launch_bounds__(INV_THREADS) void inv_index_kernel(const int32_t *__restrict__ idx,
                                                                int32_t *__restrict__ start,
                                                                int32_t *__restrict__ slot,
                                                                const int32_t *__restrict__ offsets, int M, int K,
                                                                uint32_t rk, int N, int T, int parts, int64_t nwork) {
  extern __shared__ uint32_t inv_lds[];  // counters, wave sums, a spare word per lane
  __shared__ uint32_t live[1024 / 32];   // the experts with queries (M <= 1024 = INV_THREADS)
  const int per_head = M * K;
  uint32_t *cnt = inv_lds, *wsum = inv_lds + T;
  // a head's ranges on consecutive slots of one XCD, which share its sets in L2
  const int64_t w = xcd_slot((int)blockIdx.x, (int)(gridDim.x / NXCD));
  if (w >= nwork) return;
  const int64_t bh = w / parts;
  const int t0 = (int)(w % parts) * T;
  const uint32_t nt = (uint32_t)min(N - t0, T);
  const int32_t *ih = idx + bh * per_head;
  for (uint32_t i = threadIdx.x; i < nt; i += INV_THREADS) cnt[i] = 0;
  {
    const int32_t *of = offsets + bh * (M + 1);
    const int i = (int)threadIdx.x;
    const uint64_t m = __ballot(i < M && of[min(i + 1, M)] > of[min(i, M)]);
    if ((i & 63) == 0) {
      live[i >> 5] = (uint32_t)m;
      live[(i >> 5) + 1] = (uint32_t)(m >> 32);
    }
  }
  __syncthreads();
  uint32_t below = 0;
  // (entries of other tokens count into a word of their lane past the
  // counters: atomics without branches, whose results wait only once)
  uint32_t *const spare = inv_lds + T + 2 * INV_WAVES + (threadIdx.x & 63);
  inv_entries(ih, per_head, (uint32_t)K, rk, live, [&](const int(&)[16], const int(&t)[16]) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const uint32_t r = (uint32_t)t[q] - (uint32_t)t0;
      below += (uint32_t)t[q] < (uint32_t)t0 ? 1u : 0u;
      atomicAdd(r < nt ? &cnt[r] : spare, 1u);
    }
  });
  __syncthreads();
  // exclusive scan of the counts from the base (consecutive runs per thread)
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t per = (nt + INV_THREADS - 1) / INV_THREADS;
  const uint32_t b0 = min(nt, threadIdx.x * per), b1 = min(nt, b0 + per);
  uint32_t sum = 0;
  for (uint32_t i = b0; i < b1; ++i) sum += cnt[i];
  const uint32_t incl = wave_inclusive_scan(sum), bw = wave_sum_u32(below);
  if (lane == 63) {
    wsum[wv] = incl;
    wsum[INV_WAVES + wv] = bw;
  }
  __syncthreads();
  uint32_t before = incl - sum, base = 0, all = 0;
#pragma unroll
  for (int i = 0; i < INV_WAVES; ++i) {
    before += i < wv ? wsum[i] : 0u;
    all += wsum[i];
    base += wsum[INV_WAVES + i];
  }
  before += base;
  for (uint32_t i = b0; i < b1; ++i) {
    const uint32_t c = cnt[i];
    cnt[i] = before;
    before += c;
  }
  __syncthreads();
  int32_t *sh = start + bh * (N + 1) + t0;
  for (uint32_t i = threadIdx.x; i < nt; i += INV_THREADS) sh[i] = (int32_t)cnt[i];
  if (threadIdx.x == 0 && t0 + (int)nt == N) sh[nt] = (int32_t)(base + all);
  __syncthreads();  // (the copy above reads the starts before the atomics move them)
  // place: cnt holds each token's next free position (< base + all <= per_head)
  int32_t *sl = slot + bh * per_head;
  inv_entries(ih, per_head, (uint32_t)K, rk, live, [&](const int(&e)[16], const int(&t)[16]) {
    uint32_t r[16], pos[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      r[q] = (uint32_t)t[q] - (uint32_t)t0;
      pos[q] = atomicAdd(r[q] < nt ? &cnt[r[q]] : spare, 1u);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (r[q] < nt) sl[pos[q]] = e[q];
  });
}

// Exclusive scan of cnt over each head's N tokens into start [BH, N + 1]
// (1024 threads per head, consecutive runs per thread; the merge rounds'
// positions of the surviving tokens).
__global__ __launch_bounds__(1024) void inv_scan_kernel(const int32_t *__restrict__ cnt, int32_t *__restrict__ start,
                                                        int N) {
  __shared__ uint32_t wsum[16];
  const int64_t bh = blockIdx.x;
  const int per = (N + 1023) / 1024;
  const int b0 = threadIdx.x * per, b1 = min(N, b0 + per);
  uint32_t sum = 0;
  for (int i = b0; i < b1; ++i) sum += (uint32_t)cnt[bh * N + i];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t incl = wave_inclusive_scan(sum);
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t before = incl - sum, all = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    before += i < w ? wsum[i] : 0u;
    all += wsum[i];
  }
  for (int i = b0; i < b1; ++i) {
    start[bh * (N + 1) + i] = (int32_t)before;
    before += (uint32_t)cnt[bh * N + i];
  }
  if (threadIdx.x == 0) start[bh * (N + 1) + N] = (int32_t)all;
}

// dk_acc, dv_acc of every token = the sum of its staged per-expert rows
// (written, not added: the first contribution). One thread per 4 dims.
template <int D>
__global__ __launch_bounds__(256) void inv_gather_kernel(const float *__restrict__ stage,
                                                         const int32_t *__restrict__ start,
                                                         const int32_t *__restrict__ slot, float *__restrict__ dk,
                                                         float *__restrict__ dv, int64_t rows, int N, int per_head) {
  constexpr int C = D / 4;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = t / C;
  const int c = (int)(t % C);
  if (row >= rows) return;
  const int64_t bh = row / N;
  const int tok = (int)(row % N);
  const int s0 = start[bh * (N + 1) + tok], s1 = start[bh * (N + 1) + tok + 1];
  float4 xk = make_float4(0.f, 0.f, 0.f, 0.f), xv = xk;
  for (int i = s0; i < s1; ++i) {
    const int64_t src = (bh * (int64_t)per_head + slot[bh * (int64_t)per_head + i]) * (2 * D) + 4 * c;
    const float4 yk = *reinterpret_cast<const float4 *>(stage + src);
    const float4 yv = *reinterpret_cast<const float4 *>(stage + src + D);
    xk.x += yk.x; xk.y += yk.y; xk.z += yk.z; xk.w += yk.w;
    xv.x += yv.x; xv.y += yv.y; xv.z += yv.z; xv.w += yv.w;
  }
  *reinterpret_cast<float4 *>(dk + row * D + 4 * c) = xk;
  *reinterpret_cast<float4 *>(dv + row * D + 4 * c) = xv;
}

// The gradients in the io type: dq = the direct part + the pooling backward
// of the landmark queries' gradient (each token of window W_i receives
// dq_lm_i / |W_i|), dk, dv from their accumulators. One thread per 16 dims
// (four 4-dim chunks, FIN_TPR threads per row side by side on each chunk),
// so a token's windows are found once per 16 dims. Along each axis a
// position lies in at most two adaptive windows, among floor(pos * g / G) -
// 1 .. + 1.
template <int D> constexpr int FIN_TPR = D / 16;  // threads per row
template <typename T, int D, bool POOL, bool KV = true>
__global__ __launch_bounds__(256) void bwd_finish_kernel(const float *__restrict__ dq_direct,
                                                         const float *__restrict__ dq_lm,
                                                         const float *__restrict__ dk_acc,
                                                         const float *__restrict__ dv_acc, T *__restrict__ dq,
                                                         T *__restrict__ dk, T *__restrict__ dv, int64_t rows, int N,
                                                         int M, int gh, int gw, int lh, int lw) {
  constexpr int C = FIN_TPR<D>;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = t / C;
  const int c = (int)(t % C);
  if (row >= rows) return;
  int64_t bh;
  int tok;
  if (rows <= (int64_t)UINT32_MAX) {  // (32-bit division where the rows allow it)
    bh = (int64_t)((uint32_t)row / (uint32_t)N);
    tok = (int)((uint32_t)row - (uint32_t)bh * (uint32_t)N);
  } else {
    bh = row / N;
    tok = (int)(row % N);
  }
  const int64_t at = row * D + 4 * c;  // chunk j at at + 4 C j
  float4 x[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const float4 *>(dq_direct + at + 4 * C * j);
  if (POOL) {
    // 32-bit index arithmetic: positions stay below 2^16 (N <= 65536) and
    // window counts at most 1024 (M <= 1024), so every product below is
    // under 2^27
    const uint32_t pr = (uint32_t)tok / (uint32_t)gw, pc = (uint32_t)tok - pr * (uint32_t)gw;
    const int ar = (int)(pr * (uint32_t)lh / (uint32_t)gh), ac = (int)(pc * (uint32_t)lw / (uint32_t)gw);
    for (int a = max(0, ar - 1); a <= min(lh - 1, ar + 1); ++a) {
      const int r0 = (int)((uint32_t)a * (uint32_t)gh / (uint32_t)lh);
      const int r1 = (int)(((uint32_t)(a + 1) * (uint32_t)gh + (uint32_t)lh - 1u) / (uint32_t)lh);
      if ((int)pr < r0 || (int)pr >= r1) continue;
      for (int b = max(0, ac - 1); b <= min(lw - 1, ac + 1); ++b) {
        const int s0 = (int)((uint32_t)b * (uint32_t)gw / (uint32_t)lw);
        const int s1 = (int)(((uint32_t)(b + 1) * (uint32_t)gw + (uint32_t)lw - 1u) / (uint32_t)lw);
        if ((int)pc < s0 || (int)pc >= s1) continue;
        const float inv = 1.f / (float)((r1 - r0) * (s1 - s0));
        const float *src = dq_lm + (bh * M + a * lw + b) * D + 4 * c;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 y = *reinterpret_cast<const float4 *>(src + 4 * C * j);
          x[j].x += y.x * inv;
          x[j].y += y.y * inv;
          x[j].z += y.z * inv;
          x[j].w += y.w * inv;
        }
      }
    }
  }
  auto put = [&](T *dst, int j, float4 f) {
    T vals[4] = {from_f32<T>(f.x), from_f32<T>(f.y), from_f32<T>(f.z), from_f32<T>(f.w)};
    if (sizeof(T) == 2)
      *reinterpret_cast<uint2 *>(dst + at + 4 * C * j) = *reinterpret_cast<const uint2 *>(vals);
    else
      *reinterpret_cast<uint4 *>(dst + at + 4 * C * j) = *reinterpret_cast<const uint4 *>(vals);
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) put(dq, j, x[j]);
  if (KV) {  // (else the landmark-value key pass wrote dk and dv)
    float4 yk[4], yv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      yk[j] = *reinterpret_cast<const float4 *>(dk_acc + at + 4 * C * j);
      yv[j] = *reinterpret_cast<const float4 *>(dv_acc + at + 4 * C * j);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      put(dk, j, yk[j]);
      put(dv, j, yv[j]);
    }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Rows per chunk for a pass of `blocks` blocks per head and chunk that writes
// M rows of partial sums per chunk: a multiple of `unit` (at least two units),
// at most `most`, such that the launch has about `target` workgroups and the
// head's partial sums fit the N rows of their buffer.
static int bwd_chunk(const mita_cfg_t &c, int blocks, int unit, int most, int64_t target) {
  const int64_t want = (BH(c) * blocks * c.N + target - 1) / target;
  int64_t n = std::min<int64_t>(std::max<int64_t>(2 * unit, (want + unit - 1) / unit * unit), most);
  while (n < c.N && (c.N + n - 1) / n * c.M > c.N) n += unit;
  return (int)n;
}

template <typename T, int D>
static hipError_t bwd_t(const mita_cfg_t &c, const BwdBufs &b, hipStream_t st) {
  BwdArgs a{};
  a.q = b.q;
  a.k = b.k;
  a.v = b.v;
  a.o = b.o;
  a.dO = b.dO;
  a.q_lm = b.q_lm;
  a.v_lm = b.v_lm;
  a.idx = b.idx;
  a.perm = b.perm;
  a.offsets = b.offsets;
  a.tile_start = b.tile_start;
  a.lse_lm = b.lse_lm;
  a.dv_lm = b.dv_lm_acc;
  a.dq = b.dq_direct;
  a.dk = b.dk_acc;
  a.dv = b.dv_acc;
  a.dq_lm = b.dq_lm_acc;
  a.dv_lm_out = b.dv_lm_acc;
  a.q_lse = b.q_lse;
  a.q_D = b.q_D;
  a.N = c.N;
  a.M = c.M;
  a.topk = c.k;
  a.scale = eff_scale(c);
  const unsigned bh = (unsigned)BH(c);
  hipError_t err;
  // dQ of the MiTA attention, and each query's log-sum-exp and D
  int tiles = (c.N + ATT_TQ - 1) / ATT_TQ;
  if (c.use_routed) tiles = (tiles + c.M + NXCD - 1) / NXCD * NXCD;
  const dim3 grid((unsigned)tiles, bh);
  const int nlist = (c.use_shared ? c.M : 0) + (c.use_routed ? c.k : 0);
  bool done = false;
  if constexpr (sizeof(T) == 2) {
    // bf16 with the key row list in LDS: the DMA-tiled kernel
    if (list_in_lds(nlist, bwd16_tiles_lds<D>())) {
      constexpr int NG = BWD16_DQ_GROUPS;
      const dim3 blk(256 / NG);
      const size_t dyn = (size_t)nlist * sizeof(uint32_t);
      if (c.use_shared && c.use_routed)
        hipLaunchKernelGGL((bwd_att16_kernel<D, true, true, NG>), grid, blk, dyn, st, a);
      else if (c.use_routed)
        hipLaunchKernelGGL((bwd_att16_kernel<D, false, true, NG>), grid, blk, dyn, st, a);
      else
        hipLaunchKernelGGL((bwd_att16_kernel<D, true, false, NG>), grid, blk, dyn, st, a);
      done = true;
    }
  }
  if (!done) {
    if (c.use_shared && c.use_routed)
      hipLaunchKernelGGL((bwd_kernel<T, D, BWD_ATT, true, true>), grid, dim3(256), 0, st, a);
    else if (c.use_routed)
      hipLaunchKernelGGL((bwd_kernel<T, D, BWD_ATT, false, true>), grid, dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL((bwd_kernel<T, D, BWD_ATT, true, false>), grid, dim3(256), 0, st, a);
  }
  if ((err = launched("bwd_attend_kernel", st)) != hipSuccess) return err;
  KvArgs kv{};
  kv.q = b.q;
  kv.k = b.k;
  kv.v = b.v;
  kv.dO = b.dO;
  kv.q_lm = b.q_lm;
  kv.v_lm = b.v_lm;
  kv.idx = b.idx;
  kv.q_lse = b.q_lse;
  kv.q_D = b.q_D;
  kv.perm = c.use_routed ? b.perm : nullptr;
  kv.offsets = c.use_routed ? b.offsets : nullptr;
  kv.stage = b.stage;
  // the landmark rows' partial sums, in the buffers of the keys' sums, which
  // are not in use yet: at most N rows per head (bwd_chunk)
  kv.part_k = b.dk_acc;
  kv.part_v = b.dv_acc;
  kv.dq_lm = b.dq_lm_acc;
  kv.N = c.N;
  kv.M = c.M;
  kv.topk = c.k;
  kv.scale = eff_scale(c);
  const bool fused_finish = sizeof(T) == 2 && c.use_shared;
  if (c.use_shared) {
    // shared keys (the landmarks): partial sums per landmark block and query
    // chunk, then their sums with the landmark rows' log-sum-exps. About one
    // workgroup per CU slot (three 4-wave workgroups per CU; the fp32
    // kernel's two): fewer leave CUs idle, more only add partial sums.
    int nchunk = 0;
    auto shared_keys = [&](int kb, int64_t target) {
      kv.nblk = (c.M + kb - 1) / kb;
      kv.qchunk = bwd_chunk(c, kv.nblk, 64, c.N, target);
      nchunk = (c.N + kv.qchunk - 1) / kv.qchunk;
      kv.ntotal = kv.nblk * nchunk;
      return dim3((unsigned)((kv.ntotal + NXCD - 1) / NXCD * NXCD), bh);
    };
    if constexpr (sizeof(T) == 2) {
      constexpr int NG = BWD16_GROUPS<D>;
      bool two = false;
      if constexpr (D == 64) {
        two = c.M <= 64;  // two waves cover the block
        if (two) {
          const dim3 g = shared_keys(KvTile<D, NG, 2>::KB, 1536);
          hipLaunchKernelGGL((bwd_kv16_kernel<D, KV_SHARED, NG, 2>), g, dim3(128), 0, st, kv);
        }
      }
      if (!two) {
        const dim3 g = shared_keys(KvTile<D, NG, 4>::KB, 768);
        hipLaunchKernelGGL((bwd_kv16_kernel<D, KV_SHARED, NG, 4>), g, dim3(256), 0, st, kv);
      }
    } else {
      const dim3 g = shared_keys(BWD_KB, 512);
      hipLaunchKernelGGL((bwd_kv_kernel<D, false>), g, dim3(256), 0, st, kv);
    }
    if ((err = launched("bwd_kv_shared_kernel", st)) != hipSuccess) return err;
    const int64_t mrows = BH(c) * c.M;
    hipLaunchKernelGGL((bwd_prep_kernel<T, D>), dim3((unsigned)((mrows + 3) / 4)), dim3(256), 0, st,
                       kv.part_k, kv.part_v, nchunk, (const T *)b.v_lm, b.dq_lm_acc, b.dv_lm_acc,
                       sizeof(T) == 2 ? (bf16_t *)b.dv_lm16 : nullptr, b.D_lm, (const float2 *)b.part_ml, b.lse_lm,
                       mrows, c.M, score_chunks(c));
    if ((err = launched("bwd_prep_kernel", st)) != hipSuccess) return err;
  }
  if (c.use_routed) {
    // routed keys: per-expert sums staged, then summed per token
    auto routed_keys = [&](int kb) {
      kv.nblk = (c.k + kb - 1) / kb;
      kv.ntotal = c.M * kv.nblk;
      return dim3((unsigned)((kv.ntotal + NXCD - 1) / NXCD * NXCD), bh);
    };
    if constexpr (sizeof(T) == 2) {
      constexpr int NG = BWD16_GROUPS<D>;
      bool two = false;
      if constexpr (D == 64) {
        // Two waves cover the block, unless there are few blocks of many queries:
        // then a block's chain of stages counts, and the two other waves double
        // the stage (us with two and with four waves, k = 49: 12 heads of 13818
        // tokens, M = 16 112 and 83; 12 of 512, M = 16 11.6 and 11.0; 48 of 4096,
        // M = 16 49.5 and 39.6, M = 64 57.0 and 60.8; 12 of 196, M = 16 9.8 and 9.9;
        // 384 of 196 43.7 and 54.6).
        two = c.k <= 64 && !(BH(c) * c.M <= 1024 && c.N >= 32 * c.M);
        if (two) {
          const dim3 g = routed_keys(KvTile<D, NG, 2>::KB);
          hipLaunchKernelGGL((bwd_kv16_kernel<D, KV_ROUTED, NG, 2>), g, dim3(128), 0, st, kv);
        }
      }
      if (!two) {
        const dim3 g = routed_keys(KvTile<D, NG, 4>::KB);
        hipLaunchKernelGGL((bwd_kv16_kernel<D, KV_ROUTED, NG, 4>), g, dim3(256), 0, st, kv);
      }
    } else {
      const dim3 g = routed_keys(BWD_KB);
      hipLaunchKernelGGL((bwd_kv_kernel<D, true>), g, dim3(256), 0, st, kv);
    }
    if ((err = launched("bwd_kv_kernel", st)) != hipSuccess) return err;
    const int per_head = c.M * c.k;
    // token ranges per head: about one workgroup per CU over all heads (a
    // head's ranges on one XCD), at least 256 tokens each, at most INV_TMAX
    const int64_t heads = BH(c), per_xcd = (heads + NXCD - 1) / NXCD;
    int parts = (int)std::max<int64_t>(1, 256 / (NXCD * per_xcd));
    parts = std::min(parts, std::max(1, c.N / 256));
    parts = std::max(parts, (c.N + INV_TMAX - 1) / INV_TMAX);
    const int span = (c.N + parts - 1) / parts;
    parts = (c.N + span - 1) / span;
    const int64_t nwork = heads * parts;
    const uint32_t rk = (uint32_t)std::min<uint64_t>(UINT32_MAX, (1ull << 32) / (uint64_t)c.k);
    hipLaunchKernelGGL(inv_index_kernel, dim3((unsigned)((nwork + NXCD - 1) / NXCD * NXCD)), dim3(INV_THREADS),
                       (size_t)(span + 2 * INV_WAVES + 64) * 4, st, b.idx, b.inv_start, b.inv_slot, b.offsets, c.M, c.k,
                       rk, c.N, span, parts, nwork);
    if ((err = launched("inv_index_kernel", st)) != hipSuccess) return err;
    if (!fused_finish) {  // (else the landmark-value key pass sums the staged rows)
      const int64_t rows = BH(c) * c.N;
      hipLaunchKernelGGL((inv_gather_kernel<D>), dim3((unsigned)((rows * (D / 4) + 255) / 256)), dim3(256), 0, st,
                         b.stage, b.inv_start, b.inv_slot, b.dk_acc, b.dv_acc, rows, c.N, per_head);
      if ((err = launched("inv_gather_kernel", st)) != hipSuccess) return err;
    }
  } else if (!fused_finish) {  // no routed keys: the landmark values' sums are added to zero
    const int64_t nd = BH(c) * c.N * c.d;
    if ((err = launch_zero2((int32_t *)b.dk_acc, nd, (int32_t *)b.dv_acc, nd, st)) != hipSuccess) return err;
  }
  if (c.use_shared) {
    // the landmark values (Eq. landmark-value)
    const int nlb = (c.M + BWD_TQ - 1) / BWD_TQ;
    if constexpr (sizeof(T) == 2) {
      // bf16: the landmark queries' gradient by landmark blocks and key
      // chunks (partial sums per chunk), then the keys' gradient by token
      // blocks with all landmark rows streamed; that kernel's spare blocks add
      // up the partial sums, and it also sums the routed keys' staged rows and
      // writes dk, dv (no gather pass, no fp32 accumulators of the keys)
      constexpr int NG = BWD16_GROUPS<D>;
      a.dv_lm16 = b.dv_lm16;
      a.D_lm = b.D_lm;
      a.dq_part = b.dk_acc;
      a.chunk = bwd_chunk(c, nlb, BWD16_TK, BWD16_LMV_CHUNK, 1024);
      const int nch16 = (c.N + a.chunk - 1) / a.chunk;
      hipLaunchKernelGGL((bwd_att16_kernel<D, false, false, NG, true>), dim3((unsigned)(nlb * nch16), bh),
                         dim3(256 / NG), (size_t)a.chunk * sizeof(uint32_t), st, a);
      if ((err = launched("bwd_landmark_kernel", st)) != hipSuccess) return err;
      kv.dv_lm16 = b.dv_lm16;
      kv.lse_lm = b.lse_lm;
      kv.D_lm = b.D_lm;
      kv.inv_start = c.use_routed ? b.inv_start : nullptr;
      kv.inv_slot = c.use_routed ? b.inv_slot : nullptr;
      kv.dk_out = b.dk;
      kv.dv_out = b.dv;
      kv.dq_part = b.dk_acc;
      kv.nred = nch16;
      kv.ntotal = (c.N + KvTile<D, NG, 4>::KB - 1) / KvTile<D, NG, 4>::KB;
      const int nred_blocks = std::min(8, (c.M * D / 4 + 255) / 256);
      const unsigned nxl = (unsigned)((kv.ntotal + NXCD - 1) / NXCD * NXCD + nred_blocks);
      hipLaunchKernelGGL((bwd_kv16_kernel<D, KV_LMV, NG, 4>), dim3(nxl, bh), dim3(256), 0, st, kv);
      if ((err = launched("bwd_kv_landmark_kernel", st)) != hipSuccess) return err;
    } else {
      // (its atomic adds to the landmark rows come once per chunk)
      a.chunk = bwd_chunk(c, nlb, BWD_TK, BWD_CHUNK, 512);
      const int nch = (c.N + a.chunk - 1) / a.chunk;
      hipLaunchKernelGGL((bwd_kernel<T, D, BWD_LMV, true, false>), dim3((unsigned)(nlb * nch), bh), dim3(256), 0,
                         st, a);
      if ((err = launched("bwd_landmark_kernel", st)) != hipSuccess) return err;
    }
  }
  const int64_t rows = BH(c) * c.N;
  const int64_t threads = rows * FIN_TPR<D>;
  const dim3 fg((unsigned)((threads + 255) / 256));
  if (fused_finish)
    hipLaunchKernelGGL((bwd_finish_kernel<T, D, true, false>), fg, dim3(256), 0, st, b.dq_direct, b.dq_lm_acc,
                       b.dk_acc, b.dv_acc, (T *)b.dq, (T *)b.dk, (T *)b.dv, rows, c.N, c.M, c.grid_h, c.grid_w,
                       c.lm_h, c.lm_w);
  else if (c.use_shared)
    hipLaunchKernelGGL((bwd_finish_kernel<T, D, true>), fg, dim3(256), 0, st, b.dq_direct, b.dq_lm_acc, b.dk_acc,
                       b.dv_acc, (T *)b.dq, (T *)b.dk, (T *)b.dv, rows, c.N, c.M, c.grid_h, c.grid_w, c.lm_h, c.lm_w);
  else
    hipLaunchKernelGGL((bwd_finish_kernel<T, D, false>), fg, dim3(256), 0, st, b.dq_direct, b.dq_lm_acc, b.dk_acc,
                       b.dv_acc, (T *)b.dq, (T *)b.dk, (T *)b.dv, rows, c.N, c.M, c.grid_h, c.grid_w, c.lm_h, c.lm_w);
  return launched("bwd_finish_kernel", st);
}

hipError_t launch_scan_counts(const int32_t *cnt, int32_t *start, int n, int64_t bh, hipStream_t st) {
  hipLaunchKernelGGL(inv_scan_kernel, dim3((unsigned)bh), dim3(1024), 0, st, cnt, start, n);
  return launched("scan_counts_kernel", st);
}

hipError_t launch_backward(const mita_cfg_t &c, const BwdBufs &b, hipStream_t st) {
  if (c.dtype == MITA_F32) return c.d == 64 ? bwd_t<float, 64>(c, b, st) : bwd_t<float, 128>(c, b, st);
  return c.d == 64 ? bwd_t<bf16_t, 64>(c, b, st) : bwd_t<bf16_t, 128>(c, b, st);
}

}  // namespace mita
