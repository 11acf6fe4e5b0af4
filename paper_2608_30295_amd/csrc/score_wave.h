// Score passes of the prefill kernels for bf16 over long rows of keys (the
// others are in score.h, which also says what a pass computes).  What bounds them is the
// matrix core together with the softmax arithmetic (one fma, one exp2 and one
// add per score) and, up to 128 query rows, HBM; so nothing else may stand in
// the way of the three running side by side:
//  * The query rows of the KV head stay in LDS for the whole kernel; a wave
//    keeps its own 64 keys in registers (the next 64 in flight) and runs all
//    query rows over them.  No wave waits for another between the prologue
//    and the end, so one wave's MFMAs meet the other's arithmetic, and a key
//    fragment is loaded straight into the operand registers by the one wave
//    that uses it.
//  * S^T = K Q^T with v_mfma_f32_32x32x16_bf16 (keys as A, query rows as B):
//    a lane holds one query row (column of S^T) and 16 keys of a 32 x 32
//    tile, so a row's offset and sum are one register per 32 rows, and LDS
//    serves 16 KB of fragments per 64 x 64 scores, half the matrix core's
//    time at 128 bytes per cycle.
// Measured (5 heads, 256 rows, 131008 keys, 40 launches in a row): row
// statistics 57.0 -> 49-56 us, column mass 62.7 -> 49-57 us against 16 x 16
// tiles of a K tile shared by eight waves through an LDS ring (one barrier
// per 64 keys); both sums in one pass (kBoth) 60 us.  With all-zero inputs the
// same passes take 41 us: the matrix cores' clock under load is part of it.
#pragma once

#include "score.h"

namespace catekv {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kSwWaves = 8;                 // waves per workgroup, one workgroup per compute unit
constexpr int kSwThreads = kSwWaves * 64;
constexpr int kSwRow = 17;                  // 16-byte units per LDS query row (16 + 1: rows start in different banks)

// Row r of the score block is query i = r / G of group head g = r % G.
struct SwRow {
  int i, g;
};
__device__ __forceinline__ SwRow sw_row(int r, int g_log) { return {r >> g_log, r & ((1 << g_log) - 1)}; }

// kRowEst: the sum of exp2(s c) of every row over sampled keys, from which
// kBoth estimates it over all: the first 32 keys, which prompts often give
// most of a row's mass, as themselves, and 8160 others by steps of the golden
// ratio (single keys: neighbours score alike).  Workgroup `part` takes 256 of
// them, a wave 32; est[row][part] is the log2 sum of its keys, est[row][32]
// that of the first 32.
constexpr int kSwEstParts = 32, kSwEstStride = 36;
__device__ __forceinline__ uint32_t sw_est_key(int part, int wave, int n, int64_t n_keys) {
  const uint32_t u = (uint32_t)((part * kSwWaves + wave) * 32 + n);
  return u < 32 ? u : 32 + __umulhi(u * 2654435769u, (uint32_t)(n_keys - 32));
}
__device__ __forceinline__ float sw_log2_sum(const float* e, int cnt, const bool* in) {
  float M = kMInit, L = 0.f;
#pragma unroll
  for (int i = 0; i < cnt; ++i) M = in[i] ? fmaxf(M, e[i]) : M;
#pragma unroll
  for (int i = 0; i < cnt; ++i) L += in[i] ? fast_exp2(e[i] - M) : 0.f;
  return M + __log2f(L);
}
// The estimate (log2): of eight groups of 1024 samples the mean of the five
// smallest, so that a few very large terms in some groups do not lift it
// (rho = estimate / sum <= 1 costs nothing, rho >> 1 weakens the bound), and
// the first keys.  Some group has a sum at least the mean's, so rho is at most
// n_keys / 896.  Any finite number is a valid weight: sums that it takes out of
// range are redone.
__device__ __forceinline__ float sw_est_pick(const float4 (&e)[kSwEstStride / 4], int64_t n_keys) {
  constexpr int NG = 8, PER = kSwEstParts / NG;
  static_assert(PER == 4, "a group per load");
  const bool all[PER] = {true, true, true, true};
  float g[NG];
#pragma unroll
  for (int w = 0; w < NG; ++w) {
    const float p[PER] = {e[w].x, e[w].y, e[w].z, e[w].w};
    g[w] = sw_log2_sum(p, PER, all);
  }
  bool in[NG];
#pragma unroll
  for (int w = 0; w < NG; ++w) {
    int below = 0;
#pragma unroll
    for (int v = 0; v < NG; ++v) below += g[v] < g[w] || (g[v] == g[w] && v < w);
    in[w] = below < 5;
  }
  const float s[2] = {sw_log2_sum(g, NG, in) + __log2f((float)(n_keys - 32) * (1.0f / (5 * 32 * kSwWaves * PER))),
                      e[NG].x};
  const float pick = sw_log2_sum(s, 2, all);
  return fabsf(pick) < INFINITY ? pick : 0.f;
}

// key of accumulator register r within its 32-key tile
__device__ __forceinline__ constexpr int sw_key(int r) { return (r & 3) + 8 * (r >> 2); }

// RG 32-row tiles
template <int RG, int MODE>
__global__ __launch_bounds__(kSwThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void score_wave_kernel(ScoreArgs a) {
  constexpr int KS = 8;                     // 16-dim steps of the contraction
  __shared__ uint4 s_q[RG * 32 * kSwRow];
  // Row offsets (log2 units) and sums of exp2(s c - offset) lie in registers,
  // the row tiles unrolled; kBoth has none left for them: LDS, and the row
  // tiles are a loop (unrolled, the compiler spills).
  constexpr bool EST = MODE == kRowEst, RS = MODE == kRowStats || EST, BOTH = MODE == kBoth, SUMS = RS || BOTH;
  constexpr bool GATHER = MODE == kColGather;
  static_assert(RG <= 8, "at most 256 rows");
  __shared__ float s_woff[RS ? kSwWaves : 1][RS ? RG * 32 : 1];   // kRowStats: each wave's own offsets, at the end
  __shared__ float s_off[BOTH ? RG * 32 : 1];
  __shared__ float s_l[SUMS ? kSwWaves : 1][SUMS ? RG * 32 : 1];
  float off_r[BOTH ? 1 : RG], l_r[BOTH ? 1 : RG];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, half = lane >> 5;
  const int sel = blockIdx.y, cb = blockIdx.x;
  if (MODE == kColMass && a.gate && !a.gate[sel]) return;
  if (EST && cb == 0 && blockIdx.z == 0 && threadIdx.x == 0) a.rho[sel] = a.redo[sel] = 0;
  const int h = a.heads[sel];
  const int G = a.G;
  const int row0 = EST ? blockIdx.z * (RG * 32) : 0;                      // first query row

  // this wave's keys: a run of whole units of the block's key columns (32
  // keys, or 64 where a chunk spans 64)
  const int64_t col0 = (int64_t)cb * a.cb_tokens;
  const int n_cols = (int)(min(col0 + a.cb_tokens, a.n_keys) - col0);
  const int ul = a.unit_log;
  const int units = (n_cols + (1 << ul) - 1) >> ul;
  const int c_lo = (units * wave / kSwWaves) << ul;                       // first column, from col0
  const int c_hi = min((units * (wave + 1) / kSwWaves) << ul, n_cols);
  // query row i sees columns up to lim + i; columns below c_plain (a whole
  // number of units) need no mask: they lie before the end and at or before
  // every row's position
  const int lim = a.causal ? (int)max((int64_t)-(1 << 30), min((int64_t)(1 << 30), a.q_pos0 - a.key_off - col0)) : 1 << 30;
  const int c_plain = GATHER || EST ? c_lo : max(c_lo, min(c_hi, lim + 1) >> ul << ul);
  // A plain run starts and ends with a step of 32 keys and takes 64 at a time
  // between: all waves' first requests meet at the memory, and the matrix
  // cores idle until they are served, and the memory idles under the last
  // step.  Where a chunk spans 64 keys (column modes) every step is 64.
  const bool steps32 = (MODE != kColMass && !BOTH) || ul == 5;
  const int pu = (c_plain - c_lo) >> 5;                                   // plain keys, in 32s
  const int n_full = steps32 ? max(pu - 1, 0) >> 1 : pu >> 1;             // 64-key tiles
  const bool has_tail = steps32 && pu > 0 && !(pu & 1);                   // and a last step of 32
  const int c_full = steps32 ? c_lo + 32 : c_lo;                          // first column of the full tiles
  const char* kb = reinterpret_cast<const char*>(a.k) +
                   ((size_t)h * a.n + (size_t)(a.key_off + col0)) * (kD * 2);

  // ---- K fragments: tile t2 of 32 keys, step ks: 16 bytes of key row n ------
  const uint32_t voff = (uint32_t)n * (kD * 2) + (uint32_t)half * 16;
  uint4 kf[2][2][KS];
  // shares a tile is requested in (kBoth: two row tiles each, looped over)
  constexpr int kSlots = BOTH ? (RG < 2 ? 1 : RG / 2) : RG;
  // share `slot` of the 32 keys from column col, and of those `step` further (NF = 2), all valid, into f:
  // at least four 32-byte steps together, so that a request's 128-byte lines are used whole
  auto load_slot = [&](uint4 (&f)[2][KS], int col, auto nf_tag, int slot, int step = 32) {
    constexpr int TOT = decltype(nf_tag)::value * KS, NSH = kSlots < TOT / 4 ? kSlots : TOT / 4, PER = TOT / NSH;
    if (slot % (kSlots / NSH)) return;
    const char* p = kb + (size_t)col * (kD * 2);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = slot / (kSlots / NSH) * PER + u;
      f[x / KS][x % KS] = ldg16(p + (x / KS) * step * (kD * 2) + voff + (x % KS) * 32);
    }
  };
  auto load_all = [&](uint4 (&f)[2][KS], int col, auto nf_tag) {
#pragma unroll
    for (int s = 0; s < kSlots; ++s) load_slot(f, col, nf_tag, s);
  };
  auto load_clamped = [&](uint4 (&f)[2][KS], int col) {   // keys past the block's end re-read its last one
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const char* p = kb + (size_t)min(col + 32 * t + n, n_cols - 1) * (kD * 2) + half * 16;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) f[t][ks] = ldg16(p + ks * 32);
    }
  };

  // kBoth: the samples of a row's sum, one row per thread, picked from while
  // the query rows are on their way
  static_assert(!BOTH || RG * 32 <= kSwThreads, "one row per thread");
  float4 ev[BOTH ? kSwEstStride / 4 : 1];
  const SwRow er = sw_row(min((int)threadIdx.x, RG * 32 - 1), a.g_log);
  if constexpr (BOTH) {
    const float* e = a.est + ((size_t)sel * a.rp + min(er.i, a.lq - 1) * G + er.g) * kSwEstStride;
#pragma unroll
    for (int u = 0; u < kSwEstStride / 4; ++u) ev[u] = *reinterpret_cast<const float4*>(e + 4 * u);
    compiler_fence();
  }
  // The query rows go first and alone: requested beside the first keys of all
  // workgroups (16 MB) they wait behind them, 8-12 us instead of ~2.
  constexpr int QP = RG * 32 * 16 / kSwThreads;           // 16-byte pieces of query rows per thread
  uint4 qv[QP];
#pragma unroll
  for (int u = 0; u < QP; ++u) {
    const int e = u * kSwThreads + threadIdx.x;
    const SwRow q = sw_row(row0 + (e >> 4), a.g_log);
    const uint32_t row = (uint32_t)(h * G + q.g) * a.lq + min(q.i, a.lq - 1);
    qv[u] = ldg16(reinterpret_cast<const char*>(a.q) + (size_t)row * (kD * 2) + (e & 15) * 16);
  }
  // kColGather: 32 gathered keys from column col; past the block's end its last one again
  auto load_gathered = [&](uint4 (&f)[KS], int col) {
    const uint32_t x = min(col + n, n_cols - 1) + (uint32_t)col0, cs = (uint32_t)a.cand_cs;
    const int64_t key = min((int64_t)a.cand[(size_t)sel * a.n_cand + x / cs] * cs + x % cs, a.cand_keys - 1);
    const char* p = reinterpret_cast<const char*>(a.k) + ((size_t)h * a.n + (size_t)key) * (kD * 2) + half * 16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = ldg16(p + ks * 32);
  };
  if constexpr (EST) {
    const char* p = reinterpret_cast<const char*>(a.k) +
                    ((size_t)h * a.n + sw_est_key(cb, wave, n, a.n_keys)) * (kD * 2) + half * 16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[0][0][ks] = ldg16(p + ks * 32);
  }
  auto load_off = [&](int s) -> float {
    const SwRow q = sw_row(s, a.g_log);
    if (q.i >= a.lq) return INFINITY;
    return a.rowoff[(size_t)sel * a.rp + q.i * G + q.g];
  };
  if constexpr (BOTH) {
    for (int s = lane; s < RG * 32; s += 64) s_l[wave][s] = 0.f;
    if (threadIdx.x < RG * 32) s_off[threadIdx.x] = er.i < a.lq ? sw_est_pick(ev, a.n_keys) : INFINITY;
  } else {
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      off_r[rg] = RS ? kMInit : load_off(rg * 32 + n);
      l_r[rg] = 0.f;
    }
  }
#pragma unroll
  for (int u = 0; u < QP; ++u) {
    const int e = u * kSwThreads + threadIdx.x;
    const bool ok = sw_row(row0 + (e >> 4), a.g_log).i < a.lq;
    s_q[(e >> 4) * kSwRow + (e & 15)] = ok ? qv[u] : make_uint4(0, 0, 0, 0);
  }
  barrier_lds_only();
  using T1 = std::integral_constant<int, 1>;
  using T2 = std::integral_constant<int, 2>;
  using Y = std::true_type;
  using N = std::false_type;
  if (pu > 0) load_all(kf[1], c_lo, T1{});

  const uint4* qn = s_q + n * kSwRow + half;
  float cm[2][16];        // column modes: the lane's column sums of the tile
  const float c = a.c;

  auto mfma = [&](const uint4 (&f)[KS], const uint4 (&bf)[KS]) {
    floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f[ks]), __builtin_bit_cast(bf16x8, bf[ks]),
                                                    acc, 0, 0, 0);
    return acc;
  };
  // ---- end of a tile ---------------------------------------------------------
  // kColMass: sums over the 32 lanes of the 32 column sums a lane holds, each
  // lane left with one key's total: row swap, then mirror, half mirror, xor 2
  // and xor 1, halving the values each time.  Lane bits (5..0) then hold key
  // bits 2, 5, 4, 3, 1, 0.  keys: 32 or 64, the tile's; only theirs are stored.
  auto finish_cols = [&](int col, int keys) {
    float x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(cm[0][r]), __float_as_uint(cm[1][r]), false, false);
      x[r] = __uint_as_float(w[0]) + __uint_as_float(w[1]);
    }
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = (b3 ? x[r + 8] : x[r]) + dpp<kDppMirror>(b3 ? x[r] : x[r + 8]);
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = (b2 ? x[r + 4] : x[r]) + dpp<kDppHalfMirror>(b2 ? x[r] : x[r + 4]);
#pragma unroll
    for (int r = 0; r < 2; ++r) x[r] = (b1 ? x[r + 2] : x[r]) + dpp<kDppXor2>(b1 ? x[r] : x[r + 2]);
    float v = (b0 ? x[1] : x[0]) + dpp<kDppXor1>(b0 ? x[0] : x[1]);
    v *= 1.0f / (float)G;
    const int key = (lane & 3) | (half << 2) | ((lane & 12) << 1) | ((lane & 16) << 1);
    const int64_t kc = col0 + col + key;
    const bool ok = key < keys && col + key < c_hi;
    if (a.cs_fused > 0) {
      const int cs = a.cs_fused;
      float m = ok ? v : -INFINITY;
      if (cs >= 2) m = fmaxf(m, dpp<kDppXor1>(m));
      if (cs >= 4) m = fmaxf(m, dpp<kDppXor2>(m));
      if (cs >= 8) m = max_xor32(m);
      if (cs >= 16) m = fmaxf(m, dpp<kDppHalfMirror>(m));
      if (cs >= 32) m = fmaxf(m, dpp<kDppMirror>(m));
      if (cs >= 64) m = max_xor16(m);
      if (ok && (key & (cs - 1)) == 0) a.chunks[(size_t)sel * a.n_chunks + kc / cs] = m;
    } else if (ok) {
      a.colmass[(size_t)sel * a.n_keys + kc] = v;
    }
  };

  // ---- one tile: NT2 tiles of 32 keys from column col over all query rows ----
  // FIRST (row statistics): each row's offset is its maximum over the first 32
  // keys (kMInit for a row that sees none of them: it then sees none of the
  // run, as a row's visible keys form a prefix of the key range).  Later
  // terms are added against it with no running maximum: up to 2^128 they stay
  // finite; a sum that overflows is written as it is (inf), and the merge
  // recomputes that block's statistics exactly.
  // The phases of a row tile (MFMAs of 32 keys, their arithmetic) are kept
  // apart and in order: with two waves per SIMD one wave's MFMAs run beside
  // the other's arithmetic.  (The two interleaved inside a wave, one MFMA then
  // two scores, measured 25% slower.)  The next row tile's fragments are read
  // behind the last MFMAs that use the present ones.
  uint4 bf[KS];
  auto read_rows = [&](int rg) {
    compiler_fence();   // keeps the fragments of one row tile, not of all, in registers
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) bf[ks] = qn[rg * 32 * kSwRow + ks * 2];
    compiler_fence();
  };
  read_rows(0);
  // ahead(slot) requests a share of the next tile's keys: a wave that asks
  // for all 16 KB at once stands at the full memory pipeline instead of at its
  // MFMAs (3-5 us of 50 at the sizes above).
  auto tile = [&](uint4 (&f)[2][KS], int col, auto nt_tag, auto mask_tag, auto first_tag, auto&& ahead) {
    constexpr int NT2 = decltype(nt_tag)::value;
    constexpr bool MASK = decltype(mask_tag)::value, FIRST = decltype(first_tag)::value;
    auto rows = [&](int rg) {
      float off;
      if constexpr (BOTH) off = s_off[rg * 32 + n];
      else off = off_r[rg];
      int last = c_hi - 1 - col - 4 * half;               // MASK: last visible key of this lane's row in the tile
      if (MASK) last = min(last, lim + sw_row(rg * 32 + n, a.g_log).i - col - 4 * half);
      float ls = 0.f;
#pragma unroll
      for (int t = 0; t < NT2; ++t) {
        floatx16 acc = mfma(f[t], bf);
        __builtin_amdgcn_sched_barrier(0);
        if (t == NT2 - 1) read_rows((rg + 1) & (RG - 1));
        __builtin_amdgcn_sched_barrier(0);
        if (MASK && MODE != kColMass && !GATHER) {
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[r] = t * 32 + sw_key(r) <= last ? acc[r] : -INFINITY;
        }
        if constexpr (FIRST) if (t == 0) {
          float m = acc[0];
#pragma unroll
          for (int r = 1; r < 16; ++r) m = fmaxf(m, acc[r]);
          off = fmaxf(kMInit, max_xor32(m) * c);          // c > 0: the maximum of s c is c times that of s
          off_r[rg] = off;
        }
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(acc[r], c, -off));
        if (!RS) {
#pragma unroll
          for (int r = 0; r < 16; ++r) cm[t][r] = !BOTH && rg == 0 ? p[r] : cm[t][r] + p[r];
        }
        if (SUMS) {
#pragma unroll
          for (int s = 8; s > 0; s >>= 1)
#pragma unroll
            for (int r = 0; r < s; ++r) p[r] += p[r + s];
          ls += p[0];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (RS) {
        l_r[rg] += ls;
      } else if constexpr (BOTH) {
        ls = add_xor32(ls);                               // both halves hold the same row
        if (half == 0) atomicAdd(&s_l[wave][rg * 32 + n], ls);   // this wave's own word
      }
    };
    if (BOTH) {
#pragma unroll
      for (int t = 0; t < NT2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) cm[t][r] = 0.f;
    }
#pragma unroll
    for (int slot = 0; slot < kSlots; ++slot) {
      ahead(slot);
      if constexpr (!BOTH) {
        rows(slot);
      } else {
#pragma unroll 1
        for (int rg = slot * (RG / kSlots); rg < (slot + 1) * (RG / kSlots); ++rg) rows(rg);
      }
    }
    if (MODE == kColMass || BOTH || GATHER) {
      if (NT2 == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) cm[1][r] = 0.f;
      }
      finish_cols(col, NT2 * 32);
    }
  };
  // ---- the run: 32 keys, full tiles, 32 keys, then the masked rest -----------
  auto none = [](int) {};
  if (pu > 0) {
    // with no full tile: the first keys again, so that the loads in flight are the same on every path
    const int c1 = n_full > 0 ? c_full : c_lo, step1 = n_full > 0 ? 32 : 0;
    if (steps32)
      tile(kf[1], c_lo, T1{}, N{}, std::integral_constant<bool, RS>{}, [&](int s) { load_slot(kf[0], c1, T2{}, s, step1); });
    else
      load_all(kf[0], c1, T2{});
    int i = 0;
    for (; i + 2 < n_full; i += 2) {        // tile i in buffer 0; i + 1 and i + 2 exist
      const int col = c_full + 64 * i;
      tile(kf[0], col, T2{}, N{}, N{}, [&](int s) { load_slot(kf[1], col + 64, T2{}, s); });
      tile(kf[1], col + 64, T2{}, N{}, N{}, [&](int s) { load_slot(kf[0], col + 128, T2{}, s); });
    }
    if (i + 1 < n_full) {
      const int col = c_full + 64 * i;
      tile(kf[0], col, T2{}, N{}, N{}, [&](int s) { load_slot(kf[1], col + 64, T2{}, s); });
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[0][t][ks] = kf[1][t][ks];
      ++i;
    }
    // the last step of 32 (read, where there is none, for the same reason)
    if (i < n_full)
      tile(kf[0], c_full + 64 * i, T2{}, N{}, N{}, [&](int s) { load_slot(kf[1], c_plain - 32, T1{}, s); });
    else
      load_all(kf[1], c_plain - 32, T1{});
    if (has_tail) tile(kf[1], c_plain - 32, T1{}, N{}, N{}, none);
  }
  bool started = pu > 0;                    // kRowStats: offsets taken
  if constexpr (GATHER) {                   // 32 gathered keys at a time
    if (c_lo < c_hi) load_gathered(kf[0][0], c_lo);
    for (int col = c_lo; col < c_hi; col += 32) {
      if (col + 32 < c_hi) load_gathered(kf[1][0], col + 32);
      tile(kf[0], col, T1{}, N{}, N{}, none);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[0][0][ks] = kf[1][0][ks];
    }
    return;
  }
  if constexpr (EST) tile(kf[0], 0, T1{}, N{}, Y{}, none);
  for (int col = c_plain; !EST && col < c_hi; col += 64) {
    load_clamped(kf[0], col);
    if (RS && !started) {
      tile(kf[0], col, T2{}, Y{}, Y{}, none);
      started = true;
    } else {
      tile(kf[0], col, T2{}, Y{}, N{}, none);
    }
  }

  // ---- row sums: the lanes of a row, then the waves --------------------------
  if constexpr (SUMS) {
    if constexpr (RS) {
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        const float ls = add_xor32(l_r[rg]);              // both halves hold the same row and offset
        if (half == 0) {
          s_woff[wave][rg * 32 + n] = off_r[rg];
          s_l[wave][rg * 32 + n] = ls;
        }
      }
    }
    __syncthreads();
    for (int s = threadIdx.x; s < RG * 32; s += kSwThreads) {
      const SwRow q = sw_row(row0 + s, a.g_log);
      if (q.i >= a.lq) continue;
      float M = kMInit, L = 0.f;
      if constexpr (RS) {
        float2 v[kSwWaves];
#pragma unroll
        for (int w = 0; w < kSwWaves; ++w) v[w] = make_float2(s_woff[w][s], s_l[w][s]);
        if (EST && cb == 0) {                             // the first 32 keys apart, seven waves for eight
          a.est[((size_t)sel * a.rp + q.i * G + q.g) * kSwEstStride + kSwEstParts] = v[0].x + __log2f(v[0].y);
          v[0] = make_float2(kMInit, 0.f);
        }
#pragma unroll
        for (int w = 0; w < kSwWaves; ++w) M = fmaxf(M, v[w].x);
#pragma unroll
        for (int w = 0; w < kSwWaves; ++w) L += v[w].y * fast_exp2(v[w].x - M);
      } else {                                            // the same offset in every wave
        M = s_off[s];
#pragma unroll
        for (int w = 0; w < kSwWaves; ++w) L += s_l[w][s];
      }
      if constexpr (EST)
        a.est[((size_t)sel * a.rp + q.i * G + q.g) * kSwEstStride + cb] = M + __log2f(cb == 0 ? L * (8.f / 7.f) : L);
      else
        a.rowpart[((size_t)sel * a.n_colblk + cb) * a.rp + q.i * G + q.g] = make_float2(M, L);
    }
  }
}

// 32-row tiles (1, 2, 4 or 8) for up to 256 rows
inline int sw_row_tiles(int rows) {
  int rg = 1;
  while (rg * 32 < rows) rg *= 2;
  return rg;
}

template <int MODE>
inline hipError_t launch_score_wave(dim3 grid, hipStream_t s, ScoreArgs a) {
  if (MODE == kRowStats || MODE == kRowEst) a.unit_log = 5;
  a.g_log = __builtin_ctz((unsigned)a.G);
#define CATEKV_SW(RG) \
  if (rg == RG) { hipLaunchKernelGGL((score_wave_kernel<RG, MODE>), grid, dim3(kSwThreads), 0, s, a); return hipGetLastError(); }
  const int rg = sw_row_tiles(a.R) / (int)grid.z;
  CATEKV_SW(1) CATEKV_SW(2) CATEKV_SW(4) CATEKV_SW(8)
#undef CATEKV_SW
  return hipErrorInvalidValue;
}

}  // namespace catekv
