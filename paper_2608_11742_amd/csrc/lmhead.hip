// LM head fused with the per-position vocabulary statistics the scheduler
// needs (entropy, log-sum-exp, max logit, argmax, top-K).  The [R][V] logits
// never leave the chip.
//
// Pass 1 (lmhead_kernel): a workgroup owns a tile of hidden rows and one
// slice of the vocabulary.  For each vocabulary tile it runs the MFMA
// mainloop, scales the logits, stages them as fp32 in LDS and lets 2 or 4
// threads per row scan 32 or 64 logits each, updating a running max m,
// s = sum exp(l - m), t = sum exp(l - m) (l - m) (m and t in log2 units
// while scanning, natural units in the partials) and a sorted top-16.  At
// the end of its slice every thread writes its partial state.
// Pass 2 (merge_kernel): one workgroup per row merges all partials:
//   M = max m_p, S = sum s_p e^(m_p - M), T = sum e^(m_p - M) (t_p + (m_p - M) s_p)
//   lse = M + log S, H = log S - T / S, lmax = M,
// and the top 16 of the partials' lists: the entries no worse than a bound
// that 16 of the lists' heads reach, sorted.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "mainloop.h"

namespace dllm {

namespace {

constexpr int kK = DLLM_TOPK_REG;
// Workgroups of a launch: one per CU (the 256-row tile's LDS holds one), each
// walking its vocabulary slice.  Two rounds of half-length slices measured
// 4-6% slower at 512 and 4096 rows: every slice pays its first tile, where
// the empty top-16 lists make many logits candidates, and the merge folds
// twice the partials.
// The small tile's workgroups hold 48 KB of LDS and 172 registers a thread, so
// two run on a CU, and one streams its weights while the other scans.
constexpr int kTargetWg = 256, kTargetWgSmall = 512;
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;

// Tiles of BM rows by COLS vocabulary entries: 256 x 256 (8 waves of 64 x 128,
// the projection GEMMs' tile), 128 x 256 (8 waves of 64 x 64) and 64 x 128 (4
// waves of 32 x 64); lm_tile picks one.
// kSegs scan threads per row, each scanning kSegCols logits per pass; a pass
// stages kSegs * kSegCols columns of the fp32 logit tile in LDS.
// The MFMA blocks are computed transposed (TRANS), so that a lane holds 4
// consecutive logits of one row and stages them with one 16-byte LDS write;
// bf16 256-row tiles take the two-group mainloop of the projections; the
// smaller ones (few rows: the vocabulary streams from HBM) the early-release
// TileMma schedule.
template <typename T, int BM_>
struct LmCfg {
  using Type = T;
  static constexpr int BM = BM_;
  static constexpr int kCols = BM == 64 ? 128 : 256;         // vocabulary tile
  static constexpr int kThreads = BM == 64 ? 256 : 512;
  static constexpr int kMinBlocks = BM == 64 ? 2 : 1;
  static constexpr int kWavesM = BM == 256 ? 4 : 2, kWavesN = BM == 128 ? 4 : 2;
  using TM = std::conditional_t<BM == 256 && std::is_same_v<T, bf16_t>, PingPongMma<T, true>,
                                TileMma<T, BM, kCols, kWavesM, kWavesN, true, BM != 256>>;
  static constexpr int kSegs = kThreads / BM;
  static constexpr int kSegCols = BM == 64 ? 32 : 64;        // logits per scan thread per pass
  static constexpr int kSegStride = kSegCols * 4 + 16;       // padded segment bytes
  static constexpr int kPassCols = kSegs * kSegCols;
  static constexpr int kPasses = kCols / kPassCols;
  static constexpr int kRowStride = kSegs * kSegStride + 16;   // padded row bytes
  static constexpr int kStageBytes = BM * kRowStride;
  static constexpr int kSmem = TM::kSmem > kStageBytes ? TM::kSmem : kStageBytes;
  static constexpr int kBoundRank = kK / kSegs - 1;            // see the pruning bound below
  static_assert(kPasses == 1 || kPassCols == TM::kWTN, "a pass is the whole tile or one wave column");
  static_assert(kSegs * (kSegCols / 8) >= kK, "the seed bound covers the top 16");
};

// Tile times of a launch with n vocabulary slices: rounds of workgroups times
// the tiles of a slice.
int tile_times(int bm, int R, int V, int n) {
  return cdiv(cdiv(R, bm) * n, bm == 64 ? kTargetWgSmall : kTargetWg) * cdiv(cdiv(V, bm == 64 ? 128 : 256), n);
}

// Vocabulary slices: as many as one round of workgroups holds, or one more
// where rounding up needs fewer tile times over all rounds.
int slices_for(int bm, int R, int V) {
  const int rt = cdiv(R, bm), vt = cdiv(V, bm == 64 ? 128 : 256), target = bm == 64 ? kTargetWgSmall : kTargetWg;
  const int up = std::max(1, std::min(vt, cdiv(target, rt))), down = std::max(1, std::min(vt, target / rt));
  return tile_times(bm, R, V, up) < tile_times(bm, R, V, down) ? up : down;
}

// Row tile of an LM head over R rows and V vocabulary entries.
int lm_tile(int dtype, int R, int V) {
  // 2 partials a row and slice instead of 4; first, so that the products of
  // tile counts below stay within int
  if (R > 32768) return 256;
  const bool few = cdiv(R, 128) * cdiv(V, 256) < kTargetWg / 2;   // 128 x 256 tiles would leave half the CUs idle
  if (R <= 64 || few) return 64;
  if (R <= 128) return 128;
  const int t128 = tile_times(128, R, V, slices_for(128, R, V));
  // the fp32 matrix cores bound every tile: two 64 x 128 ones share a CU, so
  // each takes half the time of a 128 x 256 one (352 rows, vocabulary 32000: 3
  // against 2 tile times, 252 against 317 us; 512 rows: 4 against 2, 320 both)
  if (!dtype) return tile_times(64, R, V, slices_for(64, R, V)) < 2 * t128 ? 64 : 128;
  // d 4096: a 128 x 256 tile takes about 73 us, a 256 x 256 tile 1.72 times
  // that (352 rows, vocabulary 126464: 6 against 4 tile times, 472 against
  // 537 us; 512 rows: 8 against 4, 602 against 554)
  const int t256 = tile_times(256, R, V, slices_for(256, R, V));
  return 100 * t128 < 172 * t256 ? 128 : 256;
}

struct Partials {
  float* m;
  float* s;
  float* t;
  float* tv;     // [R][P][16]
  int32_t* ti;   // [R][P][16]
  int P;
};

__device__ __forceinline__ void topk_insert(float (&tv)[kK], int (&ti)[kK], float v, int id) {
  float cv = v;
  int ci = id;
#pragma unroll
  for (int k = 0; k < kK; ++k) {
    const bool gt = better(cv, ci, tv[k], ti[k]);
    const float ov = tv[k];
    const int oi = ti[k];
    tv[k] = gt ? cv : ov;
    ti[k] = gt ? ci : oi;
    cv = gt ? ov : cv;
    ci = gt ? oi : ci;
  }
}

template <typename T, int BM>
__global__ __launch_bounds__((LmCfg<T, BM>::kThreads), (LmCfg<T, BM>::kMinBlocks)) void lmhead_kernel(
    const T* __restrict__ Hs, const T* __restrict__ W, int R,
                                                             int d, int V, const float* __restrict__ row_scale,
                                                             const int32_t* __restrict__ rs_idx, int rs_n, int rs_lim,
                                                             float scale, int mask_id, int row_tiles,
                                                             int n_slices,
                                                             int vtiles, Partials part) {
  using Cfg = LmCfg<T, BM>;
  using TM = typename Cfg::TM;
  constexpr int kSegs = Cfg::kSegs, kRowStride = Cfg::kRowStride, kCols = Cfg::kCols;
  constexpr int kSegCols = Cfg::kSegCols, kSegStride = Cfg::kSegStride;
  __shared__ __attribute__((aligned(16))) uint8_t smem[Cfg::kSmem];

  // XCD-contiguous ids, walked in groups of 8 row tiles: the 32 workgroups an
  // XCD runs at a time cover 8 row tiles x 4 vocabulary slices, so each step
  // of their vocabulary loops fetches 12 operand panels into that XCD's L2
  // (16 row tiles x 2 slices would fetch 18)
  int rt, slice;
  map_tile(blockIdx.x, gridDim.x, row_tiles, n_slices, 8, rt, slice);
  const int t_begin = int((long long)slice * vtiles / n_slices);
  const int t_end = int((long long)(slice + 1) * vtiles / n_slices);
  const int m0 = rt * BM;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kWavesN = kCols / TM::kWTN;
  const int wm = wave / kWavesN, wn = wave % kWavesN;
  // scan role: row tid / kSegs, segment tid % kSegs
  const int srow = tid / kSegs, sseg = tid % kSegs;
  float m = -INFINITY, s = 0.f, t = 0.f;
  // This thread's sorted top 16.  With 256-row tiles the mainloop needs
  // nearly every register, so between tiles the list lives in the thread's
  // partials slot of the workspace (loaded before the scan, stored after it);
  // with 128-row tiles it stays in registers.
  constexpr bool kListInMemory = BM == 256;
  const int row = m0 + srow;
  const bool own_row = row < R;   // rows past R scan clamped copies and are discarded
  size_t slot = size_t(min(row, R - 1)) * part.P + size_t(slice) * kSegs + sseg;
  float tv[kK];
  int ti[kK];
#pragma unroll
  for (int k = 0; k < kK; ++k) { tv[k] = -INFINITY; ti[k] = 0x7fffffff; }
  // Pruning bound of the row, shared by its kSegs scan threads: the worst
  // (by value, then id) of their (16 / kSegs)-th best entries.  Each thread
  // holds 16 / kSegs entries at least as good as that, so at least 16
  // entries of the row are at least as good as the bound, and a logit that
  // is not strictly better cannot reach the row's top 16.  It rises about as
  // fast as the row's 16th best over all its segments, kSegs times faster
  // than a thread's own 16th best, which keeps the (wave-divergent)
  // insertions rare.
  float bv = -INFINITY;
  int bi = 0x7fffffff;

  // logit scale of this thread's scan row
  const int srow_c = min(row, R - 1);
  auto row_logit_scale = [&]() {
    return scale *
           (row_scale ? row_scale[rs_idx ? min(max(rs_idx[srow_c % rs_n], 0), rs_lim - 1) : srow_c % rs_n] : 1.0f);
  };
  float rs_row = row_logit_scale();

  // the bound from the kSegs threads of this row (consecutive lanes)
  auto refresh_bound = [&]() {
    float v = tv[Cfg::kBoundRank];
    int i = ti[Cfg::kBoundRank];
#pragma unroll
    for (int x = 1; x < kSegs; x <<= 1) {
      const float ov = __shfl_xor(v, x, 64);
      const int oi = __shfl_xor(i, x, 64);
      if (better(v, i, ov, oi)) { v = ov; i = oi; }
    }
    bv = v;
    bi = i;
  };

  const uint32_t row_bytes = uint32_t(d) * sizeof(T);
  for (int vt = t_begin; vt < t_end; ++vt) {
    // opaque per tile: keeps the compiler from hoisting the slot addresses
    // out of the tile loop, where they would stay live across the mainloop
    if constexpr (kListInMemory) asm volatile("" : "+v"(slot));
    const int n0 = vt * kCols;
    auto a_off = [&](int r) -> uint32_t { return uint32_t(min(m0 + r, R - 1)) * row_bytes; };
    auto b_off = [&](int r) -> uint32_t { return uint32_t(min(n0 + r, V - 1)) * row_bytes; };
    f32x4 acc[TM::kFM][TM::kFN];
    TM::run(smem, reinterpret_cast<const uint8_t*>(Hs), reinterpret_cast<const uint8_t*>(W), a_off, b_off,
            d / TM::kKPerStage, acc);
    if constexpr (kListInMemory) {
      if (vt > t_begin && own_row) {
        m = part.m[slot] * kLog2e;   // log2 units while scanning
        s = part.s[slot];
        t = part.t[slot] * kLog2e;
#pragma unroll
        for (int k = 0; k < kK; ++k) {
          tv[k] = part.tv[slot * kK + k];
          ti[k] = part.ti[slot * kK + k];
        }
      } else {
        m = -INFINITY;
        s = t = 0.f;
#pragma unroll
        for (int k = 0; k < kK; ++k) { tv[k] = -INFINITY; ti[k] = 0x7fffffff; }
      }
      refresh_bound();
      rs_row = row_logit_scale();
    }
#pragma unroll
    for (int pass = 0; pass < Cfg::kPasses; ++pass) {
    // stage this pass's scaled logits: LDS row r, pass column c at
    // r * kRowStride + (c / kSegCols) * kSegStride + (c % kSegCols) * 4
    if (Cfg::kPasses == 1 || wn == pass) {
#pragma unroll
      for (int mi = 0; mi < TM::kFM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TM::kFN; ++ni) {
          // (transposed blocks) row 16 mi + lane % 16, columns 16 ni + 4 (lane / 16) + 0..3
          const int r = wm * TM::kWTM + mi * 16 + (lane & 15);
          const unsigned c = wn * TM::kWTN + ni * 16 + 4 * (lane >> 4) - pass * Cfg::kPassCols;   // >= 0
          *reinterpret_cast<f32x4*>(smem + r * kRowStride + (c / kSegCols) * kSegStride + (c % kSegCols) * 4) =
              acc[mi][ni];
        }
    }
    __syncthreads();
    // scan kSegCols logits of row srow: running statistics, and a bit mask of the
    // logits that may beat the pruning bound (candidates for the top 16)
    const uint8_t* base = smem + srow * kRowStride + sseg * kSegStride;
    const int c0 = n0 + pass * Cfg::kPassCols + sseg * kSegCols;
    const bool all_ok = c0 + kSegCols <= V && (mask_id < c0 || mask_id >= c0 + kSegCols);
    if (vt == t_begin && pass == 0) {
      // The slice's top-16 lists are still empty, which would make every
      // logit a candidate.  Seed the bound instead: each thread takes the
      // smallest of the maxima of its groups of 8 logits (as many logits are at
      // least that large), the row the smallest over its kSegs threads, so at
      // least 16 logits of the row are at least as large as the bound and no
      // smaller logit can reach the row's top 16.
      float seed = INFINITY;
#pragma unroll
      for (int g8 = 0; g8 < kSegCols; g8 += 8) {
        float gm = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int col = c0 + g8 + e;
          const float v = *reinterpret_cast<const float*>(base + (g8 + e) * 4) * rs_row;
          if (all_ok || (col < V && col != mask_id)) gm = fmaxf(gm, v);
        }
        seed = fminf(seed, gm);
      }
#pragma unroll
      for (int x = 1; x < kSegs; x <<= 1) seed = fminf(seed, __shfl_xor(seed, x, 64));
      if (better(seed, 0x7fffffff, bv, bi)) {   // only ever raises the bound
        bv = seed;
        bi = 0x7fffffff;
      }
    }
    uint64_t cand = 0;
    if (__all(all_ok)) {
      // Every logit of the wave's segments is valid: branch-free scan in
      // log2 units (x = logit * log2 e): one FMA, one exp2 and one FMA per
      // logit; the reference max moves by selects.  Candidates are the
      // logits with x at least the bound in log2 units less a relative
      // 1e-6 (x and the bound round differently, by a few ulp at most), a
      // superset of those that beat the bound; the insertion below checks
      // each one exactly.
      const float c2 = rs_row * kLog2e;
      const float b2 = bv * kLog2e;
      const float bv2 = own_row ? b2 - fabsf(b2) * 1e-6f : INFINITY;
#pragma unroll
      for (int c4 = 0; c4 < kSegCols; c4 += 4) {
        const float4 v4 = *reinterpret_cast<const float4*>(base + c4 * 4);
        const float x[4] = {v4.x * c2, v4.y * c2, v4.z * c2, v4.w * c2};
        const float gmax = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
        const float mnew = fmaxf(m, gmax);
        const float alpha = __builtin_amdgcn_exp2f(m - mnew);   // 1 if unchanged, 0 from -inf
        const float d = alpha == 0.f ? 0.f : m - mnew;
        t = alpha * (t + d * s);
        s = alpha * s;
        m = mnew;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float y = x[e] - m;
          const float ex = __builtin_amdgcn_exp2f(y);
          s += ex;
          t = fmaf(ex, y, t);
          cand |= uint64_t(x[e] >= bv2) << (c4 + e);
        }
      }
    } else {
#pragma unroll
    for (int c4 = 0; c4 < kSegCols; c4 += 4) {
      const float4 v4 = *reinterpret_cast<const float4*>(base + c4 * 4);
      const float vv[4] = {v4.x * rs_row, v4.y * rs_row, v4.z * rs_row, v4.w * rs_row};
      bool ok[4];
      float cmax = -INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int col = c0 + c4 + e;
        ok[e] = all_ok || (col < V && col != mask_id);
        if (ok[e]) cmax = fmaxf(cmax, vv[e] * kLog2e);
      }
      if (cmax > m) {  // rescale the running sums to the new max (log2 units)
        if (m > -INFINITY) {
          const float alpha = __builtin_amdgcn_exp2f(m - cmax);
          t = alpha * (t + (m - cmax) * s);
          s = alpha * s;
        }
        m = cmax;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!ok[e]) continue;
        const float x = vv[e] * kLog2e - m;
        const float ex = __builtin_amdgcn_exp2f(x);
        s += ex;
        t += ex * x;
        if (own_row && better(vv[e], c0 + c4 + e, bv, bi)) cand |= uint64_t(1) << (c4 + e);
      }
    }
    }
    // insert the candidates; the wave loops as often as its busiest lane has candidates
    while (__any(cand != 0)) {
      if (cand) {
        const int pos = __builtin_ctzll(cand);
        cand &= cand - 1;
        const float v = *reinterpret_cast<const float*>(base + pos * 4) * rs_row;
        if (better(v, c0 + pos, tv[kK - 1], ti[kK - 1])) topk_insert(tv, ti, v, c0 + pos);
      }
    }
    // the next pass prunes with the bound these insertions raised
    if (pass + 1 < Cfg::kPasses) refresh_bound();
    __syncthreads();
    }
    if constexpr (!kListInMemory) refresh_bound();
    const bool last = vt + 1 == t_end;
    if (own_row && (kListInMemory || last)) {
      part.m[slot] = m * kLn2;   // natural units in the partials
      part.s[slot] = s;
      part.t[slot] = t * kLn2;
#pragma unroll
      for (int k = 0; k < kK; ++k) {
        part.tv[slot * kK + k] = tv[k];
        part.ti[slot * kK + k] = ti[k];
      }
    }
  }
}

// Sort the 64 lanes' (value, id) pairs by better(), best in lane 0.
__device__ __forceinline__ void wave_sort(float& v, int& i) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int size = 2; size <= 64; size <<= 1)
#pragma unroll
    for (int d = size >> 1; d > 0; d >>= 1) {
      const float w = __shfl_xor(v, d, 64);
      const int j = __shfl_xor(i, d, 64);
      // lanes of even blocks of `size` sort best first, odd ones best last
      const bool keep_better = ((lane & size) == 0) == ((lane & d) == 0);
      const bool other = better(w, j, v, i) == keep_better;
      if (other && (w != v || j != i)) { v = w; i = j; }
    }
}

// One workgroup of W = blockDim.x / 64 waves per row (W grows with the number
// of partials).  The row's top 16 lie in few of its partials' sorted lists:
// the waves sort their lanes' best list heads, and then the best 16 of every
// wave; the 16th is a bound that at least 16 logits of the row reach, so only
// the entries no worse than it are candidates (some 30 of P * 16).  They are
// gathered in LDS and wave 0 sorts them, 48 at a time behind the best 16 so far.
// Latency bound.  Folding every list into a per-lane top 16 took 44 us for 32
// rows of 1024 partials and 64 us for 2048; a bound per wave instead of per row
// 23 us for 2048 (some 300 candidates, sorted one 48 after the other); ranking
// by counting instead of sorting 28 us; contiguous copies of the list heads and
// merging the lists of a row's scan threads in pass 1 gained nothing.
__global__ __launch_bounds__(512) void merge_kernel(Partials part, int R, StatsOut out) {
  constexpr int kMaxW = 8, kCap = 1024;
  __shared__ float red_m[kMaxW], red_s[kMaxW], red_t[kMaxW], top_v[kMaxW * kK];
  __shared__ int top_i[kMaxW * kK];
  __shared__ float cv[kCap];
  __shared__ int ci[kCap];
  __shared__ int n_cand;
  const int row = blockIdx.x;
  const int W = blockDim.x >> 6, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (row >= R) return;
  const size_t base = size_t(row) * part.P;
  // this thread's partials: their maximum and their best list head
  float M = -INFINITY, hv = -INFINITY;
  int hi = 0x7fffffff;
  for (int p = threadIdx.x; p < part.P; p += blockDim.x) {
    M = fmaxf(M, part.m[base + p]);
    const float v = part.tv[(base + p) * kK];
    const int i = part.ti[(base + p) * kK];
    if (better(v, i, hv, hi)) { hv = v; hi = i; }
  }
  M = wave_max(M);
  wave_sort(hv, hi);
  if (lane < kK) { top_v[wave * kK + lane] = hv; top_i[wave * kK + lane] = hi; }
  if (lane == 0) red_m[wave] = M;
  if (threadIdx.x == 0) n_cand = 0;
  __syncthreads();
  M = red_m[0];
  for (int w = 1; w < W; ++w) M = fmaxf(M, red_m[w]);
  if (W > 1) {   // every wave: the better of the waves' heads l and l + 64 in lane l, sorted
    const int e2 = lane + 64;
    hv = lane < W * kK ? top_v[lane] : -INFINITY;
    hi = lane < W * kK ? top_i[lane] : 0x7fffffff;
    if (e2 < W * kK && better(top_v[e2], top_i[e2], hv, hi)) { hv = top_v[e2]; hi = top_i[e2]; }
    wave_sort(hv, hi);
  }
  const float bv = __shfl(hv, kK - 1, 64);
  const int bi = __shfl(hi, kK - 1, 64);
  float S = 0.f, Tt = 0.f;
  for (int p = threadIdx.x; p < part.P; p += blockDim.x) {
    const float mp = part.m[base + p];
    if (mp == -INFINITY) continue;  // a partial that saw no valid logit
    const float w = fast_exp(mp - M);
    const float sp = part.s[base + p];
    S += w * sp;
    Tt += w * (part.t[base + p] + (mp - M) * sp);
    const float* pv = part.tv + (base + p) * kK;
    const int32_t* pi = part.ti + (base + p) * kK;
    for (int k = 0; k < kK; ++k) {   // sorted: the first entry below the bound ends the list
      const float v = pv[k];
      const int i = pi[k];
      if (i == 0x7fffffff || better(bv, bi, v, i)) break;
      const int at = atomicAdd(&n_cand, 1);
      if (at < kCap) { cv[at] = v; ci[at] = i; }
    }
  }
  S = wave_sum(S);
  Tt = wave_sum(Tt);
  if (lane == 0) { red_s[wave] = S; red_t[wave] = Tt; }
  __syncthreads();
  if (wave != 0) return;
  S = red_s[0];
  Tt = red_t[0];
  for (int w = 1; w < W; ++w) { S += red_s[w]; Tt += red_t[w]; }
  // Sort the candidates: the ids are unique, so the order does not depend on
  // how they were gathered.  Or sort every entry, where the candidates
  // overflow the buffer: with more than four waves the bound is the 16th best
  // of pairs of heads, so up to 31 threads' lists can reach it, and past 1024
  // partials a thread has up to four lists of 16.
  const bool all = n_cand > kCap;
  const int n = all ? part.P * kK : n_cand;
  auto entry = [&](int e, float& v, int& i) {
    v = e >= n ? -INFINITY : all ? part.tv[base * kK + e] : cv[e];
    i = e >= n ? 0x7fffffff : all ? part.ti[base * kK + e] : ci[e];
  };
  float v;
  int i;
  entry(lane, v, i);
  wave_sort(v, i);
  for (int e = 64; e < n; e += 64 - kK) {
    if (lane >= kK) entry(e + lane - kK, v, i);
    wave_sort(v, i);
  }
  if (lane < out.k) {
    out.topk_id[size_t(row) * out.k + lane] = i;
    out.topk_logit[size_t(row) * out.k + lane] = v;
  }
  if (lane == 0) {
    out.argmax[row] = i;
    const float logS = logf(S);
    out.lmax[row] = M;
    out.lse[row] = M + logS;
    out.H[row] = logS - Tt / S;
  }
}

// one workgroup per probed logit (a wave each took 31 us at d 4096)
template <typename T>
__global__ __launch_bounds__(256) void probe_kernel(const T* __restrict__ Hs, const T* __restrict__ W, int d, int V,
                                                    int R, const int32_t* __restrict__ row,
                                                    const int32_t* __restrict__ tok, int n,
                                                    const float* __restrict__ row_scale,
                                                    const int32_t* __restrict__ rs_idx, int n_pos, int rs_lim,
                                                    float scale, float* __restrict__ out) {
  __shared__ float part[4];
  const int p = blockIdx.x;
  const int r = min(max(row[p], 0), R - 1);
  const T* h = Hs + size_t(r) * d;
  const T* w = W + size_t(min(max(tok[p], 0), V - 1)) * d;
  float acc = 0.f;
#pragma unroll 8
  for (int c = threadIdx.x; c < d; c += 256) acc += load_f(h + c) * load_f(w + c);
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  acc = part[0] + part[1] + part[2] + part[3];
  if (threadIdx.x == 0) out[p] = acc * scale * (row_scale ? row_scale[rs_idx ? min(max(rs_idx[r % n_pos], 0), rs_lim - 1) : r % n_pos] : 1.0f);
}

int partials_per_row(int bm, int R, int V) { return slices_for(bm, R, V) * (bm == 256 ? 2 : 4); }
static_assert(LmCfg<bf16_t, 256>::kSegs == 2 && LmCfg<bf16_t, 128>::kSegs == 4 && LmCfg<bf16_t, 64>::kSegs == 4,
              "partials_per_row");

Partials carve(void* ws, int R, int P) {
  Partials pt;
  uint8_t* p = static_cast<uint8_t*>(ws);
  const size_t n = size_t(R) * P;
  pt.m = reinterpret_cast<float*>(p);
  pt.s = pt.m + n;
  pt.t = pt.s + n;
  pt.tv = pt.t + n;
  pt.ti = reinterpret_cast<int32_t*>(pt.tv + n * kK);
  pt.P = P;
  return pt;
}

}  // namespace

size_t lmhead_workspace(int dtype, int R, int V) {
  return size_t(R) * partials_per_row(lm_tile(dtype, R, V), R, V) * (3 + 2 * kK) * 4 + 256;
}

hipError_t lmhead_partials(int dtype, const void* h, const void* w, int R, int d, int V, const float* row_scale,
                           const int32_t* rs_idx, int rs_n, int rs_lim, float scale, int mask_id, void* ws,
                           hipStream_t s) {
  if (d <= 0 || d % (dtype ? 64 : 32)) return hipErrorInvalidValue;   // the mainloop runs stages in pairs
  const int bm = lm_tile(dtype, R, V);
  auto go = [&](auto cfg, auto kern) {
    using Cfg = decltype(cfg);
    using T = typename Cfg::Type;
    const int ns = slices_for(bm, R, V), rt = cdiv(R, bm), vt = cdiv(V, Cfg::kCols);
    const Partials part = carve(ws, R, partials_per_row(bm, R, V));
    hipLaunchKernelGGL(kern, dim3(rt * ns), dim3(Cfg::kThreads), 0, s, static_cast<const T*>(h),
                       static_cast<const T*>(w), R, d, V, row_scale, rs_idx, rs_n, rs_lim, scale, mask_id, rt, ns, vt,
                       part);
  };
  if (dtype) {
    if (bm == 256) go(LmCfg<bf16_t, 256>{}, lmhead_kernel<bf16_t, 256>);
    else if (bm == 128) go(LmCfg<bf16_t, 128>{}, lmhead_kernel<bf16_t, 128>);
    else go(LmCfg<bf16_t, 64>{}, lmhead_kernel<bf16_t, 64>);
  } else {
    if (bm == 256) go(LmCfg<float, 256>{}, lmhead_kernel<float, 256>);
    else if (bm == 128) go(LmCfg<float, 128>{}, lmhead_kernel<float, 128>);
    else go(LmCfg<float, 64>{}, lmhead_kernel<float, 64>);
  }
  return hipGetLastError();
}

hipError_t lmhead_merge(int dtype, int R, int V, const StatsOut& out, void* ws, hipStream_t s) {
  const int bm = lm_tile(dtype, R, V);
  const Partials part = carve(ws, R, partials_per_row(bm, R, V));
  const int waves = std::min(8, std::max(1, cdiv(part.P, 128)));
  hipLaunchKernelGGL(merge_kernel, dim3(R), dim3(64 * waves), 0, s, part, R, out);
  return hipGetLastError();
}

hipError_t probe_logits(int dtype, const void* h, const void* w, int d, int V, int R, const int32_t* row,
                        const int32_t* tok, int n, const float* row_scale, const int32_t* rs_idx, int n_pos,
                        int rs_lim, float scale, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (dtype)
    hipLaunchKernelGGL(probe_kernel<bf16_t>, dim3(n), dim3(256), 0, s, static_cast<const bf16_t*>(h),
                       static_cast<const bf16_t*>(w), d, V, R, row, tok, n, row_scale, rs_idx, n_pos, rs_lim, scale, out);
  else
    hipLaunchKernelGGL(probe_kernel<float>, dim3(n), dim3(256), 0, s, static_cast<const float*>(h),
                       static_cast<const float*>(w), d, V, R, row, tok, n, row_scale, rs_idx, n_pos, rs_lim, scale, out);
  return hipGetLastError();
}

}  // namespace dllm
