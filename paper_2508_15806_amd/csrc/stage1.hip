// Stage 1 of SurfaceLogicKV (Section 3.2, Algorithm 1) on gfx950: for every attention row,
// the top-K set by radix select and the four weight cells; then a fixed-order reduction over
// the rows of each head and the SF / LG / INF scores.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>
#include <type_traits>

#include "device_utils.h"
#include "launch.h"
#include "slkv_internal.h"

namespace slkv {

constexpr int kS1Threads = 256;   // workgroup of the general row path
constexpr int kS1TopK = 64;       // largest K of the resident row path

// LDS of the row paths with NT threads: the candidate lists of the resident path (per wave; a needle's
// neighbouring tokens fall to one wave) and the histogram of the general path share one area.
template <int NT>
struct RowLds {
  static constexpr int NW = NT / kWave;
  static constexpr int kWaveCand = NW == 1 ? 512 : (NW == 2 ? 256 : 128);
  union {
    struct {
      uint64_t key[NW * kWaveCand];   // (order-preserving key of the weight) << 32 | ~position
      float val[NW * kWaveCand];
    } cand;
    uint32_t hist[kHistBins];
  };
  uint32_t sh_scan[NW], res[2], sh_u[NW], cnt[NW];
  double sh_d[NW], tot[NW], tnw[NW];
  float bound[NW], tau;
};

__device__ __forceinline__ void store_cells(double* c, double WO, double WD, double tot, double tnw) {
  const double WS = fmax(0.0, tnw - WO);
  c[0] = WO;
  c[1] = WD;
  c[2] = WS;
  c[3] = tot - WO - WD - WS;
}

// Resident row path: the row is read once, NG 16-byte groups per thread, and stays in registers.  Rows begin
// where the row before them ends, so a row of any length begins at some float of a 16-byte group: the groups
// are counted from the aligned address at or below the row's begin (`lead` floats before it).  The floats of the
// first group that belong to the row before are taken out; those of a last group that is not whole (it may reach
// past the tensor) are held one each by the first threads.
// A lower bound of the K-th largest weight comes from maxima per lane in each wave (K distinct elements); the
// few weights at or above the bound are collected in LDS and ranked exactly (larger first, equal weights by
// lower position).  Returns false, with nothing written, if a list overflows (many ties at the bound).
// Bound: HBM up to 45052 weights.  32 x 32 heads x 16 rows of 16384 floats (1 GiB): 160-165 us, 6.6 TB/s.  Rows of 13867
// floats went through the general path, five sweeps over memory: 350 us for 227 MB; here 42 us, 5.4 TB/s.  Longer rows take
// 1024 threads, whose 128 registers do not hold 16 groups and the rest (60 spilled), and such a workgroup fills its CU, so that
// no row's loads run beside another's reduction: 1024 rows of 65532 weights 79 us, 3.4 TB/s (general path 512 us).  Above 65533 weights the
// general path is all there is: 512 rows of 131072 920 us, 0.3 TB/s.
// Rows of a call: of any length; of whole 16-byte groups (n % 4 == 0); of a multiple of 16 KiB (n % 4096 == 0).
constexpr int kRowsAny = 0, kRowsWhole = 1, kRowsAligned = 2;
template <int NT, int NG, int ROWS>
__device__ __forceinline__ bool row_cells_resident(const float* __restrict__ W, int32_t n, int32_t needle_start,
                                                   int32_t needle_len, int32_t topk, double* __restrict__ c_out, RowLds<NT>& S) {
  constexpr int NW = NT / kWave, kWaveCand = RowLds<NT>::kWaveCand;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  constexpr bool WHOLE = ROWS != kRowsAny, ALIGNED = ROWS == kRowsAligned;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int32_t ne = needle_start + needle_len;
  const int32_t lead = WHOLE ? 0 : (int32_t)((reinterpret_cast<uintptr_t>(W) >> 2) & 3u);
  const int32_t end = lead + n;                        // floats are counted from the aligned address
  const int32_t ngroups = end >> 2;                    // whole groups (at least one: n >= 4)
  const f32x4* W4 = reinterpret_cast<const f32x4*>(W - lead);

  // group i of this thread: i * NT + tid; all loads are issued first.  The rows are read exactly once:
  // non-temporal loads (they do not displace anything in the caches) stream about 13 % faster than plain
  // ones on this part.
  //   ALIGNED: such rows all begin at the same memory channel.  Workgroups therefore begin 0, 8, 16 or 24 KiB into their row, and all add up from 24 KiB on, when what they
  // have read first is there: a row's sums have one order, wherever it stands in the call.
  auto group = [&](int i) __attribute__((always_inline)) { return i * NT + tid; };
  constexpr int STEP = ALIGNED ? 8192 / (16 * NT) : 0;
  static_assert(3 * STEP < NG, "four places to begin at");
  f32x4 v[NG];
  auto load_from = [&](auto first_c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      const int i = (u + decltype(first_c)::value) % NG;
      v[i] = __builtin_nontemporal_load(W4 + min(group(i), ngroups - 1));   // past the end: loaded again, never used
    }
  };
  switch (ALIGNED ? blockIdx.x & 3 : 0) {
    case 0: load_from(std::integral_constant<int, 0>{}); break;
    case 1: load_from(std::integral_constant<int, STEP>{}); break;
    case 2: load_from(std::integral_constant<int, 2 * STEP>{}); break;
    default: load_from(std::integral_constant<int, 3 * STEP>{});
  }
  const int32_t jx = 4 * ngroups + tid - lead;         // position of this thread's float of the last group
  const bool have_x = !WHOLE && tid < (end & 3) && jx >= 0;
  const float vx = have_x ? W[jx] : 0.f;
  const int32_t jn = needle_start + tid;
  const float nd = W[jn < ne ? jn : needle_start];

  double tot = 0.0, tnw = 0.0;           // row sum and needle sum, in double
  if (!WHOLE && tid == 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (c < lead) v[0][c] = 0.f;
  }
  // M maxima per lane (of its groups i, i + M, ...): enough disjoint subsets of the row that the K-th largest of
  // their maxima lies close to the K-th largest weight
  constexpr int M = NW == 1 ? 4 : NW == 2 ? 2 : 1;
  float mx[M];
  uint32_t seen = 0;                       // bit m: subset m has data
#pragma unroll
  for (int m = 0; m < M; ++m) mx[m] = -INFINITY;
#pragma unroll
  for (int u = 0; u < NG; ++u) {
    const int i = (u + 3 * STEP) % NG;
    if (group(i) < ngroups) {
      seen |= 1u << i % M;
      tot += (double)v[i].x;
      tot += (double)v[i].y;
      tot += (double)v[i].z;
      tot += (double)v[i].w;
      if (!WHOLE && i == 0 && tid == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
          if (c < lead) v[0][c] = -INFINITY;
      }
      mx[i % M] = fmaxf(fmaxf(mx[i % M], fmaxf(v[i].x, v[i].y)), fmaxf(v[i].z, v[i].w));
    }
  }
  if (!WHOLE) {
    tot += (double)vx;
    if (have_x) mx[0] = fmaxf(mx[0], vx);
  }
  if (jn < ne) tnw = (double)nd;
  for (int32_t j = jn + NT; j < ne; j += NT) tnw += (double)W[j];
  tot = wave_sum<double>(tot);
  tnw = wave_sum<double>(tnw);

  // Each wave finds a value at or below the ceil(K/NW)-th largest of its 64 M maxima (bisection on the
  // upper 20 bits of the order-preserving key, with ballots).  At least K weights are >= the smallest of
  // the waves' values, so it bounds the K-th largest from below.
  const uint32_t want = (uint32_t)(topk + NW - 1) / NW;
  uint32_t mkey[M];
#pragma unroll
  for (int m = 0; m < M; ++m) mkey[m] = seen >> m & 1u || (m == 0 && have_x) ? float_key(mx[m]) : 0u;   // subsets without data never count
  auto reach = [&](uint32_t t) __attribute__((always_inline)) {
    uint32_t c = 0;
#pragma unroll
    for (int m = 0; m < M; ++m) c += (uint32_t)__popcll(__ballot(mkey[m] >= t));
    return c;
  };
  // (it starts below the bits that all maxima share and ends where exactly as many as wanted reach the value)
  uint32_t tkey = 0;
  {
    uint32_t least = 0xffffffffu, most = 0u;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      least = min(least, mkey[m] ? mkey[m] : 0xffffffffu);
      most = max(most, mkey[m]);
    }
    least = wave_reduce_to_last(least, [](uint32_t a, uint32_t b) { return min(a, b); });
    most = wave_reduce_to_last(most, [](uint32_t a, uint32_t b) { return max(a, b); });
    least = (uint32_t)__builtin_amdgcn_readlane((int)least, kWave - 1);
    most = (uint32_t)__builtin_amdgcn_readlane((int)most, kWave - 1);
    int b = 31;
    if (reach(1u) >= want) {
      b = 31 - __clz((int)(least ^ most));                     // (-1: all equal)
      tkey = b < 12 ? least & 0xfffff000u : b < 31 ? least & (0xfffffffeu << b) : 0u;
    }
    for (; b >= 12; --b) {
      const uint32_t trial = tkey | (1u << b), c = reach(trial);
      if (c >= want) tkey = trial;
      if (c == want) break;
    }
  }
  // the float whose key is tkey (low bits cleared: not above the value found); 0 keys: -inf
  float bound = tkey == 0 ? -INFINITY : __uint_as_float((tkey & 0x80000000u) ? (tkey ^ 0x80000000u) : ~tkey);
  if (NW > 1) {
    if (lane == 0) {
      S.tot[wv] = tot;
      S.tnw[wv] = tnw;
      S.bound[wv] = bound;
    }
    __syncthreads();
    tot = S.tot[0];
    tnw = S.tnw[0];
    bound = S.bound[0];
#pragma unroll 4
    for (int i = 1; i < NW; ++i) {
      tot += S.tot[i];
      tnw += S.tnw[i];
      bound = fminf(bound, S.bound[i]);
    }
  }

  // Candidates of this wave go to its own part of the list; the slot of a lane is the number
  // of candidates found so far plus the candidates of the same element in lower lanes.
  uint32_t base = 0;                   // wave-uniform
  float* my_val = S.cand.val + wv * kWaveCand;
  uint64_t* my_key = S.cand.key + wv * kWaveCand;
  auto collect = [&](bool is, float x, int32_t j) __attribute__((always_inline)) {
    const unsigned long long mask = __ballot(is);
    if (mask) {
      const uint32_t slot = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if (is && slot < (uint32_t)kWaveCand) {
        my_val[slot] = x;
        my_key[slot] = ((uint64_t)float_key(x) << 32) | (uint32_t)(~(uint32_t)j);
      }
      base += (uint32_t)__popcll(mask);
    }
  };
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int32_t g = group(i);
    const float bnd = g < ngroups ? bound : INFINITY;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int32_t j = 4 * g + c - lead;              // (before the row: -inf by now, listed only under a bound of -inf)
      collect(v[i][c] >= bnd && (WHOLE || i > 0 || c == 3 || j >= 0), v[i][c], j);
    }
  }
  if (!WHOLE) collect(have_x && vx >= bound, vx, jx);
  if (lane == 0) S.cnt[wv] = base;
  __syncthreads();
  uint32_t nc = 0;
  bool fits = true;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const uint32_t ci = S.cnt[i];
    nc += ci;
    fits = fits && ci <= (uint32_t)kWaveCand;
  }
  if (!(fits && nc >= (uint32_t)topk)) return false;   // (the same in every thread)
  // A candidate belongs to T_k if fewer than K candidates are ahead of it (larger, or equal at a lower
  // position: one comparison of the packed keys).  Up to 256 candidates are handled by the first wave alone,
  // one or four of them in each lane, every lane's read by all in turn; the other waves retire.
  auto candidate = [&](uint32_t c, uint64_t& key, float& x) __attribute__((always_inline)) {
    uint32_t part = 0, idx = c;
#pragma unroll
    for (int i = 0; i < NW - 1; ++i) {
      const uint32_t ci = S.cnt[i];
      if (part == (uint32_t)i && idx >= ci) {
        idx -= ci;
        part = i + 1;
      }
    }
    const bool have = c < nc;
    key = have ? S.cand.key[part * kWaveCand + idx] : 0ull;      // (the filler is ahead of nothing)
    x = have ? S.cand.val[part * kWaveCand + idx] : 0.f;
  };
  double wo = 0.0, wd = 0.0;
  auto add = [&](bool in, uint64_t key, float x) __attribute__((always_inline)) {
    const int32_t px = (int32_t)(~(uint32_t)key);
    if (in && px >= needle_start && px < ne) wo += (double)x;
    else if (in) wd += (double)x;
  };
  auto rank_in_wave = [&](auto per_c) __attribute__((always_inline)) {
    constexpr int PER = decltype(per_c)::value;
    uint64_t mine[PER];
    float x[PER];
    uint32_t ahead[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      candidate(q * kWave + lane, mine[q], x[q]);
      ahead[q] = 0;
    }
    // More than one candidate a lane: first a value that exactly K of them reach, by bisection; only where equal weights
    // stand at the cut there is none, and each is ranked.
    bool exact = false;
    uint32_t cut = 0;
    if (PER > 1) {
      for (int b = 31; b >= 0 && !exact; --b) {
        const uint32_t trial = cut | (1u << b);
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) c += (uint32_t)__popcll(__ballot((uint32_t)(mine[q] >> 32) >= trial));
        if (c >= (uint32_t)topk) cut = trial;
        exact = c == (uint32_t)topk;
      }
    }
    if (exact) {
#pragma unroll
      for (int q = 0; q < PER; ++q) ahead[q] = (uint32_t)(mine[q] >> 32) >= cut ? 0u : (uint32_t)topk;
    } else
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int cnt = min((int)nc - p * kWave, kWave);
#pragma unroll 4
      for (int o = 0; o < cnt; ++o) {
        const uint64_t ko = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine[p] >> 32), o) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine[p], o);
#pragma unroll
        for (int q = 0; q < PER; ++q) ahead[q] += ko > mine[q] ? 1u : 0u;
      }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) add((uint32_t)(q * kWave + lane) < nc && ahead[q] < (uint32_t)topk, mine[q], x[q]);
    wo = wave_sum<double>(wo);
    wd = wave_sum<double>(wd);
  };
  if (nc <= (uint32_t)kWave * 4u) {
    if (wv != 0) return true;
    if (nc <= (uint32_t)kWave) rank_in_wave(std::integral_constant<int, 1>{});
    else rank_in_wave(std::integral_constant<int, 4>{});
  } else {
    for (uint32_t c = tid; c < (nc + NT - 1) / NT * NT; c += NT) {
      uint64_t mine;
      float x;
      candidate(c, mine, x);
      uint32_t ahead = 0;
#pragma unroll 1
      for (int p = 0; p < NW; ++p) {
        const uint32_t cnt = S.cnt[p];
        for (uint32_t o = 0; o < cnt; ++o) ahead += S.cand.key[p * kWaveCand + o] > mine ? 1u : 0u;
      }
      add(c < nc && ahead < (uint32_t)topk, mine, x);
    }
    wo = block_sum<NT, double>(wo, S.sh_d);
    wd = block_sum<NT, double>(wd, S.sh_d);
  }
  if (tid == 0) store_cells(c_out, wo, wd, tot, tnw);
  return true;
}

// General row path: any length, any K, any number of equal weights; the row is read from memory in every sweep.
// RARE: reached from the resident path only, so kept small.
template <int NT, bool RARE>
__device__ __forceinline__ void row_cells_general(const float* __restrict__ W, int32_t n, int32_t needle_start,
                                                  int32_t needle_len, int32_t topk, double* __restrict__ c_out, RowLds<NT>& S) {
  const int tid = threadIdx.x;
  const int32_t ne = needle_start + needle_len;
  auto& hist = S.hist;
  auto& sh_scan = S.sh_scan;
  auto& res = S.res;
  auto& sh_d = S.sh_d;
  auto& sh_u = S.sh_u;
  // f(position, value) over the row
  auto sweep = [&](auto f) __attribute__((always_inline)) {
    if constexpr (RARE) {
#pragma unroll 1
      for (int32_t j = tid; j < n; j += NT) f(j, W[j]);
    } else {
      for (int32_t j = tid; j < n; j += NT) f(j, W[j]);
    }
  };
  double tot = 0.0, tnw = 0.0;           // row sum and needle sum, in double
  sweep([&](int32_t, float x) { tot += (double)x; });
  for (int32_t j = needle_start + tid; j < ne; j += NT) tnw += (double)W[j];
  tot = block_sum<NT, double>(tot, sh_d);
  tnw = block_sum<NT, double>(tnw, sh_d);

  // K-th largest weight: three histogram levels over the order-preserving key
  uint32_t prefix = 0, k = (uint32_t)topk;
#pragma unroll 1
  for (int level = 0; level < 3; ++level) {
    const int shift = level == 0 ? 21 : (level == 1 ? 10 : 0);
    const int bits = level == 2 ? 10 : 11;
    for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
    __syncthreads();
    sweep([&](int32_t, float x) {
      const uint32_t key = float_key(x);
      if (level == 0 || (key >> (shift + bits)) == prefix) atomicAdd(&hist[(key >> shift) & ((1u << bits) - 1u)], 1u);
    });
    __syncthreads();
    select_bin<NT>(hist, k, sh_scan, res);
    prefix = (prefix << bits) | res[0];
    k = res[1];
    __syncthreads();
  }
  const uint32_t tau = prefix;
  const uint32_t need_eq = k;            // elements equal to the K-th value that are inside T_k

  // mass above the threshold, inside / outside the needle; census of the ties
  double wo = 0.0, wd = 0.0;
  uint32_t eq_all = 0, eq_needle = 0;
  float tau_val = 0.f;
  sweep([&](int32_t j, float x) {
    const uint32_t key = float_key(x);
    const bool inn = j >= needle_start && j < ne;
    if (key > tau) {
      if (inn) wo += (double)x; else wd += (double)x;
    } else if (key == tau) {
      eq_all += 1;
      eq_needle += inn ? 1u : 0u;
      tau_val = x;
    }
  });
  wo = block_sum<NT, double>(wo, sh_d);
  wd = block_sum<NT, double>(wd, sh_d);
  eq_all = block_sum<NT, uint32_t>(eq_all, sh_u);
  eq_needle = block_sum<NT, uint32_t>(eq_needle, sh_u);
  // every tie has the same value; fetch it from any thread that saw one
  if (tid == 0) S.tau = 0.f;
  __syncthreads();
  if (float_key(tau_val) == tau) S.tau = tau_val;
  __syncthreads();
  tau_val = S.tau;

  uint32_t take_needle;                  // ties inside the needle that belong to T_k
  if (need_eq == eq_all) {
    take_needle = eq_needle;
  } else {
    // ties are cut: T_k takes the need_eq ties of lowest position.  Find that position bound
    // by a radix select on the inverted position among the ties, then count.
    uint32_t p2 = 0, k2 = need_eq;
#pragma unroll 1
    for (int level = 0; level < 3; ++level) {
      const int shift = level == 0 ? 21 : (level == 1 ? 10 : 0);
      const int bits = level == 2 ? 10 : 11;
      for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
      __syncthreads();
      sweep([&](int32_t j, float x) {
        if (float_key(x) != tau) return;
        const uint32_t key = ~(uint32_t)j;
        if (level == 0 || (key >> (shift + bits)) == p2) atomicAdd(&hist[(key >> shift) & ((1u << bits) - 1u)], 1u);
      });
      __syncthreads();
      select_bin<NT>(hist, k2, sh_scan, res);
      p2 = (p2 << bits) | res[0];
      k2 = res[1];
      __syncthreads();
    }
    const int32_t last_pos = (int32_t)(~p2);
    uint32_t cntn = 0;
    sweep([&](int32_t j, float x) {
      if (float_key(x) == tau && j <= last_pos && j >= needle_start && j < ne) cntn += 1;
    });
    take_needle = block_sum<NT, uint32_t>(cntn, sh_u);
  }
  if (tid == 0) store_cells(c_out, wo + (double)tau_val * (double)take_needle, wd + (double)tau_val * (double)(need_eq - take_needle), tot, tnw);
}

// One workgroup per row; cells[row] = (WO, WD, WS, Wide).  NG = 0: the general path.  MW: wavefronts of a SIMD that the registers leave room for; with rows of a
// multiple of 16 KiB no more than 4 (5 where MW is) run there, though fewer registers would do: 16384 weights 170 us a GiB with 5 workgroups to a CU, 159 with 4.
template <int NT, int NG, int ROWS, int MW>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(MW, ROWS == kRowsAligned ? (MW < 4 ? 4 : MW) : 8))) void row_cells_kernel(const float* __restrict__ rows, int32_t n, int32_t needle_start,
                                                          int32_t needle_len, int32_t topk, double* __restrict__ cells) {
  __shared__ RowLds<NT> S;
  const float* W = rows + (int64_t)blockIdx.x * n;
  double* c = cells + (int64_t)blockIdx.x * 4;
  if constexpr (NG > 0) {
    if (row_cells_resident<NT, NG, ROWS>(W, n, needle_start, needle_len, topk, c, S)) return;
    __syncthreads();                     // the candidate lists have been read
  }
  row_cells_general<NT, (NG > 0)>(W, n, needle_start, needle_len, topk, c, S);
}

// Steps 5-7 of Algorithm 1 (0/0 = 0); a component that is switched off enters as 0.
__device__ __forceinline__ void sf_lg(double WO, double WD, double WS, int use_wo, int use_wd, int use_ws, double& SF,
                                      double& LG) {
  WO = use_wo ? WO : 0.0;
  WD = use_wd ? WD : 0.0;
  WS = use_ws ? WS : 0.0;
  SF = (WO + WD) > 0.0 ? WO / (WO + WD) : 0.0;
  LG = (WO + WS) > 0.0 ? WO / (WO + WS) : 0.0;
}

// One wave per head: adds the head's T rows (a fixed tree: results are bit-reproducible) into the accumulators
// (fresh: which count as zero and are not read) and finalises SF, LG, INF (Algorithm 1, steps 5-7).  STRIDE 5:
// the accumulators of slkv_score_heads; STRIDE 8: those of slkv_score_heads_ex, which also carry the sums of the
// per-row SF and LG.
// Bound: the latency of one load and, with STRIDE 8, of the rows' divisions: a lane per row (one thread per head,
// its rows one after the other, took 5.4 us on 1024 heads x 16 rows).
constexpr int kReduceHeads = 4;          // heads (waves) of a workgroup

template <int STRIDE>
__global__ __launch_bounds__(64 * kReduceHeads) void head_reduce_kernel(const double* __restrict__ cells, int32_t heads, int32_t T,
                                                                        double* __restrict__ acc, double* __restrict__ scores,
                                                                        int fresh, int macro, int use_wo, int use_wd, int use_ws) {
  const int lane = threadIdx.x & 63;
  const int hd = blockIdx.x * kReduceHeads + (threadIdx.x >> 6);
  if (hd >= heads) return;
  double* A = acc + (int64_t)hd * STRIDE;
  double was = 0.0;                      // lane i: accumulator i
  if (!fresh && lane < STRIDE) was = A[lane];
  const double2* c2 = reinterpret_cast<const double2*>(cells) + (int64_t)hd * T * 2;
  double a[STRIDE == 8 ? 6 : 4] = {};
  for (int t = lane; t < T; t += kWave) {
    const double2 lo = c2[t * 2], hi = c2[t * 2 + 1];
    a[0] += lo.x;
    a[1] += lo.y;
    a[2] += hi.x;
    a[3] += hi.y;
    if constexpr (STRIDE == 8) {
      double sf, lg;
      sf_lg(lo.x, lo.y, hi.x, use_wo, use_wd, use_ws, sf, lg);
      a[4] += sf;
      a[5] += lg;
    }
  }
#pragma unroll
  for (int i = 0; i < (STRIDE == 8 ? 6 : 4); ++i) {
    const double s = wave_sum<double>(a[i]);
    was += lane == (i < 4 ? i : i + 1) ? s : 0.0;
  }
  was += lane == 4 ? (double)T : 0.0;
  if (lane < STRIDE) A[lane] = was;
  if (scores) {
    double now[STRIDE];
#pragma unroll
    for (int i = 0; i < STRIDE; ++i) now[i] = __shfl(was, i, kWave);
    double SF, LG;
    if (STRIDE == 8 && macro) {
      SF = now[4] > 0.0 ? now[STRIDE == 8 ? 5 : 0] / now[4] : 0.0;
      LG = now[4] > 0.0 ? now[STRIDE == 8 ? 6 : 0] / now[4] : 0.0;
    } else {
      sf_lg(now[0], now[1], now[2], use_wo, use_wd, use_ws, SF, LG);
    }
    const double INF = (SF + LG) > 0.0 ? 2.0 * SF * LG / (SF + LG) : 0.0;
    if (lane < 3) scores[(int64_t)hd * 3 + lane] = lane == 0 ? SF : lane == 1 ? LG : INF;
  }
}

// ------------------------------------------------------------------------------------------
// Stage 1 straight from the decode queries and the context keys (Section 3.1, Eq. 2-4 feeding
// Algorithm 1): the attention rows are never written anywhere.  One workgroup owns 64 query rows
// of one KV head (the T decode steps of its G query heads) and all n keys.
//
// With 64 rows per key the work is bound by reading the keys (64 flop per byte), so the kernel is
// built as a stream: each of the 8 waves takes every 8th sub-tile of 32 keys, loads it straight
// from memory into the operand registers of the 32x32x16 bf16 MFMA (a lane: 16 bytes of one key
// row per load; nothing is staged in LDS and the waves never wait for each other inside a chunk),
// keeps two sub-tiles in flight, and multiplies it with both 32-row tiles of the queries, which
// stay in registers for a chunk.  A lane owns two query rows (one per row tile) and, per sub-tile, 16 keys of
// each: it keeps the running softmax statistics and the needle mass of its rows.
// Logits at or above the row's bound are appended to the row's candidate list in LDS: a lane counts
// its own ones of both row tiles first, so that a step waits for one pair of LDS atomics and not for one per entry.
// The keys are cut into chunks: the first kQkFirst keys, then chunks as long as everything before
// them.  After every chunk the waves meet, the bound of a row becomes a value at or a little below the K-th largest
// entry of its list (the K-th largest logit so far) and the list is cut back to the entries at or above it;
// since a chunk holds as many keys as came before, about K new entries join the K carried ones, and a
// list of 256 has room for K = 64 and five standard deviations more, or for logits that rise along the
// context.  The first two sub-tiles of every wave on the next chunk are in flight while the waves meet.
// The first chunk, which has no bound to start from, stays in registers: a wave's two sub-tiles
// give 8 maxima per lane and row, the 16 lanes of a row 128 maxima of disjoint key subsets, whose
// K-th largest is a lower bound of the row's K-th largest logit; then the logits are collected.
// At the end the bisection goes on until exactly K entries are left; where equal or almost equal logits prevent that, the
// entries are ranked (larger logit first, equal logits by lower position).  The K winners become
// weights with the row's log-sum-exp and are split into WO / WD by needle membership.  A row whose
// list overflows (many equal logits at the top, or logits that keep rising along the context) is
// flagged and redone by qk_fallback_kernel.
// Calls with too few heads and rows for the chip, or a little more than it takes at once, cut the keys into `nsplit` ranges of
// `range` keys: a workgroup then leaves its range's statistics and K largest logits per row to qk_merge_kernel.
// d = 64 spills no register; d = 128 takes all 256 and spills 23, LDS addresses mostly, which come back from scratch memory after
// every meeting (11.5 MiB in the call below).
// 32 layers x 8 KV heads x 16384 keys x 64 rows, K = 32: 316 -> 241 us (4.5 TB/s of keys; a large copy runs at 5.3) against
// chunks half as long as what came before with lists of 128, a first chunk of 1024 keys walked twice, an 18-step
// bisection at every chunk, an LDS atomic per entry and the queries in registers throughout; 6 meetings of the waves
// instead of 11.  With the meetings of half of the workgroups (7 then) between those of the others 231 (4.65 TB/s).
constexpr int kQkThreads = 512;      // 8 waves
constexpr int kQkWaves = kQkThreads / 64;
constexpr int kQkRows = 64;          // two row tiles of 32
constexpr int kQkStripe = 32 * kQkWaves;   // keys the waves take together: chunk ends are multiples of it
constexpr int kQkFirst = 2 * kQkStripe;    // keys of the first chunk: two sub-tiles per wave
constexpr int kQkSubsets = kQkWaves * 2 * 8;    // key subsets per row whose maxima are taken in the first chunk
constexpr int kQkCand = 256;         // entries of a row's list
constexpr int kQkStride = kQkCand + 8;     // conflict-free for the 8 rows a wave looks after; entry kQkCand takes what overflows
constexpr int kQkSlack = 6;          // between chunks a list may keep this many entries more than K
constexpr int kQkMaxSplit = 32;      // key ranges of a head
constexpr int kQkFallbackWGs = 128;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 qk_bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float qk_f32x16;
typedef uint32_t qk_u32x4 __attribute__((ext_vector_type(4)));
union QkPack16 {
  qk_u32x4 u;
  qk_bf16x8 b;
};

struct QkLds {
  float cand_x[kQkRows][kQkStride];                         // scaled logits (log2 domain); first chunk: the subset maxima [row][(wave, half, i)]
  int32_t cand_p[kQkRows][kQkStride];
  union {
    __attribute__((aligned(16))) unsigned char q[kQkRows][128 * 2 + 16];   // the queries (padded rows)
    struct {                                                // in the last meeting, when the queries have been read: statistics of the rows' 16 lanes
      float st_m[kQkRows][2 * kQkWaves], st_s[kQkRows][2 * kQkWaves], st_t[kQkRows][2 * kQkWaves];
    };
  };
  float bound[kQkRows];
  uint32_t cnt[kQkRows];
  uint32_t ovf[kQkRows];
};

// Floats of a (row, key range) record: largest logit, sum, needle sum, overflow flag; the K largest logits (NaN beyond the
// range's keys); their positions.
__host__ __device__ constexpr int qk_record(int topk) { return 4 + 2 * topk; }

// Sum / maximum / minimum over the 8 lanes that look after a row: neighbours in the quad, then the other quad (DPP).
template <class F>
__device__ __forceinline__ uint32_t over_8_lanes(uint32_t v, F f) {
  v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
  v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
  return f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));   // row_half_mirror
}
__device__ __forceinline__ uint32_t sum_8(uint32_t v) {
  return over_8_lanes(v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ float sum_8(float v) {
  return __uint_as_float(over_8_lanes(__float_as_uint(v), [](uint32_t a, uint32_t b) { return __float_as_uint(__uint_as_float(a) + __uint_as_float(b)); }));
}
__device__ __forceinline__ float max_8(float v) {
  return __uint_as_float(over_8_lanes(__float_as_uint(v), [](uint32_t a, uint32_t b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); }));
}
__device__ __forceinline__ double sum_8(double v) {
#pragma unroll
  for (int m = 1; m < 8; m *= 2) v += __shfl_xor(v, m, 64);
  return v;
}

template <int DK>
__global__ __launch_bounds__(kQkThreads) void qk_cells_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kmat,
                                                                 int Hq, int Hkv, int T, int n_keys, int rowgroups,
                                                                 int nsplit, int range, int first_needle, int needle_len, int topk,
                                                                 float c_log2, double* __restrict__ cells,
                                                                 unsigned char* __restrict__ overflow, float* __restrict__ part) {
  constexpr int KK = DK / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char qk_smem[];
  QkLds& S = *reinterpret_cast<QkLds*>(qk_smem);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  static_assert(kQkSubsets <= kQkStride, "the subset maxima of the first chunk live in the (still empty) candidate lists");
  static_assert(kQkSubsets == 128 && kQkCand == 256 && kQkRows == 8 * kQkWaves, "eight lanes hold the maxima or a half or all of the candidates of a row, 16 or 32 each");
  constexpr int RPW = kQkRows / kQkWaves;            // rows a wave looks after between the chunks
  const int G = Hq / Hkv, R = G * T;
  const int split = blockIdx.x % nsplit, group = blockIdx.x / nsplit;
  const int rg = group % rowgroups, seg = group / rowgroups;             // seg = l * Hkv + kvh
  // this workgroup's keys, and the needle, from here on counted from the start of its range
  const int key_base = split * range, n = min(range, n_keys - key_base), needle_start = first_needle - key_base;
  const int l = seg / Hkv, kvh = seg % Hkv;
  const int row0 = rg * kQkRows;
  const int nrows = min(kQkRows, R - row0);
  const int64_t rowid0 = ((int64_t)l * Hq + (int64_t)kvh * G) * T + row0;   // first global row of this workgroup
  const uint16_t* qbase = q + rowid0 * DK;
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(kmat + ((int64_t)seg * n_keys + key_base) * DK);
  const int ne = needle_start + needle_len;

  for (int i = tid; i < kQkRows; i += kQkThreads) {
    S.cnt[i] = 0;
    S.ovf[i] = 0;
    S.bound[i] = INFINITY;
  }
  constexpr int PPR = DK / 8;                          // 16-byte pieces of a row
  for (int i = tid; i < kQkRows * PPR; i += kQkThreads)
    *reinterpret_cast<qk_u32x4*>(&S.q[i / PPR][i % PPR * 16]) =
        *reinterpret_cast<const qk_u32x4*>(qbase + (int64_t)min(i / PPR, nrows - 1) * DK + i % PPR * 8);
  // the queries of this lane's rows inside the workgroup, l32 and 32 + l32: read from LDS for every chunk, so that their
  // registers are free while the waves meet
  qk_bf16x8 qreg[2][KK];
  auto load_queries = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        QkPack16 p;
        p.u = *reinterpret_cast<const qk_u32x4*>(&S.q[mt * 32 + l32][kk * 32 + half * 16]);
        qreg[mt][kk] = p.b;
      }
  };
  float m_run[2] = {-INFINITY, -INFINITY}, s_run[2] = {0.f, 0.f}, t_run[2] = {0.f, 0.f};   // running maximum, sum of exp2(x - max), the same over the needle
  float bound_raw[2];

  // one sub-tile of 32 keys starting at key_s: 16 bytes of key row (key_s + l32) per load (clamped at the end of the keys)
  auto issue = [&](int key_s, qk_u32x4 (&kf)[KK]) __attribute__((always_inline)) {
    const uint32_t off = (uint32_t)min(key_s + l32, n - 1) * (uint32_t)(DK * 2) + (uint32_t)half * 16u;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = *reinterpret_cast<const qk_u32x4*>(kbase + (off + (uint32_t)kk * 32u));
  };
  // MFMAs of one sub-tile against both row tiles: acc[mt][i] = q(row mt*32 + l32) . k(key_s + 8*(i/4) + 4*half + i%4),
  // not yet scaled by log2(e)/sqrt(d)
  auto mfma_sub = [&](const qk_u32x4 (&kf)[KK], qk_f32x16 (&acc)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      QkPack16 p;
      p.u = kf[kk];
      if (kk == 0) {
        qk_f32x16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p.b, qreg[0][kk], z, 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p.b, qreg[1][kk], z, 0, 0, 0);
      } else {
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p.b, qreg[0][kk], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p.b, qreg[1][kk], acc[1], 0, 0, 0);
      }
    }
  };
  // the last sub-tile of the keys: what lies beyond them counts as -inf
  auto mask_sub = [&](int key_s, qk_f32x16 (&acc)[2]) __attribute__((always_inline)) {
    if (key_s + 32 > n) {
      const int key0 = key_s + 4 * half;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (key0 + 8 * (i >> 2) + (i & 3) >= n) acc[mt][i] = -INFINITY;
    }
  };
  // Three-operand maxima written out: from fmaxf the compiler makes two instructions that only canonicalise for each
  // that compares.  The first maximum is the compiler's: reading the MFMA's result there, it keeps the
  // distance that the hardware asks for between the two, and the others follow it.
  auto max_16 = [&](const qk_f32x16& a) __attribute__((always_inline)) {
    float r = fmaxf(a[14], a[15]);
#pragma unroll
    for (int i = 0; i < 14; i += 2) asm("v_max3_f32 %0, %0, %1, %2" : "+v"(r) : "v"(a[i]), "v"(a[i + 1]));
    return r;
  };
  // softmax statistics of the 16 unscaled logits a of row tile mt; returns their maximum.  Straight-line
  // code (it is scheduled among the MFMAs of the next sub-tile); the needle mass of the few sub-tiles
  // that touch the needle is added by needle_mass() afterwards.
  auto stats = [&](int mt, const qk_f32x16& a) __attribute__((always_inline)) {
    const float mxr = max_16(a);
    const float mn = fmaxf(m_run[mt], mxr * c_log2);
    const float mu = mn == -INFINITY ? 0.f : mn;
    const float scale = __builtin_amdgcn_exp2f(m_run[mt] - mu);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(fmaf(a[i], c_log2, -mu));
    s_run[mt] = s_run[mt] * scale + sum;
    t_run[mt] = t_run[mt] * scale;
    m_run[mt] = mn;
    return mxr;
  };
  // after stats(): the weights of the sub-tile's needle keys, against the same (updated) reference
  auto needle_mass = [&](int mt, int key0, const qk_f32x16& a) __attribute__((always_inline)) {
    if (key0 + 32 > needle_start && key0 < ne) {
      const float mu = m_run[mt] == -INFINITY ? 0.f : m_run[mt];
      float tsum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = key0 + 8 * (i >> 2) + (i & 3);
        if (key >= needle_start && key < ne) tsum += __builtin_amdgcn_exp2f(fmaf(a[i], c_log2, -mu));
      }
      t_run[mt] += tsum;
    }
  };
  // The logits at or above the bounds join the rows' lists (mx: the largest unscaled logit of each 16; bound_raw:
  // the bound in unscaled units, rounded down, so that the test never misses one).
  auto collect = [&](int key0, const qk_f32x16 (&a)[2], const float (&mx)[2]) __attribute__((always_inline)) {
    if (mx[0] >= bound_raw[0] || mx[1] >= bound_raw[1]) {
      uint32_t slot0 = 0, slot1 = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        slot0 += a[0][i] >= bound_raw[0] ? 1u : 0u;
        slot1 += a[1][i] >= bound_raw[1] ? 1u : 0u;
      }
      slot0 = atomicAdd(&S.cnt[l32], slot0);
      slot1 = atomicAdd(&S.cnt[32 + l32], slot1);
      auto append = [&](int mt, uint32_t slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (a[mt][i] >= bound_raw[mt]) {
            const uint32_t at = min(slot++, (uint32_t)kQkCand);
            S.cand_x[mt * 32 + l32][at] = a[mt][i] * c_log2;
            S.cand_p[mt * 32 + l32][at] = key0 + 8 * (i >> 2) + (i & 3);
          }
      };
      append(0, slot0);
      append(1, slot1);
    }
  };
  // This wave's sub-tiles of [key_lo, key_hi) (multiples of kQkStripe, key_hi clipped to n) as a
  // software pipeline: the MFMAs of a sub-tile are issued among the statistics of the sub-tile
  // before it (the two sets of accumulators alternate), and the loads of the sub-tile after it are
  // in flight.  front(mt, a) runs inside that mix and returns a value that back(key0, a, values)
  // takes afterwards (and may branch).  The
  // wave's first two sub-tiles are already on their way into kfA and kfB, requested by prefetch().
  qk_u32x4 kfA[KK], kfB[KK];
  auto prefetch = [&](int key_lo, int key_hi) __attribute__((always_inline)) {
    if (key_lo + wv * 32 < key_hi) issue(key_lo + wv * 32, kfA);
    if (key_lo + wv * 32 + kQkStripe < key_hi) issue(key_lo + wv * 32 + kQkStripe, kfB);
  };
  auto walk = [&](int key_lo, int key_hi, auto front, auto back) __attribute__((always_inline)) {
    int ks = key_lo + wv * 32;
    if (ks >= key_hi) return;
    qk_f32x16 accA[2], accB[2];
    mfma_sub(kfA, accA);
    // one pipelined step: the sub-tile at ks is in `cur`; the next one goes from kn into `nxt`, and kc is refilled
    auto pstep = [&](qk_f32x16 (&cur)[2], qk_f32x16 (&nxt)[2], qk_u32x4 (&kc)[KK], qk_u32x4 (&kn)[KK]) __attribute__((always_inline)) {
      const int key0 = ks + 4 * half;
      float v[2];
      // kc held the current sub-tile, whose MFMAs have been issued: refill it with the sub-tile after the next
      if (ks + 2 * kQkStripe < key_hi) issue(ks + 2 * kQkStripe, kc);
      mfma_sub(kn, nxt);
      v[0] = front(0, cur[0]);
      v[1] = front(1, cur[1]);
#pragma unroll
      for (int g = 0; g < 2 * KK; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);   // eight vector instructions of the statistics
      }
      // the statistics are complete here (they must not sink below the branches that follow)
      asm volatile("" ::"v"(v[0]), "v"(v[1]), "v"(s_run[0]), "v"(s_run[1]), "v"(m_run[0]), "v"(m_run[1]));
      back(key0, cur, v);
      ks += kQkStripe;
    };
    // the wave's last sub-tile of the walk (the only one that can reach past the end of the keys)
    auto last = [&](qk_f32x16 (&cur)[2]) __attribute__((always_inline)) {
      const int key0 = ks + 4 * half;
      mask_sub(ks, cur);
      const float v[2] = {front(0, cur[0]), front(1, cur[1])};
      back(key0, cur, v);
    };
    int rem = (key_hi - ks + kQkStripe - 1) / kQkStripe;   // sub-tiles of this wave still to finish (>= 1); the current one is in accA
    while (rem >= 3) {
      pstep(accA, accB, kfA, kfB);
      pstep(accB, accA, kfB, kfA);
      rem -= 2;
    }
    if (rem == 2) {
      pstep(accA, accB, kfA, kfB);
      last(accB);
    } else {
      last(accA);
    }
  };
  // The bounds of the wave's 8 rows at once: 8 lanes per row, NE values per lane (NaN: no value).  Bisection from lo
  // (reached by `reach` >= K values of the row) towards the largest value until at most K + slack values are at or above
  // lo, or lo cannot be told from the K-th largest: lo stays at or below that one throughout.
  const int grow = wv * RPW + (lane >> 3), gl = lane & 7;
  auto bisect = [&](const auto& x, auto ne_c, float& lo, uint32_t reach, uint32_t slack, int steps) __attribute__((always_inline)) {
    constexpr int NE = decltype(ne_c)::value;
    float hi = x[0];
#pragma unroll
    for (int j = 1; j < NE; ++j) hi = fmaxf(hi, x[j]);
    hi = max_8(hi);
    if (__any(lo == -INFINITY)) {                        // no bound yet: the smallest finite value, if enough reach it
      float mn = INFINITY;
#pragma unroll
      for (int j = 0; j < NE; ++j) mn = fminf(mn, x[j] > -INFINITY ? x[j] : INFINITY);
      mn = -max_8(-mn);
      uint32_t c = 0;
#pragma unroll
      for (int j = 0; j < NE; ++j) c += x[j] >= mn ? 1u : 0u;
      c = sum_8(c);
      if (lo == -INFINITY && c >= (uint32_t)topk) {
        lo = mn;
        reach = c;
      }
    }
#pragma unroll 1
    for (int it = 0; it < steps; ++it) {
      const float mid = lo + 0.5f * (hi - lo);
      const bool open = reach > (uint32_t)topk + slack && mid > lo && mid <= hi;   // (false for infinities and NaN)
      if (!__any(open)) break;
      uint32_t c = 0;
#pragma unroll
      for (int j = 0; j < NE; ++j) c += x[j] >= mid ? 1u : 0u;
      c = sum_8(c);
      if (open) {
        if (c >= (uint32_t)topk) {
          lo = mid;
          reach = c;
        } else {
          hi = mid;
        }
      }
    }
  };
  // Between the chunks: new bounds, and the entries below them leave the lists (an overflowed list sends its row to the
  // fallback).
  auto update_lists = [&](uint32_t slack, int steps, auto ne_c) __attribute__((always_inline)) {
    constexpr int NE = decltype(ne_c)::value;
    const uint32_t c = S.cnt[grow];
    const bool over = c > (uint32_t)kQkCand || S.ovf[grow];
    float lo = S.bound[grow];
    float x[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const float v = S.cand_x[grow][gl + 8 * j];
      x[j] = gl + 8 * j < (int)c ? v : __builtin_nanf("");
    }
    if (c < (uint32_t)topk) lo = -INFINITY;              // cannot happen for a row of finite logits: keeps everything
    else bisect(x, ne_c, lo, c, slack, steps);
    // in order, 16 entries of a lane at a time: no entry moves up, so none is overwritten before it is read
    uint32_t kept = 0;
#pragma unroll
    for (int j0 = 0; j0 < NE; j0 += 16) {
      int32_t pos[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) pos[j] = S.cand_p[grow][gl + 8 * (j0 + j)];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const bool keep = x[j0 + j] >= lo;
        const uint32_t in_row = (uint32_t)(__ballot(keep) >> (lane & 56)) & 255u;
        if (keep) {
          const uint32_t at = kept + __popc(in_row & ((1u << gl) - 1u));
          S.cand_x[grow][at] = x[j0 + j];
          S.cand_p[grow][at] = pos[j];
        }
        kept += __popc(in_row);
      }
    }
    if (gl == 0) {
      S.cnt[grow] = over ? 0u : kept;
      S.ovf[grow] = over ? 1u : 0u;
      S.bound[grow] = over || grow >= nrows ? INFINITY : lo;
    }
  };
  // After the first barrier of a meeting no wave reads its queries any more (each does so once per chunk, before its walk);
  // only then may the statistics of the last one take their place in LDS.  Each wave writes its lanes' share of all rows
  // there, and the second barrier stands before the rows are put together.
  auto meet = [&](bool done) __attribute__((always_inline)) {
    __syncthreads();
    if (done) {
      // statistics of a row: its 16 lanes -> log-sum-exp and needle mass
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        S.st_m[mt * 32 + l32][wv * 2 + half] = m_run[mt];
        S.st_s[mt * 32 + l32][wv * 2 + half] = s_run[mt];
        S.st_t[mt * 32 + l32][wv * 2 + half] = t_run[mt];
      }
    }
    const uint32_t slack = done ? 0u : (uint32_t)kQkSlack;
    const int steps = done ? 40 : 24;
    if (__any(S.cnt[grow] > (uint32_t)kQkCand / 2)) update_lists(slack, steps, std::integral_constant<int, kQkCand / 8>{});
    else update_lists(slack, steps, std::integral_constant<int, kQkCand / 16>{});
    __syncthreads();
  };

  // this lane's bounds from the rows' bounds in LDS; the unscaled form is lowered by a few ulps so
  // that a logit whose scaled value reaches the bound never fails the test
  auto load_bounds = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const float raw = (mt * 32 + l32 < nrows ? S.bound[mt * 32 + l32] : INFINITY) / c_log2;
      // (no bound: any finite logit; those of -inf, masked keys among them, weigh nothing)
      bound_raw[mt] = raw == INFINITY ? raw : fmaxf(raw - fabsf(raw) * 4.8e-7f, -3.4028235e38f);
    }
  };
  // Keys of the chunk from n_lo on: as many as came before, in whole stripes, and a small rest of the keys with them.
  // With d = 128 every second workgroup of an XCD (they are dealt to 8 in turn) has its chunk ends half an octave before the others': while one
  // half of the chip meets, the other has the memory to itself.  32 x 8 heads, us: 2600 keys 77.8 -> 76.0, 6000 119.6 -> 116.6, 16384 237.8 -> 231.6, 8 x 8
  // heads x 40000 189.3 -> 184.6.  It costs a meeting more: 1000 keys 42.0 -> 43.2.  Four groups instead of two: 16384 the same, 3000 2 % slower than one.
  // d = 64, 10123 keys: 121.7 -> 122.7.  A row's result does not depend on which half it falls to: chunks end at whole stripes, so that a wave has the same sub-tiles in the same order, and
  // the lists end with the same K entries.  (Only a row whose list overflows in one half alone would come from the fallback there, with other last digits.)
  const bool half_octave = DK == 128 && n >= 5 * kQkFirst && (blockIdx.x >> 3 & 1);
  auto chunk_end = [&](int n_lo) __attribute__((always_inline)) {
    const int hi = half_octave && n_lo == kQkFirst ? n_lo + kQkStripe : 2 * n_lo;
    return n - hi <= hi / 8 ? n : hi;
  };

  int c_lo, c_hi = min(n, kQkFirst);
  {
    // the first chunk: both sub-tiles of the wave in registers
    const int ks[2] = {wv * 32, wv * 32 + kQkStripe};
    qk_f32x16 acc[2][2];
    issue(ks[0], kfA);
    issue(ks[1], kfB);
    __syncthreads();                                  // lists empty, queries there
    load_queries();
    mfma_sub(kfA, acc[0]);
    mfma_sub(kfB, acc[1]);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      mask_sub(ks[j], acc[j]);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        stats(mt, acc[j][mt]);
        needle_mass(mt, ks[j] + 4 * half, acc[j][mt]);
      }
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      float* const mxl = &S.cand_x[mt * 32 + l32][(wv * 2 + half) * 8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        mxl[i] = fmaxf(fmaxf(acc[0][mt][2 * i], acc[0][mt][2 * i + 1]), fmaxf(acc[1][mt][2 * i], acc[1][mt][2 * i + 1])) * c_log2;
    }
    if (c_hi < n) prefetch(c_hi, chunk_end(c_hi));
    __syncthreads();
    float nb = -INFINITY;
    {
      float x[kQkSubsets / 8];
#pragma unroll
      for (int j = 0; j < kQkSubsets / 8; ++j) x[j] = S.cand_x[grow][gl + 8 * j];
      bisect(x, std::integral_constant<int, kQkSubsets / 8>{}, nb, kQkSubsets, 2, 24);
    }
    __syncthreads();                                  // the maxima have been read: the lists may fill
    if (gl == 0) S.bound[grow] = grow < nrows ? nb : INFINITY;
    __syncthreads();
    load_bounds();
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (ks[j] < n) {
        float mx[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) mx[mt] = max_16(acc[j][mt]);
        collect(ks[j] + 4 * half, acc[j], mx);
      }
  }
  for (;;) {
    const bool done = c_hi >= n;
    // every list now holds all logits so far that are at or above the row's bound, hence the K largest
    meet(done);
    if (done) break;
    load_queries();
    load_bounds();
    c_lo = c_hi;
    c_hi = chunk_end(c_lo);
    walk(c_lo, c_hi,
         [&](int mt, const qk_f32x16& a) __attribute__((always_inline)) { return stats(mt, a); },
         [&](int key0, const qk_f32x16 (&a)[2], const float (&mx)[2]) __attribute__((always_inline)) {
           needle_mass(0, key0, a[0]);
           needle_mass(1, key0, a[1]);
           collect(key0, a, mx);
         });
    if (c_hi < n) prefetch(c_hi, chunk_end(c_hi));
  }
  {
    const float m0 = S.st_m[grow][gl], m1 = S.st_m[grow][gl + 8];
    const float M = max_8(fmaxf(m0, m1));
    const float mu = M == -INFINITY ? 0.f : M;
    const float f0 = __builtin_amdgcn_exp2f(m0 - mu), f1 = __builtin_amdgcn_exp2f(m1 - mu);
    const float ssum = sum_8(S.st_s[grow][gl] * f0 + S.st_s[grow][gl + 8] * f1);
    const float tsum = sum_8(S.st_t[grow][gl] * f0 + S.st_t[grow][gl + 8] * f1);
    const float lse = M + log2f(ssum);
    const double tnw = (double)tsum / (double)ssum;
    const uint32_t c = S.cnt[grow];
    const bool over = S.ovf[grow] != 0;
    float* const rec = nsplit > 1 ? part + ((rowid0 + min(grow, nrows - 1)) * nsplit + split) * qk_record(topk) : nullptr;
    double wo = 0.0, wd = 0.0;
    for (uint32_t i = gl; i < c; i += 8) {
      const float x = S.cand_x[grow][i];
      const int32_t pos = S.cand_p[grow][i];
      uint32_t rank = 0;
      if (c > (uint32_t)topk)                          // larger logit first, equal logits by lower position
        for (uint32_t j = 0; j < c; ++j) {
          const float xj = S.cand_x[grow][j];
          rank += (xj > x || (xj == x && S.cand_p[grow][j] < pos)) ? 1u : 0u;
        }
      if (rec) {
        if (c <= (uint32_t)topk) rank = i;
        if (grow < nrows && rank < (uint32_t)topk) {
          rec[4 + rank] = x;
          rec[4 + topk + rank] = __int_as_float(pos + key_base);
        }
      } else if (rank < (uint32_t)topk) {
        const double wgt = (double)__builtin_amdgcn_exp2f(x - lse);
        if (pos >= needle_start && pos < ne) wo += wgt; else wd += wgt;
      }
    }
    if (rec) {
      if (grow < nrows) {
        for (uint32_t i = c + gl; i < (uint32_t)topk; i += 8) rec[4 + i] = __builtin_nanf("");   // (fewer than K keys)
        if (gl == 0) {
          rec[0] = M;
          rec[1] = ssum;
          rec[2] = tsum;
          rec[3] = over ? 1.f : 0.f;
        }
      }
      return;
    }
    wo = sum_8(wo);
    wd = sum_8(wd);
    if (gl == 0 && grow < nrows) {
      overflow[rowid0 + grow] = over ? 1 : 0;
      if (!over) {
        const double WS = fmax(0.0, tnw - wo);
        double* cdst = cells + (rowid0 + grow) * 4;
        cdst[0] = wo;
        cdst[1] = wd;
        cdst[2] = WS;
        cdst[3] = 1.0 - wo - wd - WS;                  // a softmax row sums to one
      }
    }
  }
}

// The key ranges of a row put together, one wave per row: statistics, the K largest of the ranges' K largest logits (NE
// of them per lane) and the row's cells.  Bound by the round trip of its loads; 512 rows x 32 ranges x 32 entries: 5 us.
template <int NE>
__global__ __launch_bounds__(256) void qk_merge_kernel(const float* __restrict__ part, int64_t rows, int nsplit, int topk,
                                                       int needle_start, int needle_len, double* __restrict__ cells,
                                                       unsigned char* __restrict__ overflow) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int record = qk_record(topk);
  const float* const rec = part + row * nsplit * record;
  float x[NE];
  int32_t pos[NE];
  const int entries = nsplit * topk;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int e = min(j * 64 + lane, entries - 1), sp = e / topk;
    const float* const at = rec + sp * record + 4 + (e - sp * topk);
    x[j] = at[0];
    pos[j] = __float_as_int(at[topk]);
  }
  const float* const head = rec + min(lane, nsplit - 1) * record;
  const float m = lane < nsplit ? head[0] : -INFINITY, sm = lane < nsplit ? head[1] : 0.f, tm = lane < nsplit ? head[2] : 0.f;
  const bool over = __any(lane < nsplit && head[3] != 0.f);
#pragma unroll
  for (int j = 0; j < NE; ++j)
    if (j * 64 + lane >= entries) x[j] = __builtin_nanf("");
  auto wave_max = [](float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
  };
  const float M = wave_max(m), mu = M == -INFINITY ? 0.f : M;
  const float f = __builtin_amdgcn_exp2f(m - mu);
  const float ssum = wave_sum<float>(sm * f), tsum = wave_sum<float>(tm * f);
  const float lse = M + log2f(ssum);
  const double tnw = (double)tsum / (double)ssum;

  // a value that exactly K entries reach, if equal logits allow it, by bisection as in qk_cells_kernel
  auto reaching = [&](float v) __attribute__((always_inline)) {
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < NE; ++j) c += (uint32_t)__popcll(__ballot(x[j] >= v));
    return c;
  };
  float hi = x[0], lo = INFINITY;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    hi = fmaxf(hi, x[j]);
    lo = fminf(lo, x[j] > -INFINITY ? x[j] : INFINITY);
  }
  hi = wave_max(hi);
  lo = -wave_max(-lo);
  uint32_t reach = reaching(lo);
  if (reach < (uint32_t)topk) lo = -INFINITY;
#pragma unroll 1
  for (int it = 0; it < 48; ++it) {
    const float mid = lo + 0.5f * (hi - lo);
    if (!(reach > (uint32_t)topk && mid > lo && mid <= hi)) break;
    const uint32_t c = reaching(mid);
    if (c >= (uint32_t)topk) {
      lo = mid;
      reach = c;
    } else {
      hi = mid;
    }
  }
  double wo = 0.0, wd = 0.0;
#pragma unroll
  for (int j = 0; j < NE; ++j)
    if (x[j] >= lo) {
      uint32_t rank = 0;
      if (reach > (uint32_t)topk)                        // larger logit first, equal logits by lower position
        for (int e = 0; e < entries; ++e) {
          const float* const at = rec + e / topk * record + 4 + e % topk;
          rank += (at[0] > x[j] || (at[0] == x[j] && __float_as_int(at[topk]) < pos[j])) ? 1u : 0u;
        }
      if (rank < (uint32_t)topk) {
        const double wgt = (double)__builtin_amdgcn_exp2f(x[j] - lse);
        if (pos[j] >= needle_start && pos[j] < needle_start + needle_len) wo += wgt; else wd += wgt;
      }
    }
  wo = wave_sum<double>(wo);
  wd = wave_sum<double>(wd);
  if (lane == 0) {
    overflow[row] = over ? 1 : 0;
    if (!over) {
      const double WS = fmax(0.0, tnw - wo);
      double* cdst = cells + row * 4;
      cdst[0] = wo;
      cdst[1] = wd;
      cdst[2] = WS;
      cdst[3] = 1.0 - wo - wd - WS;
    }
  }
}

// Rows flagged by qk_cells_kernel: the row's weights are written to this workgroup's slot of the
// workspace (plain dot products, softmax in three sweeps) and go through the general path of the
// row kernel, which handles any number of equal weights.
template <int DK>
__global__ __launch_bounds__(kS1Threads) void qk_fallback_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kmat,
                                                                 int Hq, int Hkv, int T, int n, int64_t nrows_total,
                                                                 int needle_start, int needle_len, int topk, float c_log2,
                                                                 const unsigned char* __restrict__ overflow, float* __restrict__ slots,
                                                                 double* __restrict__ cells) {
  __shared__ RowLds<kS1Threads> rowlds;
  __shared__ float qs[DK];
  __shared__ float red[kS1Threads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int G = Hq / Hkv;
  float* W = slots + (int64_t)blockIdx.x * n;
  auto block_max = [&](float v) {
#pragma unroll
    for (int dlt = 32; dlt > 0; dlt >>= 1) v = fmaxf(v, __shfl_xor(v, dlt, 64));
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    float o = red[0];
    for (int i = 1; i < kS1Threads / 64; ++i) o = fmaxf(o, red[i]);
    return o;
  };
  auto block_add = [&](float v) {
    v = wave_sum<float>(v);
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    float o = red[0];
    for (int i = 1; i < kS1Threads / 64; ++i) o += red[i];
    return o;
  };
  // rows blockIdx.x, blockIdx.x + gridDim.x, ... are this workgroup's; their flags are read 256 at a time
  __shared__ int64_t todo[kS1Threads];
  __shared__ uint32_t ntodo;
  for (int64_t base = blockIdx.x; base < nrows_total; base += (int64_t)gridDim.x * kS1Threads) {
    __syncthreads();
    if (tid == 0) ntodo = 0;
    __syncthreads();
    const int64_t mine = base + (int64_t)tid * gridDim.x;
    if (mine < nrows_total && overflow[mine]) todo[atomicAdd(&ntodo, 1u)] = mine;
    __syncthreads();
    const uint32_t cnt = ntodo;
  for (uint32_t it = 0; it < cnt; ++it) {
    const int64_t row = todo[it];
    const int64_t hq_l = row / T;                     // l * Hq + hq
    const int l = (int)(hq_l / Hq), hq = (int)(hq_l % Hq);
    const uint16_t* kb = kmat + ((int64_t)l * Hkv + hq / G) * n * DK;
    __syncthreads();
    for (int p = tid; p < DK; p += kS1Threads) qs[p] = __uint_as_float((uint32_t)q[row * DK + p] << 16);
    __syncthreads();
    float mx = -INFINITY;
    for (int j = tid; j < n; j += kS1Threads) {
      float acc = 0.f;
      for (int p = 0; p < DK; p += 2) {
        const uint32_t pr = *reinterpret_cast<const uint32_t*>(kb + (int64_t)j * DK + p);
        acc = fmaf(qs[p], __uint_as_float(pr << 16), acc);
        acc = fmaf(qs[p + 1], __uint_as_float(pr & 0xffff0000u), acc);
      }
      const float x = acc * c_log2;
      W[j] = x;
      mx = fmaxf(mx, x);
    }
    mx = block_max(mx);
    float sum = 0.f;
    for (int j = tid; j < n; j += kS1Threads) {
      const float e = __builtin_amdgcn_exp2f(W[j] - mx);
      W[j] = e;
      sum += e;
    }
    sum = block_add(sum);
    const float inv = 1.f / sum;
    for (int j = tid; j < n; j += kS1Threads) W[j] *= inv;
    __threadfence_block();
    __syncthreads();
    row_cells_general<kS1Threads, true>(W, n, needle_start, needle_len, topk, cells + row * 4, rowlds);
    __syncthreads();
  }
  }
}

}  // namespace slkv

using namespace slkv;

extern "C" size_t slkv_score_heads_workspace_bytes(int32_t L, int32_t H, int32_t T, int64_t n) {
  (void)n;
  if (L < 1 || H < 1 || T < 1) return 0;
  return (size_t)L * H * T * 4 * sizeof(double);
}

namespace {

slkv_status run_score_heads(const float* d_rows, int32_t L, int32_t H, int32_t T, int64_t n, int64_t needle_start,
                            int32_t needle_len, int32_t topk, double* d_acc, double* d_scores, void* d_workspace,
                            size_t workspace_bytes, void* hip_stream, const slkv_score_params* prm, bool fresh) {
  if (!d_rows || !d_acc || !d_workspace) return fail(SLKV_ERR_NULL, "d_rows, d_acc and d_workspace are required");
  if (L < 1 || H < 1 || T < 1 || n < 1) return fail(SLKV_ERR_BAD_ARG, "L, H, T, n must be >= 1");
  if (n >= (int64_t(1) << 31)) return fail(SLKV_ERR_BAD_ARG, "n >= 2^31");
  const int64_t nrows = (int64_t)L * H * T;
  if (nrows >= (int64_t(1) << 31)) return fail(SLKV_ERR_BAD_ARG, "L*H*T >= 2^31");
  if (needle_len < 1 || needle_start < 0 || needle_start + needle_len > n)
    return fail(SLKV_ERR_BAD_ARG, "needle [%lld, +%d) outside [0, %lld)", (long long)needle_start, needle_len, (long long)n);
  if (topk < 1 || topk > n) return fail(SLKV_ERR_BAD_ARG, "topk %d outside 1..n", topk);
  const void* ptrs[] = {d_rows, d_acc, d_scores, d_workspace};
  for (const void* ptr : ptrs)
    if (reinterpret_cast<uintptr_t>(ptr) % 16) return fail(SLKV_ERR_BAD_ARG, "device pointer %p not 16-byte aligned", ptr);
  const size_t need = slkv_score_heads_workspace_bytes(L, H, T, n);
  if (workspace_bytes < need) return fail(SLKV_ERR_WORKSPACE, "workspace %zu < %zu bytes", workspace_bytes, need);

  hipStream_t st = (hipStream_t)hip_stream;
  double* cells = (double*)d_workspace;
  // Whole 16-byte groups of a row, up to three floats of the row before it included: the threads of a row
  // hold them.  Up to K = kS1TopK the list of one wave has room for all of them and half as many
  // again (2048 rows of 16384 weights: K = 64 35 us, K = 65 210 us).
  //   The form is the smallest that holds the row: slots beyond its end cost as much as others, and so do waves beyond those that
  // four workgroups to a CU need to read while they rank: above 4096 groups three workgroups of 256 threads with 18 to 28 groups each, not two of 512, and up to
  // 11264 groups two of 512 threads, not one of 1024.  512 MiB of rows, us, with 4, 8 or 16 groups a thread alone / with all forms: 1030 weights 236 / 217, 2052
  // 146 / 136, 4100 127 / 99, 6000 96 / 88, 8196 128 / 95, 9000 119 / 92, 12000 96 / 84, 16390 172 / 88, 20000 144 / 95, 24000 125 / 93, 26000 120 / 107,
  // 33000 235 / 106, 40000 202 / 96, 45000 188 / 97; 4096 90, 8192 85, 16384 88, 32760 104 (the same form).  Each form against the next larger one, at its longest rows less 256
  // weights: 64 threads x 6 154 / 161, x 8 124 / 137, x 10 113 / 115 (rows of no whole groups 117 / 122), x 12 99 / 105, x 16 86 / 97; 128 x 10 81 / 84, x 12 80 / 87, x 14 79 / 83, x 16
  // 79 / 88; 256 x 10 78 / 80, x 12 81 / 87, x 14 80 / 83, x 16 80 / 83, x 18 80 / 92, x 20 87 / 93, x 24 84 / 88, x 28 83 / 97; 512 x 16 91 / 93, x 18 91 / 97, x 20 85 / 87, x 22 84 / 151.  Below 2000 weights the time is that of the instructions
  // of a row (bound, list, ranks), which one wave executes.
  const int64_t groups = (n % 4 == 0 ? n : n + 3) / 4;
  {
    ScopedKernelTimer tm(SLKV_K_ROW_CELLS, st);
    bool launched = false;
    auto launch = [&](auto nt, auto ng, auto mw) {
      constexpr int NT = decltype(nt)::value, NG = decltype(ng)::value, MW = decltype(mw)::value;
      if (launched || (NG && (topk > kS1TopK || n < 4 || groups > NT * NG))) return;
      launched = true;
      auto rows = [&](auto rows_c) {
        SLKV_LAUNCH((row_cells_kernel<NT, NG, decltype(rows_c)::value, MW>), dim3((unsigned)nrows), dim3(NT), 0, st, d_rows, (int32_t)n,
                    (int32_t)needle_start, needle_len, topk, cells);
      };
      // 512 MiB to 1 GiB of rows of a multiple of 16 KiB, us a GiB, in one order / four: 8192 weights 157 / 152, 12288 158.5 / 154.5, 16384 164.5 / 159, 20480 164 / 154.5; not
      // 4096 157 / 157, 24576 157 / 158.5, 28672 156 / 156, 32768 166 / 170.5, 36864 163 / 166.5, 40960 159 / 161, 45056 158.5 / 160.
      constexpr bool kAligned = (NT == 128 || NT == 256) && NG > 0 && NG <= 20 && NT * NG % 1024 == 0;   // (such rows fill their form)
      if (n % 4 != 0) rows(std::integral_constant<int, kRowsAny>{});
      else if (kAligned && n % 4096 == 0) rows(std::integral_constant<int, (kAligned ? kRowsAligned : kRowsWhole)>{});
      else rows(std::integral_constant<int, kRowsWhole>{});
    };
    auto forms = [&](auto nt, auto mw, auto... ng) { (launch(nt, ng, mw), ...); };   // by groups a thread
#define SLKV_C(x) std::integral_constant<int, x>{}
    forms(SLKV_C(64), SLKV_C(4), SLKV_C(4));
    forms(SLKV_C(64), SLKV_C(5), SLKV_C(6), SLKV_C(8));
    forms(SLKV_C(64), SLKV_C(4), SLKV_C(10), SLKV_C(12), SLKV_C(16));
    forms(SLKV_C(128), SLKV_C(5), SLKV_C(10), SLKV_C(12));
    forms(SLKV_C(128), SLKV_C(4), SLKV_C(14), SLKV_C(16));
    forms(SLKV_C(256), SLKV_C(5), SLKV_C(10), SLKV_C(12));
    forms(SLKV_C(256), SLKV_C(4), SLKV_C(14), SLKV_C(16));
    forms(SLKV_C(256), SLKV_C(3), SLKV_C(18), SLKV_C(20), SLKV_C(24), SLKV_C(28));
    forms(SLKV_C(512), SLKV_C(4), SLKV_C(16), SLKV_C(18), SLKV_C(20), SLKV_C(22));
    forms(SLKV_C(1024), SLKV_C(4), SLKV_C(16));
    forms(SLKV_C(kS1Threads), SLKV_C(4), SLKV_C(0));
#undef SLKV_C
  }
  const int heads = L * H;
  {
    ScopedKernelTimer tm(SLKV_K_HEAD_REDUCE, st);
    if (prm)
      SLKV_LAUNCH(head_reduce_kernel<8>, dim3((heads + kReduceHeads - 1) / kReduceHeads), dim3(64 * kReduceHeads), 0, st,
                  (const double*)cells, heads, T, d_acc,
                  d_scores, (int)fresh, (int)(prm->aggregation == SLKV_AGG_MACRO), prm->use_wo, prm->use_wd, prm->use_ws);
    else
      SLKV_LAUNCH(head_reduce_kernel<5>, dim3((heads + kReduceHeads - 1) / kReduceHeads), dim3(64 * kReduceHeads), 0, st,
                  (const double*)cells, heads, T, d_acc,
                  d_scores, (int)fresh, 0, 1, 1, 1);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SLKV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return SLKV_OK;
}

}  // namespace

extern "C" slkv_status slkv_score_heads(const float* d_rows, int32_t L, int32_t H, int32_t T, int64_t n,
                                        int64_t needle_start, int32_t needle_len, int32_t topk, double* d_acc,
                                        double* d_scores, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  clear_error();
  return run_score_heads(d_rows, L, H, T, n, needle_start, needle_len, topk, d_acc, d_scores, d_workspace, workspace_bytes,
                         hip_stream, nullptr, false);
}

namespace {

slkv_status check_score_params(const slkv_score_params* params) {
  if (params->struct_size != sizeof(slkv_score_params))
    return fail(SLKV_ERR_BAD_ARG, "params.struct_size %u != %zu", params->struct_size, sizeof(slkv_score_params));
  if (params->aggregation != SLKV_AGG_MICRO && params->aggregation != SLKV_AGG_MACRO)
    return fail(SLKV_ERR_BAD_ARG, "unknown aggregation %d", params->aggregation);
  const int32_t flags[3] = {params->use_wo, params->use_wd, params->use_ws};
  for (int32_t f : flags)
    if (f != 0 && f != 1) return fail(SLKV_ERR_BAD_ARG, "use_wo / use_wd / use_ws must be 0 or 1");
  if (params->reserved != 0) return fail(SLKV_ERR_BAD_ARG, "params.reserved must be 0");
  return SLKV_OK;
}

}  // namespace

extern "C" slkv_status slkv_score_heads_ex(const slkv_score_params* params, const float* d_rows, int32_t L, int32_t H,
                                           int32_t T, int64_t n, int64_t needle_start, int32_t needle_len, int32_t topk,
                                           double* d_acc, double* d_scores, void* d_workspace, size_t workspace_bytes,
                                           void* hip_stream) {
  clear_error();
  if (!params) return fail(SLKV_ERR_NULL, "params is NULL");
  const slkv_status ps = check_score_params(params);
  if (ps != SLKV_OK) return ps;
  return run_score_heads(d_rows, L, H, T, n, needle_start, needle_len, topk, d_acc, d_scores, d_workspace, workspace_bytes,
                         hip_stream, params, false);
}

extern "C" slkv_status slkv_score_heads_first(const slkv_score_params* params, const float* d_rows, int32_t L, int32_t H,
                                              int32_t T, int64_t n, int64_t needle_start, int32_t needle_len, int32_t topk,
                                              double* d_acc, double* d_scores, void* d_workspace, size_t workspace_bytes,
                                              void* hip_stream) {
  clear_error();
  if (params) {
    const slkv_status ps = check_score_params(params);
    if (ps != SLKV_OK) return ps;
  }
  return run_score_heads(d_rows, L, H, T, n, needle_start, needle_len, topk, d_acc, d_scores, d_workspace, workspace_bytes,
                         hip_stream, params, true);
}

// ------------------------------------------------------------------ Stage 1 from queries and keys

namespace {

struct QkLayout {
  size_t cells_bytes, flags_bytes, slots_bytes, off_flags, off_slots, total;
};

QkLayout qk_layout(int64_t rows, int64_t n) {
  auto align = [](size_t x) { return (x + 255) / 256 * 256; };
  QkLayout w;
  w.cells_bytes = align((size_t)rows * 4 * sizeof(double));
  w.flags_bytes = align((size_t)rows);
  w.slots_bytes = align((size_t)kQkFallbackWGs * (size_t)n * sizeof(float));
  w.off_flags = w.cells_bytes;
  w.off_slots = w.off_flags + w.flags_bytes;
  w.total = w.off_slots + w.slots_bytes;
  return w;
}

// LDS above the default limit is requested once per kernel instance and device.
template <int DK>
hipError_t qk_prepare() {
  static std::mutex mu;
  static uint64_t done = 0;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t(1) << dev) : 0;
  if (!(done & bit)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&qk_cells_kernel<DK>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)sizeof(QkLds));
    if (e != hipSuccess) return e;
    done |= bit;
  }
  return hipSuccess;
}

// Key ranges per head.  256 workgroups run at once, each some kStartUs for its start, end and meetings and then its keys
// one after the other; the ranges' results take another launch.  (At a range of 512 keys a workgroup does little but
// start.)  The records of the ranges lie where the fallback keeps its rows later.
// 24 groups of 64 rows x 6013 keys x d 128: 158 -> 54 us; 10 x 2318 x d 64: 100 -> 37; 24 x 8202: 197 -> 64; 270 groups (a little
// more than run at once) x 16248: 493 -> 224.
int qk_splits(int64_t groups, int64_t rows, int32_t n, int d, int32_t topk, size_t slots_bytes) {
  constexpr double kStartUs = 12, kMergeUs = 5, kUsPerKeyAndDim = 1.1e-4;
  const int64_t fit = (int64_t)(slots_bytes / ((size_t)rows * (size_t)qk_record(topk) * sizeof(float)));
  const int most = (int)std::min<int64_t>({(int64_t)kQkMaxSplit, (int64_t)n / 512, fit});
  int best = 1;
  double best_us = 0;
  for (int s = 1; s <= std::max(most, 1); ++s) {
    const double us = (double)((groups * s + 255) / 256) * (kStartUs + kUsPerKeyAndDim * d * n / s) + (s > 1 ? kMergeUs : 0);
    if (s == 1 || us < best_us) {
      best = s;
      best_us = us;
    }
  }
  return best;
}

template <int DK>
slkv_status qk_launch(const uint16_t* q, const uint16_t* k, int32_t L, int32_t Hq, int32_t Hkv, int32_t T, int32_t n,
                      int32_t needle_start, int32_t needle_len, int32_t topk, double* d_acc, double* d_scores,
                      unsigned char* ws, const QkLayout& w, hipStream_t st, bool fresh) {
  hipError_t pe = qk_prepare<DK>();
  if (pe != hipSuccess) return fail(SLKV_ERR_HIP, "kernel set-up failed: %s", hipGetErrorString(pe));
  const int G = Hq / Hkv, R = G * T, rowgroups = (R + kQkRows - 1) / kQkRows;
  const int64_t rows = (int64_t)L * Hq * T;
  double* cells = (double*)ws;
  unsigned char* flags = ws + w.off_flags;
  float* slots = (float*)(ws + w.off_slots);
  const float c_log2 = (float)(1.4426950408889634 / std::sqrt((double)DK));
  const int64_t groups = (int64_t)L * Hkv * rowgroups;
  const int want = qk_splits(groups, rows, n, DK, topk, w.slots_bytes);
  const int stripes = (n + kQkStripe - 1) / kQkStripe;
  const int range = (stripes + want - 1) / want * kQkStripe, nsplit = (n + range - 1) / range;
  {
    ScopedKernelTimer tm(SLKV_K_QK_CELLS, st);
    SLKV_LAUNCH(qk_cells_kernel<DK>, dim3((unsigned)(groups * nsplit)), dim3(kQkThreads), sizeof(QkLds), st, q, k, Hq, Hkv,
                T, n, rowgroups, nsplit, range, needle_start, needle_len, topk, c_log2, cells, flags, slots);
    if (nsplit > 1) {
      const dim3 grid((unsigned)((rows + 3) / 4));
      if (nsplit * topk <= 8 * 64)
        SLKV_LAUNCH(qk_merge_kernel<8>, grid, dim3(256), 0, st, (const float*)slots, rows, nsplit, topk, needle_start, needle_len, cells, flags);
      else
        SLKV_LAUNCH(qk_merge_kernel<kQkMaxSplit>, grid, dim3(256), 0, st, (const float*)slots, rows, nsplit, topk, needle_start, needle_len, cells,
                    flags);
    }
  }
  {
    ScopedKernelTimer tm(SLKV_K_QK_FALLBACK, st);
    SLKV_LAUNCH(qk_fallback_kernel<DK>, dim3(kQkFallbackWGs), dim3(kS1Threads), 0, st, q, k, Hq, Hkv, T, n, rows, needle_start,
                needle_len, topk, c_log2, (const unsigned char*)flags, slots, cells);
  }
  const int heads = L * Hq;
  {
    ScopedKernelTimer tm(SLKV_K_HEAD_REDUCE, st);
    SLKV_LAUNCH(head_reduce_kernel<5>, dim3((heads + kReduceHeads - 1) / kReduceHeads), dim3(64 * kReduceHeads), 0, st,
                  (const double*)cells, heads, T, d_acc,
                d_scores, (int)fresh, 0, 1, 1, 1);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SLKV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return SLKV_OK;
}

}  // namespace

extern "C" size_t slkv_score_heads_qk_workspace_bytes(int32_t L, int32_t Hq, int32_t T, int64_t n) {
  if (L < 1 || Hq < 1 || T < 1 || n < 1) return 0;
  return qk_layout((int64_t)L * Hq * T, n).total;
}

static slkv_status run_score_heads_qk(const void* d_q, const void* d_k, int32_t L, int32_t Hq, int32_t Hkv, int32_t T,
                                      int64_t n, int32_t d, int64_t needle_start, int32_t needle_len, int32_t topk,
                                      double* d_acc, double* d_scores, void* d_workspace, size_t workspace_bytes,
                                      void* hip_stream, bool fresh) {
  clear_error();
  if (!d_q || !d_k || !d_acc || !d_workspace) return fail(SLKV_ERR_NULL, "d_q, d_k, d_acc and d_workspace are required");
  if (L < 1 || Hq < 1 || Hkv < 1 || T < 1 || n < 1) return fail(SLKV_ERR_BAD_ARG, "L, Hq, Hkv, T, n must be >= 1");
  if (Hq % Hkv) return fail(SLKV_ERR_BAD_ARG, "Hq %% Hkv != 0");
  if (d != 64 && d != 128) return fail(SLKV_ERR_UNSUPPORTED, "head_dim %d (supported: 64, 128)", d);
  if (n * d * 2 >= (int64_t(1) << 31)) return fail(SLKV_ERR_UNSUPPORTED, "one head's keys span 2 GiB or more");
  const int64_t rows = (int64_t)L * Hq * T;
  if (rows >= (int64_t(1) << 31) || (int64_t)L * Hkv * (((int64_t)(Hq / Hkv) * T + kQkRows - 1) / kQkRows) >= (int64_t(1) << 31))
    return fail(SLKV_ERR_BAD_ARG, "too many rows");
  if (needle_len < 1 || needle_start < 0 || needle_start + needle_len > n)
    return fail(SLKV_ERR_BAD_ARG, "needle [%lld, +%d) outside [0, %lld)", (long long)needle_start, needle_len, (long long)n);
  if (topk < 1 || topk > n) return fail(SLKV_ERR_BAD_ARG, "topk %d outside 1..n", topk);
  if (topk > 64) return fail(SLKV_ERR_UNSUPPORTED, "topk %d > 64 (use slkv_score_heads on materialised rows)", topk);
  const void* ptrs[] = {d_q, d_k, d_acc, d_scores, d_workspace};
  for (const void* ptr : ptrs)
    if (reinterpret_cast<uintptr_t>(ptr) % 16) return fail(SLKV_ERR_BAD_ARG, "device pointer %p not 16-byte aligned", ptr);
  const QkLayout w = qk_layout(rows, n);
  if (workspace_bytes < w.total) return fail(SLKV_ERR_WORKSPACE, "workspace %zu < %zu bytes", workspace_bytes, w.total);
  hipStream_t st = (hipStream_t)hip_stream;
  if (d == 128)
    return qk_launch<128>((const uint16_t*)d_q, (const uint16_t*)d_k, L, Hq, Hkv, T, (int32_t)n, (int32_t)needle_start, needle_len,
                          topk, d_acc, d_scores, (unsigned char*)d_workspace, w, st, fresh);
  return qk_launch<64>((const uint16_t*)d_q, (const uint16_t*)d_k, L, Hq, Hkv, T, (int32_t)n, (int32_t)needle_start, needle_len, topk,
                       d_acc, d_scores, (unsigned char*)d_workspace, w, st, fresh);
}

extern "C" slkv_status slkv_score_heads_qk(const void* d_q, const void* d_k, int32_t L, int32_t Hq, int32_t Hkv, int32_t T,
                                           int64_t n, int32_t d, int64_t needle_start, int32_t needle_len, int32_t topk,
                                           double* d_acc, double* d_scores, void* d_workspace, size_t workspace_bytes,
                                           void* hip_stream) {
  return run_score_heads_qk(d_q, d_k, L, Hq, Hkv, T, n, d, needle_start, needle_len, topk, d_acc, d_scores, d_workspace,
                            workspace_bytes, hip_stream, false);
}

extern "C" slkv_status slkv_score_heads_qk_first(const void* d_q, const void* d_k, int32_t L, int32_t Hq, int32_t Hkv,
                                                 int32_t T, int64_t n, int32_t d, int64_t needle_start, int32_t needle_len,
                                                 int32_t topk, double* d_acc, double* d_scores, void* d_workspace,
                                                 size_t workspace_bytes, void* hip_stream) {
  return run_score_heads_qk(d_q, d_k, L, Hq, Hkv, T, n, d, needle_start, needle_len, topk, d_acc, d_scores, d_workspace,
                            workspace_bytes, hip_stream, true);
}
