// Stage 2b of SurfaceLogicKV (Section 3.4, Eq. 7-8, Algorithm 3) on gfx950:
//   pass 1  score_*<.., 1>  window-query x history-key logits, per-row log-sum-exp of every key chunk
//   (long histories of 16-bit keys: score_sample, score_both, .. , one pass and exact scores only where they decide)
//   pass 2  score_*<.., 2>  the chunks folded into the rows' log-sum-exp, logits again, exp(logit - lse) summed down
//                            the G*w rows -> importance
//   (where the workgroups fit the chip at once: both in one launch, score_*<.., 3>)
//   select                   1-D pooling + per-head top-k (radix select, ordered compaction)
//   gather                   kept K/V rows -> compacted ragged cache
// 16-bit keys: 32x32x16 MFMA, queries held in registers, key tiles staged in LDS (score_q_resident_kernel).  E4M3 keys
// (widened to bf16) and fp32 inputs (32x32x2 fp32 MFMA): keys held in registers, queries staged in LDS
// (score_k_resident_kernel).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "device_utils.h"
#include "launch.h"
#include "slkv_internal.h"

// Development aid, compiled only with -DSLKV_TRACE: clock stamps of chosen workgroups.
#ifdef SLKV_TRACE
__device__ long long slkv_trace_buf[64 * 1024];
#define SLKV_STAMP(wg, slot) do { if (threadIdx.x == 0 && (wg) < 1024) slkv_trace_buf[(wg) * 16 + (slot)] = wall_clock64(); } while (0)
extern "C" int slkv_trace_read(long long* h, int n) {
  return (int)hipMemcpyFromSymbol(h, HIP_SYMBOL(slkv_trace_buf), (size_t)n * sizeof(long long));
}
#else
#define SLKV_STAMP(wg, slot) do {} while (0)
#endif

namespace slkv {

// The (sequence, KV head) segments of a call, as every kernel finds them: segment s = b*hkv + h is head h of
// sequence b.
struct SegShape {
  int n;           // tokens (rows) of the segment; the last w are the window
  int tok_begin;   // its first token (row) in K / V
  int head;        // multiplied by the head stride (0 for a ragged cache)
  int kk;          // history rows to keep; -1 = keep every token
  int score_off;   // offset of the segment in the importance / pooled arrays
};

// The sample that the one pass over a long history starts from (see OneScan): kSampleGroup neighbours out of every kSampleGroup * sample_step keys, four
// keys per position kept, 2048 to 8192 in all: the more are kept, the nearer the threshold lies to the bulk of the scores, where an uncertain one
// takes in more keys.  32 segments of 20 K to 128 K keys, us of the sample and of the chosen keys: 170 kept 24 + 22 (8192 keys whatever is kept: 40 + 22);
// 1500 kept 25 + 39 (2048 keys: 20 + 53; 8192: 39 + 39); 3300 kept 31 + 42 (2048: 19 + 89).
// A workgroup of the kernels that go over the sample, and over the scores before the selection, takes a range of positions with `sampled` such keys (plan_ranges).
constexpr int kSampleGroup = 8, kRangeMost = 6144;   // (6144 positions: the scores and the list of two workgroups fit a CU's LDS)
__device__ __host__ __forceinline__ int sample_step(int m, int kk) {
  const int keys = 4 * kk < 2048 ? 2048 : 4 * kk > 8192 ? 8192 : 4 * kk;
  return m / keys > 4 ? m / keys : 4;
}
__device__ __host__ __forceinline__ int range_len(int m, int kk, int sampled) {
  const int len = sampled * sample_step(m, kk);
  return len < 512 ? 512 : len > kRangeMost ? kRangeMost : len;
}

// Up to kMaxSegPerLaunch segments: everything per segment, in a kernel argument, so that one round of loads from
// it (cold at every launch) answers a workgroup that knows its segment.
struct SegTable {
  int32_t nseg;
  int32_t tok_[kMaxSegPerLaunch], n_[kMaxSegPerLaunch], head_[kMaxSegPerLaunch], kk_[kMaxSegPerLaunch], score_[kMaxSegPerLaunch];
  int32_t out_[kMaxSegPerLaunch + 1];     // first output row of the segment
  int32_t chunk_[kMaxSegPerLaunch + 1];   // prefix of key-chunk counts (0 chunks when not ranked)
  int32_t blk_[kMaxSegPerLaunch + 1];     // prefix of selection-block counts (no block when not ranked)
  int32_t range_[kMaxSegPerLaunch + 1];   // prefix of range counts (see range_len)
  __device__ __forceinline__ int out_off(int s) const { return out_[s]; }
  __device__ __forceinline__ int chunk_begin(int s) const { return chunk_[s]; }
  __device__ __forceinline__ int blk_begin(int s) const { return blk_[s]; }
  __device__ __forceinline__ int range_begin(int s) const { return range_[s]; }
  __device__ __forceinline__ SegShape shape(int s) const { return SegShape{n_[s], tok_[s], head_[s], kk_[s], score_[s]}; }
};

// More segments: what depends on the sequence or the head alone is stored once per sequence or head and the rest
// follows from it, one round of loads later.  The words travel in the kernel argument as well if they fit (a
// decode batch of 32 sequences x 8 heads does), otherwise they are in the workspace, put there by upload_kernel.
// (With everything per segment in the workspace, a launch of 4 us per 64 segments came before the first scoring
// pass: 16 of the decode batch's 97 us.)
// The line is what a kernel argument of 4 KiB holds beside the other arguments: with 8 heads 296 segments of a ragged cache, or 416 of a
// layer call; above it an upload of 900 words at a time comes before the first pass (ragged cache, 8 heads, 200 to 420 rows
// a segment: 296 segments 46.8 us, 304 segments 53.1 us).
constexpr int kArgWords = 900;
struct SegTableBig {
  const int32_t* mem;                     // the words; NULL: words[]
  int32_t nseg, hkv, w, ragged;
  int32_t off_out, off_chunk, off_blk, off_cap;   // where in the words; at 0: first token of every sequence, or (ragged) first row of every segment
  int32_t words[kArgWords];
  // The words in the constant address space: read with scalar loads.  The table is every kernel's first argument.
  typedef const __attribute__((address_space(4))) int32_t* Words;
  __device__ __forceinline__ Words data() const {
    if (mem) return (Words)(uintptr_t)mem;
    return (Words)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(SegTableBig, words) / sizeof(int32_t);
  }
  __device__ __forceinline__ int out_off(int s) const { return data()[off_out + s]; }
  __device__ __forceinline__ int chunk_begin(int s) const { return data()[off_chunk + s]; }
  __device__ __forceinline__ int blk_begin(int s) const { return data()[off_blk + s]; }
  __device__ __forceinline__ SegShape shape(int s) const {
    const Words t = data();
    const int b = s / hkv, h = s - b * hkv, i = ragged ? s : b;
    SegShape r;
    r.tok_begin = t[i];
    r.n = t[i + 1] - r.tok_begin;
    r.head = ragged ? 0 : h;
    const int cap = t[off_cap + h];
    r.kk = r.n <= w || r.n <= cap ? -1 : min(max(cap - w, 0), r.n - w);
    r.score_off = ragged ? r.tok_begin - t[0] : hkv * r.tok_begin + h * r.n;
    return r;
  }
};

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native 16-byte vector (register friendly)

union Pack16 {
  u32x4 u;
  bf16x8 b;
};

typedef float f32x4v __attribute__((ext_vector_type(4)));

// 32x32x16 MFMA on eight 16-bit elements per lane and operand: bfloat16, or IEEE half when F16
// (the registers are typed bf16x8 either way; only the instruction reads them differently).
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <bool F16>
__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Segment of a block / row: the largest s with prefix(s) <= x (prefix non-decreasing, prefix(nseg) > x), for an x that is
// the same in all 64 lanes of a wave (all of them active).  64 prefixes are compared at a time, so that a table of up to 64 segments costs one memory round trip and one of up to 4096 two, not one per
// halving: these lookups come before a workgroup's first key.
template <class F>
__device__ __forceinline__ int find_segment_wave(int nseg, int x, F prefix) {
  const int lane = threadIdx.x & 63;
  int lo = 0, span = nseg;                             // the segment is one of lo .. lo + span - 1
  while (span > 1) {
    const int step = (span + 63) >> 6;
    const bool below = lane * step < span && prefix(min(lo + lane * step, nseg - 1)) <= x;
    const int last = max(__popcll(__ballot(below)) - 1, 0);
    lo += last * step;
    span = min(step, span - last * step);
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Merge two (max, sum) pairs of a running softmax in the log2 domain.
__device__ __forceinline__ void merge_stats(float& m, float& s, float m2, float s2) {
  float mn = fmaxf(m, m2);
  float mu = mn == -INFINITY ? 0.f : mn;
  s = s * fast_exp2(m - mu) + s2 * fast_exp2(m2 - mu);
  m = mn;
}

// Start of the second scoring pass: log-sum-exp (log2 domain) of rows row0 .. of a segment from that of its key
// chunks c0 .. c1 - 1 (part[chunk][row]; -inf for a chunk without keys for the row), in the threads tid < ROWS of the
// workgroup's NT (row row0 + tid).  The chunks of a row are dealt to NT / ROWS threads in turn, whose sums are added
// up in LDS (`fold`: NT entries), so every workgroup of the segment gets the same bits.  +inf for a row without any
// key.  ROWS >= NT: a thread per row.  Every thread must call it; ends with a barrier if LDS was used.
// (The chunk that arrives last at a per-segment ticket did this at the end of the first pass: 4 us there, against
// 0.5 to 3 us here, where the loads travel with those of the keys and queries.)
template <bool SHARED = false>   // SHARED: written by other workgroups of the same launch (see meet_chunks)
__device__ __forceinline__ float fold_rows(const float* __restrict__ part, int c0, int c1, int Rpad, int row0, int rows, int nt,
                                           float2* fold) {
  const int tid = threadIdx.x;
  const int nsub = rows < nt ? nt / rows : 1;
  const int row = nsub > 1 ? tid % rows : tid, sub = nsub > 1 ? tid / rows : 0;
  float mm = -INFINITY, ss = 0.f;
  // batches of loads that are all in flight together: as large as the chunks ask for, since each costs a round trip
  auto batches = [&](auto nb_c) __attribute__((always_inline)) {
    constexpr int NB = decltype(nb_c)::value;
    for (int c = c0 + sub; c < c1; c += NB * nsub) {
      float v[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const float* const p = part + ((int64_t)min(c + u * nsub, c1 - 1) * Rpad + row0 + row);
        v[u] = SHARED ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
      }
#pragma unroll
      for (int u = 0; u < NB; ++u) v[u] = c + u * nsub < c1 ? v[u] : -INFINITY;
      float bm = v[0];
#pragma unroll
      for (int u = 1; u < NB; ++u) bm = fmaxf(bm, v[u]);
      const float mn = fmaxf(mm, bm);
      const float mu = mn == -INFINITY ? 0.f : mn;
      ss *= fast_exp2(mm - mu);
#pragma unroll
      for (int u = 0; u < NB; ++u) ss += fast_exp2(v[u] - mu);
      mm = mn;
    }
  };
  if (sub < nsub && row0 + row < Rpad) {
    if (c1 - c0 <= 16 * nsub) batches(std::integral_constant<int, 16>{});
    else batches(std::integral_constant<int, 32>{});
  }
  if (nsub > 1) {
    fold[tid] = make_float2(mm, ss);
    __syncthreads();
    if (sub == 0)
      for (int v = 1; v < nsub; ++v) {
        const float2 o = fold[v * rows + row];
        merge_stats(mm, ss, o.x, o.y);
      }
    __syncthreads();
  }
  return ss > 0.f ? mm + __builtin_amdgcn_logf(ss) : INFINITY;
}

// As fold_rows, of the sample: a thread per row (tid < rows <= nt).  dense[0], [1] of a row: the keys at either end of the history, which are all in the
// sample; part: the sampled keys of the ranges.  No range counts more than twice their geometric mean: a single sampled key far above the rest (it
// stands for up to 64) would make the row's estimate several times too large, and one such row lowers the bound of all keys.
__device__ __forceinline__ float fold_sample(const float* __restrict__ part, const float* __restrict__ dense, int c0, int c1, int Rpad, int rows) {
  const int row = threadIdx.x;
  float ss = 0.f, mu = 0.f;
  if (row < rows && row < Rpad) {
    constexpr int NB = 32;
    float v[NB];
    const float d0 = dense[row], d1 = dense[Rpad + row];
    auto load = [&](int c) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < NB; ++u) v[u] = part[(int64_t)min(c + u, c1 - 1) * Rpad + row];
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (c + u >= c1) v[u] = -INFINITY;
    };
    float sum = 0.f, used = 0.f;
    for (int c = c0; c < c1; c += NB) {
      load(c);
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        sum += v[u] == -INFINITY ? 0.f : v[u];
        used += v[u] == -INFINITY ? 0.f : 1.f;
      }
    }
    const float cap = used > 0.f ? sum / used + 1.f : -INFINITY;
    const float mm = fmaxf(cap, fmaxf(d0, d1));
    mu = mm == -INFINITY ? 0.f : mm;
    ss = fast_exp2(d0 - mu) + fast_exp2(d1 - mu);
    for (int c = c0; c < c1; c += NB) {
      if (c1 - c0 > NB) load(c);
#pragma unroll
      for (int u = 0; u < NB; ++u) ss += v[u] == v[u] ? fast_exp2(fminf(v[u], cap) - mu) : v[u];
    }
  }
  return ss > 0.f ? mu + __builtin_amdgcn_logf(ss) : INFINITY;
}

// Where the workgroups of a segment that hold its chunks meet inside one launch: a 64-bit word per segment in the
// workspace's header, 64 bytes apart, zero before the launch and cleared by the selection.  The upper 16 bits count the
// chunks whose statistics are in memory, bit c of the others says that the workgroup of chunk c has left.
//   A workgroup waits for the others a bounded time.  They may not be on the chip together (another stream's kernels hold
// CUs, or such a launch of another call does and waits as well), so one that has waited `limit` says so in its chunk's
// bit and leaves its place to those that wait for one; nobody depends on it any more.  The bits are set and the
// count is raised in the same word, so the bits that stand when the count is full are all there will be: who sees it
// full takes its own chunk, and then, one by one, those whose bits it clears.
//   Statistics are stored and read past the caches of the XCDs (agent scope), each store complete before its chunk is
// counted: 0.9 us to store and count, 0.6 to 1.2 for the others to see it, 1.3 to read 32 chunks of 256 rows.  (With a
// release and an acquire fence at that scope, which write back and invalidate the L2s: 8 to 12 us each, 256 workgroups.)
constexpr int kMeetMost = 48, kMeetWords = 8;
constexpr int kMeetSegments = SLKV_WORKSPACE_HEADER_BYTES / (kMeetWords * 8);
typedef unsigned long long meet_t;
// The count of the other chunks has been seen full: the bits that stand; or kMeetLeft: somebody else completes this chunk.  In thread 0 alone.
constexpr meet_t kMeetLeft = ~0ull;
__device__ __forceinline__ meet_t meet_chunks(meet_t* word, int nchunks, int chunk, int limit) {
  const meet_t full = (meet_t)nchunks, bit = 1ull << chunk, bits = (1ull << nchunks) - 1;   // (a word that was not zero names no chunk that is not there)
  meet_t w = __hip_atomic_fetch_add(word, 1ull << kMeetMost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + (1ull << kMeetMost);
  if (w >> kMeetMost == full) return w & bits;
  const long long start = wall_clock64();
  do {
    __builtin_amdgcn_s_sleep(1);
    w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (w >> kMeetMost >= full) return w & bits;         // (more: some have scored a chunk already, see meet_scores)
  } while (wall_clock64() - start < limit);
  w = __hip_atomic_fetch_or(word, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (w >> kMeetMost < full) return kMeetLeft;
  // full meanwhile: this chunk again, unless somebody has taken it
  w = __hip_atomic_fetch_and(word, ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return w & bit ? w & bits & ~bit : kMeetLeft;
}
// A chunk of those in `left` that nobody else completes, or -1.  In thread 0 alone.
__device__ __forceinline__ int meet_take(meet_t* word, meet_t& left) {
  while (left) {
    const int c = __ffsll(left) - 1;
    left &= left - 1;
    if (__hip_atomic_fetch_and(word, ~(1ull << c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> c & 1) return c;
  }
  return -1;
}

// The segment finished in the launch that scores it (PASS 4).  Behind the second pass a workgroup counts the chunks it has scored in the same
// word, up to twice their number, and waits for the others as before.  Whoever sees all scored selects, each the whole segment, and takes slices
// of the kept rows from the next word, of which there are as many as chunks, until none is left.  One that has waited `limit` leaves, without a
// word: the one that counts the last chunk does not wait.  A third word counts the workgroups that touch these words no more; the last one clears them.
__device__ __forceinline__ bool meet_scores(meet_t* word, int nchunks, int scored, int limit) {
  const meet_t full = 2 * (meet_t)nchunks, add = (meet_t)scored << kMeetMost;
  if ((__hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add) >> kMeetMost == full) return true;
  const long long start = wall_clock64();
  do {
    __builtin_amdgcn_s_sleep(1);
    if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> kMeetMost == full) return true;
  } while (wall_clock64() - start < limit);
  return false;
}
__device__ __forceinline__ int meet_slice(meet_t* word) {
  return (int)min(__hip_atomic_fetch_add(word + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), (meet_t)kMeetMost);
}
__device__ __forceinline__ void meet_leave(meet_t* word, int nchunks) {
  if (__hip_atomic_fetch_add(word + 2, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 != (meet_t)nchunks) return;
#pragma unroll
  for (int i = 0; i < 3; ++i) __hip_atomic_store(word + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Per segment: the words of OneScanBounds; smallest, largest and mean rho.
constexpr int kBoundWords = 12, kBoundProbe = 4, kBoundWide = 5, kBoundRho = 6;

// Largest importance of every group of kGroup keys, counted from the segment's first one, for the selection (see select_resident_kernel): where
// a segment's groups begin.  Chunks begin at multiples of kGroup.
constexpr int kGroup = 8;
__device__ __forceinline__ int64_t group_off(int64_t score_off, int seg) { return (score_off >> 3) + seg; }
// Key of a score: its bit pattern; anything that is not a non-negative number (cannot come out of finite inputs) ranks as +infinity,
// so that every phase counts it the same way.
__device__ __forceinline__ uint32_t score_key(float v) {
  const uint32_t u = __float_as_uint(v);
  return u > 0x7f800000u ? 0x7f800000u : u;
}
// Largest of v over each 8 neighbouring lanes, in all of them.
__device__ __forceinline__ uint32_t max_8_lanes(uint32_t v) {
  v = max(v, dpp_move<0xb1>(v, v));        // quad_perm: the neighbour,
  v = max(v, dpp_move<0x4e>(v, v));        // the pair next to them,
  return max(v, dpp_move<0x141>(v, v));    // row_half_mirror: the other four
}

// The two workgroups that share a CU would otherwise run one after the other: the scheduler
// favours the older waves, the older workgroup finishes a third earlier and the younger one spends
// the end of the kernel alone on the CU, one wave per SIMD, with nothing to overlap with.  Waves
// raise their priority on even tiles and drop it on odd ones, so the workgroup that is a tile behind
// wins the issue slots for a tile.  (Measured: -0.7 us per pass on the 32K-prefix shape; the older
// workgroup still ends its loop about 5 us before the younger one.  Four priority levels falling
// with the tile index made pass 1 slower.)
__device__ __forceinline__ void tile_priority(int t) {
  if (t & 1) __builtin_amdgcn_s_setprio(0);
  else __builtin_amdgcn_s_setprio(1);
}

struct GatherArgs {
  const unsigned char* k;
  const unsigned char* v;
  unsigned char* k_out;
  unsigned char* v_out;
  int64_t k_stride_tok, k_stride_head, v_stride_tok, v_stride_head;   // elements
  int lanes_per_row, elt_bytes;
  const int32_t* pos_in;   // optional: original position of every input row (ragged input)
  int32_t* pos_out;        // optional: pos_in at the kept rows
};

constexpr int kSelHaloMax = kMaxPool / 2;
constexpr uint32_t kKeyNone = 0xffffffffu;

// What a scoring launch that also selects and copies (PASS 4) needs beside the scores.
struct FinishArgs {
  GatherArgs ga;
  float* pooled;
  int32_t* kept_idx;
  int64_t* out_offsets;    // or NULL
  int pool_kernel, pool_mode, write_pooled;
  int chunks;              // workgroups of chunks; those behind them copy segments that are not ranked
};

// Rows of a segment to output rows row0 .. row0 + rows - 1, of which pos(i) gives the i-th one's position: four 16-byte pieces of K and V in flight a thread.
template <class F>
__device__ __forceinline__ void copy_rows(const GatherArgs& ga, const SegShape& sg, int64_t row0, int rows, int nthr, F pos) {
  const int lpr = ga.lanes_per_row, shift = __builtin_ctz(lpr), pieces = rows << shift;   // (4 to 32 lanes per row: a power of two)
  const int64_t h = sg.head;
  for (int base = (int)threadIdx.x; base < pieces; base += 4 * nthr) {
    u32x4 kq[4], vq[4];
    int64_t tok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = min(base + u * nthr, pieces - 1), c = idx & (lpr - 1);
      tok[u] = (int64_t)sg.tok_begin + pos(idx >> shift);
      kq[u] = *reinterpret_cast<const u32x4*>(ga.k + (h * ga.k_stride_head + tok[u] * ga.k_stride_tok) * ga.elt_bytes + c * 16);
      vq[u] = *reinterpret_cast<const u32x4*>(ga.v + (h * ga.v_stride_head + tok[u] * ga.v_stride_tok) * ga.elt_bytes + c * 16);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = base + u * nthr;
      if (idx < pieces) {
        const int64_t row = row0 + (idx >> shift), o = (row << shift) * 16 + (idx & (lpr - 1)) * 16;
        *reinterpret_cast<u32x4*>(ga.k_out + o) = kq[u];
        *reinterpret_cast<u32x4*>(ga.v_out + o) = vq[u];
        if (ga.pos_out && (idx & (lpr - 1)) == 0) ga.pos_out[row] = ga.pos_in[tok[u]];
      }
    }
  }
}

// Workgroup `more` of those that copy segments that are not ranked: kFinishRows rows of one, or (kk == 0) of its window.
constexpr int kFinishRowsLog2 = 7;
template <class TAB>
__device__ __forceinline__ void copy_unranked(const TAB& tab, const FinishArgs& fin, int w, int more, int nthr) {
  const int lane = threadIdx.x & 63;
  for (int s0 = 0; s0 < tab.nseg; s0 += 64) {
    const int s = min(s0 + lane, tab.nseg - 1);
    const SegShape sh = tab.shape(s);
    const bool unranked = s0 + lane < tab.nseg && !(sh.kk > 0 && sh.kk < sh.n - w);
    const int rows = unranked ? tab.out_off(s + 1) - tab.out_off(s) : 0;
    const int parts = unranked ? 1 + (max(rows - 1, 0) >> kFinishRowsLog2) : 0, incl = (int)wave_incl_scan((uint32_t)parts);
    const unsigned long long past = __builtin_amdgcn_ballot_w64(incl > more);
    if (past) {
      const int l = __builtin_ctzll(past), seg = s0 + l, first = (more - __builtin_amdgcn_readlane(incl - parts, l)) << kFinishRowsLog2;
      const SegShape sg = tab.shape(seg);
      const int64_t row0 = tab.out_off(seg) + first;
      const int cnt = min(tab.out_off(seg + 1) - tab.out_off(seg) - first, 1 << kFinishRowsLog2), at = first + (sg.kk < 0 ? 0 : sg.n - w);
      if (first == 0 && threadIdx.x == 0 && fin.out_offsets) {
        fin.out_offsets[seg] = tab.out_off(seg);
        if (seg == tab.nseg - 1) fin.out_offsets[seg + 1] = tab.out_off(tab.nseg);
      }
      for (int i = threadIdx.x; i < cnt; i += nthr) fin.kept_idx[row0 + i] = at + i;
      if (cnt > 0) copy_rows(fin.ga, sg, row0, cnt, nthr, [&](int i) { return at + i; });
      return;
    }
    more -= __builtin_amdgcn_readlane(incl, 63);
  }
}

// Pooling, top-k and copy (as select_resident_kernel, with the same keys and order) of a segment of at most kFinishMost positions by a workgroup that has
// scored some of them; in `smem`, LDS that nobody reads any more.  The phases take a few us whatever they are spread over, so every workgroup of
// the segment goes through them all and copies a slice of the rows; rows of one segment travel while another is still scored or selected.
//   It takes the place of a selection with one workgroup per CU and of a gather, where both would be launched.  Three launches / one, us a call, 16-bit keys:
// a decode cache of 256 segments, 107 to 1834 kept, 56.6 / 51.1; of 128 40.4 / 38.5; 192 segments, 500 kept on average, 512 new, averages 79.2 / 65.0; 384 heads of
// 300 55.7 / 45.0; 24 prompts of 500 to 1000 48.4 / 39.5; at worst 256 segments of 300 kept each, 128 rows 35.6 / 36.1.
//   Bound by the chain of its phases, and 256 threads go through it more slowly than the 1024 of the selection kernel, so not where no gather follows: scoring and
// selection / one launch: 8 x 2 K 18.2 / 21.1, one sequence's cache 18.6 / 21.6, 16 prompts of 1 to 1.7 K 40.3 / 49.3; nor up to 64 segments (64 x 1000 kept 35.8 / 35.7);
// nor fp32 and E4M3 keys, whose kernel keeps one workgroup on a CU (E4M3 cache of 256 segments 74.1 / 74.2; fp32 4 x 1 K 19.3 / 22.6).
constexpr int kFinishMost = 2048;
constexpr int kFinishRank = 256;          // keys of a digit that are ranked by counting
constexpr int kFinishStage = (kFinishMost + 2 * kSelHaloMax) / 4 * 5 + 16;   // padded for 4 positions a thread; then a list, then the kept positions
constexpr int kFinishWords = kFinishStage + kHistBins + 48;
template <int NT, class TAB>
__device__ __forceinline__ void finish_segment(uint32_t* smem, const TAB& tab, const FinishArgs& fin, int seg, int w, const float* imp, meet_t* word,
                                               int nchunks) {
  constexpr int EPT = kFinishMost / NT;
  static_assert(EPT >= 4 && EPT <= 32 && kFinishRank <= NT, "padding of the stage; a thread per listed key");
  float* const stage = reinterpret_cast<float*>(smem);
  int32_t* const at = reinterpret_cast<int32_t*>(smem);
  uint32_t* const hist = smem + kFinishStage;
  uint32_t* const sh_scan = hist + kHistBins;                  // 16
  uint32_t* const sh_mm = sh_scan + 16;                        // 2 * NT / 64
  uint32_t* const res = sh_mm + 16;                            // [0], [1]: digit search and ranking; [2]: length of the list; [3]: slice
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  auto pad = [](int i) { return i + i / EPT; };
  const SegShape sg = tab.shape(seg);
  const int m = sg.n - w, kk = sg.kk, radius = fin.pool_kernel / 2;
  const int out0 = tab.out_off(seg), kept = tab.out_off(seg + 1) - out0, per = (kept + nchunks - 1) / nchunks;
  const float* const I = imp + sg.score_off;
  if (tid == 0) {
    res[2] = 0;
    res[3] = nchunks > 1 ? (uint32_t)meet_slice(word) : 0u;
  }
  auto score_at = [&](int j) __attribute__((always_inline)) {
    return __hip_atomic_load(I + min(max(j, 0), m - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  float ld[EPT + 1];
#pragma unroll
  for (int c = 0; c <= EPT; ++c) ld[c] = score_at((c < EPT ? c * NT + tid : kFinishMost + min(tid, 2 * radius)) - radius);
  for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
#pragma unroll
  for (int c = 0; c <= EPT; ++c) {
    const int i = c * NT + tid, j = i - radius;
    if (c < EPT || tid < 2 * radius) stage[pad(i)] = j >= 0 && j < m ? ld[c] : 0.f;
  }
  __syncthreads();
  // pooled scores of this thread's positions, in the order of select_resident_kernel (up to a radius of 3 maxima of the keys)
  const int j0 = EPT * tid;
  uint32_t key[EPT];
  {
    float a[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      a[e] = stage[pad(j0 + e)];
      key[e] = score_key(a[e]);
    }
    const bool is_max = fin.pool_mode != SLKV_POOL_AVG, by_key = is_max && radius <= 3;
    for (int t = 1; t <= 2 * radius; ++t) {
      float x[EPT];
#pragma unroll
      for (int e = 0; e < EPT; ++e) x[e] = stage[pad(j0 + e + t)];
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        if (by_key) key[e] = max(key[e], score_key(x[e]));
        else a[e] = is_max ? fmaxf(a[e], x[e]) : a[e] + x[e];
      }
    }
    const float inv_p = 1.f / (float)fin.pool_kernel;
    if (!by_key)
#pragma unroll
      for (int e = 0; e < EPT; ++e) key[e] = score_key(is_max ? a[e] : a[e] * inv_p);
  }
  uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    if (j0 + e < m) {
      kmin = min(kmin, key[e]);
      kmax = max(kmax, key[e]);
    } else {
      key[e] = kKeyNone;
    }
  }
  kmin = wave_reduce_to_last(kmin, [](uint32_t a, uint32_t b) { return min(a, b); });
  kmax = wave_reduce_to_last(kmax, [](uint32_t a, uint32_t b) { return max(a, b); });
  if (lane == 63) {
    sh_mm[wv] = kmin;
    sh_mm[NT / 64 + wv] = kmax;
  }
  __syncthreads();
  int slice = (int)res[3];
  uint32_t lo = sh_mm[0], hi = sh_mm[NT / 64], k = (uint32_t)kk;
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) {
    lo = min(lo, sh_mm[i]);
    hi = max(hi, sh_mm[NT / 64 + i]);
  }
  // the k-th largest key: 11 bits of the range at a time, until the digit's keys are few enough to be ranked by counting
  while (hi != lo) {
    const uint32_t span = hi - lo;
    const int nbits = 32 - __clz(span), shift = nbits > 11 ? nbits - 11 : 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const uint32_t dk = key[e] - lo;                         // (a key below lo wraps to a difference above any span)
      if (dk <= span) atomicAdd(&hist[dk >> shift], 1u);
    }
    __syncthreads();
    select_bin<NT>(hist, k, sh_scan, res);
    const uint32_t d = res[0], cnt = hist[d];
    k = res[1];
    lo += d << shift;
    hi = min(hi, lo + ((1u << shift) - 1u));
    if (shift == 0) break;
    if (cnt <= (uint32_t)kFinishRank) {
      uint32_t* const list = smem;                             // (the scores are in registers)
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if (key[e] - lo <= hi - lo) list[atomicAdd(&res[2], 1u)] = key[e];
      __syncthreads();
      if ((uint32_t)tid < cnt) {
        const uint32_t kv = list[tid];
        uint32_t gt = 0, ge = 0;
        for (uint32_t i = 0; i < cnt; i += 4) {
#pragma unroll
          for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t o = list[i + u];
            const bool live = i + u < cnt;
            gt += live && o > kv ? 1u : 0u;
            ge += live && o >= kv ? 1u : 0u;
          }
        }
        if (gt < k && k <= ge) {                               // (every thread that holds the k-th largest value writes the same pair)
          res[0] = kv;
          res[1] = k - gt;
        }
      }
      __syncthreads();
      lo = res[0];
      k = res[1];
      break;
    }
    __syncthreads();                                           // every thread has read the digit's count
    for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
    __syncthreads();
  }
  const uint32_t tau = lo, need_eq = k;
  // ordered compaction: slot = (#greater before) + min(#equal before, need_eq)
  uint32_t gmask = 0, emask = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    gmask |= key[e] > tau && key[e] != kKeyNone ? 1u << e : 0u;
    emask |= key[e] == tau ? 1u << e : 0u;
  }
  const uint32_t ce = __popc(emask), packed = ce << 16 | __popc(gmask);
  const uint32_t excl = block_incl_scan<NT, false>(packed, sh_scan) - packed, e_before = excl >> 16;   // (its barrier: the list has been read)
  // (taken as the smaller first: of `e < need ? min(need - e, n) : 0` beside min(e, need) this compiler drops the comparison and the minimum)
  const uint32_t equal0 = min(e_before, need_eq);
  uint32_t kept_here = gmask, em = emask;
  for (uint32_t take = min(need_eq - equal0, ce); take > 0; --take) {
    kept_here |= em & (0u - em);
    em &= em - 1u;
  }
  const int slot0 = (int)((excl & 0xffffu) + equal0);
  while (slice < nchunks) {
    const int first = slice * per, rows = max(min(kept - first, per), 0);
    int slot = slot0 - first;
    for (uint32_t sel = kept_here; sel; sel &= sel - 1u, ++slot)
      if ((uint32_t)slot < (uint32_t)rows) at[slot] = j0 + __ffs(sel) - 1;
    if (slice == 0) {
      if (tid == 0 && fin.out_offsets) {
        fin.out_offsets[seg] = out0;
        if (seg == tab.nseg - 1) fin.out_offsets[seg + 1] = tab.out_off(tab.nseg);
      }
      if (fin.write_pooled) {
#pragma unroll
        for (int e = 0; e < EPT; ++e)
          if (j0 + e < m) fin.pooled[sg.score_off + j0 + e] = __uint_as_float(key[e]);
      }
    }
    int next = nchunks;
    if (tid == 0 && nchunks > 1) next = meet_slice(word);      // (on its way while the rows are copied)
    __syncthreads();
    auto pos = [&](int i) __attribute__((always_inline)) { return first + i < kk ? min(max(at[i], 0), m - 1) : m + first + i - kk; };   // (clamped as in gather_kernel)
    for (int i = tid; i < rows; i += NT) fin.kept_idx[out0 + first + i] = pos(i);
    if (rows > 0) copy_rows(fin.ga, sg, (int64_t)out0 + first, rows, NT, pos);
    if (nchunks == 1) break;
    if (tid == 0) res[3] = (uint32_t)next;
    __syncthreads();                                           // (and the positions have been read)
    slice = (int)res[3];
  }
  if (nchunks > 1 && tid == 0) meet_leave(word, nchunks);
}

// ------------------------------------------------------------------------------------------
// MFMA scoring of 16-bit inputs (bfloat16 or half).  One workgroup (4 waves) owns one chunk of history keys of one segment.
// K is staged in LDS in tiles of 64 keys (two buffers); up to kPrefetch further tiles are in
// flight from HBM into registers.  Wave (rb, ks) holds rows [rb*32*MT, (rb+1)*32*MT) of the
// G*w query rows in registers for the whole chunk and works on the 32-key sub-tiles
// ks, ks+KS, .. of every tile.  The 32x32x16 MFMA takes, per lane, 8 consecutive k-elements of
// row (lane%32) at k offset 8*(lane/32) for both operands, and returns in result register i the
// element at row 8*(i/4) + 4*(lane/32) + i%4, column lane%32.
//   PASS 1: D[key][qrow]: a lane owns one query row per MFMA tile -> sum of exp2(x - reference).
//   PASS 2: D[qrow][key]: a lane owns one key column -> sum over rows of exp2(x - lse[row]).
//   PASS 3: both, in one launch: the workgroups of a segment meet in between (meet_chunks).
//   PASS 4: as 3, and they select and copy as well (finish_segment).
// Rows beyond R and keys beyond the chunk are loaded from a clamped (valid) address and masked.
constexpr int kTileKeys = 64;
constexpr int kPrefetch = 2;

template <int DK, int MT, int RB, int PASS, int KIND, class TAB>   // KIND: 0 bf16, 1 fp16
__global__ __launch_bounds__(256, (MT <= 2 ? 2 : 1)) void score_q_resident_kernel(const TAB tab, const uint16_t* __restrict__ q,
                                                         const void* __restrict__ kmat_v, int64_t k_stride_tok,
                                                         int64_t k_stride_head, int R, int Rpad, int w, int CH,
                                                         float c_log2, float* __restrict__ part,
                                                         float* __restrict__ imp, int grid2d, uint32_t* __restrict__ gm,
                                                         meet_t* __restrict__ meet, int limit, const FinishArgs fin) {
  constexpr bool STATS = PASS != 2, BOTH = PASS >= 3, FINISH = PASS == 4;
  constexpr int KS = 4 / RB;               // waves along the keys
  constexpr int TK = kTileKeys;
  constexpr int NSUB = TK / 32 / KS;       // 32-key sub-tiles per wave per tile
  constexpr int KK = DK / 16;
  constexpr int ROWB = DK * 2 + 16;        // padded LDS row (bf16 / fp16 elements): conflict-free 16-byte reads down a column
  constexpr int CPR = DK * 2 / 16;          // 16-byte pieces per key row in memory
  constexpr int LPT = TK * CPR / 256;      // pieces per thread per tile
  constexpr int NPF = kPrefetch;
  static_assert(TK * CPR % 256 == 0 && LPT < 16, "tile must divide over the workgroup; LPT is or-ed into a wait count");
  constexpr int KTILES = 2 * TK * ROWB, FINW = FINISH ? kFinishWords * 4 : 0;
  __shared__ __attribute__((aligned(16))) unsigned char ktile_s[KTILES > FINW ? KTILES : FINW];   // (PASS 4: the selection's as well)
  unsigned char (*const ktile)[TK * ROWB] = reinterpret_cast<unsigned char (*)[TK * ROWB]>(ktile_s);
  __shared__ float red[2][RB][TK];
  __shared__ float2 comb[KS][RB * 32 * MT];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int rb = wv % RB, ks = wv / RB;
  const int l32 = lane & 31, half = lane >> 5;

  // Which chunk of which segment.  With a two-dimensional grid (grid2d; the host chooses it when the
  // segments' chunk counts are alike enough) blockIdx.y is the segment and blockIdx.x the chunk, and
  // workgroups past a segment's last chunk leave at once; otherwise blockIdx.x counts the chunks of
  // all segments and the segment is searched in the table.  The table is read through the scalar
  // cache, cold at every launch, so each dependent lookup costs a memory round trip before the
  // first key can be requested: the entries of segment blockIdx.y are therefore fetched before it
  // is known which case applies (y is 0 with a one-dimensional grid: a valid entry either way).
  struct SegEntry {
    int32_t n, tok_begin, head, qrow_off, score_off, chunk0, chunk1;
  };
  auto entry_of = [&](int s) {
    const SegShape sg = tab.shape(s);
    return SegEntry{sg.n, sg.tok_begin, sg.head, s * R, sg.score_off, tab.chunk_begin(s), tab.chunk_begin(s + 1)};
  };
  int seg = (int)blockIdx.y;
  SegEntry se = entry_of(seg);
  asm volatile("" :: "s"(se.n), "s"(se.tok_begin), "s"(se.head), "s"(se.qrow_off), "s"(se.chunk0), "s"(se.chunk1));   // fetched here, not behind the branch
  int bid;
  if (grid2d) {
    bid = se.chunk0 + (int)blockIdx.x;
    if (bid >= se.chunk1) return;
  } else {
    bid = blockIdx.x;
    if (FINISH && bid >= fin.chunks) {
      copy_unranked(tab, fin, w, bid - fin.chunks, 256);
      return;
    }
    seg = find_segment_wave(tab.nseg, bid, [&](int s) { return tab.chunk_begin(s); });
    se = entry_of(seg);
  }
  if (PASS == 1) SLKV_STAMP(256 + bid, 0);
  const int chunk = bid - se.chunk0;
  const int m = se.n - w;
  int key_begin, key_end, ntiles;
  auto set_chunk = [&](int c) __attribute__((always_inline)) {
    key_begin = c * CH;
    key_end = min(m, key_begin + CH);
    // tiles are processed in pairs (one per register slot); a surplus tile is fully masked
    ntiles = ((key_end - key_begin + TK - 1) / TK + 1) & ~1;
  };
  set_chunk(chunk);
  // uniform 64-bit base of the segment's keys + 32-bit byte offsets (the host checks the range)
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(kmat_v) +
      ((int64_t)se.head * k_stride_head + (int64_t)se.tok_begin * k_stride_tok) * 2;
  const uint32_t row_bytes = (uint32_t)k_stride_tok * 2u;
  const uint32_t piece_off = (uint32_t)(tid % CPR) * 16u;
  const int piece_row = tid / CPR;

  u32x4 pf0[LPT], pf1[LPT];
  auto issue_tile = [&](int t, u32x4 (&pf)[LPT]) __attribute__((always_inline)) {
    const int key0 = key_begin + t * TK + piece_row;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int key = min(key0 + i * (256 / CPR), key_end - 1);
      // non-temporal: a workgroup reads its keys once (plain loads measured the same in either pass)
      pf[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kbase + ((uint32_t)key * row_bytes + piece_off)));
    }
  };
  auto store_tile = [&](const u32x4 (&pf)[LPT], int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int idx = i * 256 + tid;
      *reinterpret_cast<u32x4*>(&ktile[buf][(idx / CPR) * ROWB + (idx % CPR) * 16]) = pf[i];
    }
  };
  static_assert(kPrefetch == 2, "the tile loops below are written out for two register slots");
  issue_tile(0, pf0);   // the second tile is requested after the queries: the loop can start without it

  // query rows of this wave, kept in registers for the whole chunk
  bf16x8 qreg[MT][KK];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row = min(rb * 32 * MT + mt * 32 + l32, R - 1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      Pack16 p;
      p.u = *reinterpret_cast<const u32x4*>(q + ((int64_t)se.qrow_off + row) * DK + kk * 16 + half * 8);
      qreg[mt][kk] = p.b;
    }
  }
  // pass 2: log-sum-exp of the rows from that of the segment's chunks (see fold_rows), handed to the lanes
  // through LDS once the other loads have landed
  constexpr int ROWS = RB * 32 * MT, NLSE = (ROWS + 255) / 256;
  float lse_ld[NLSE];
  float lse_r[MT][16];
  auto share_lse = [&]() __attribute__((always_inline)) {
    float* lse_s = reinterpret_cast<float*>(&comb[0][0]);
    static_assert(sizeof(comb) >= NLSE * 256 * sizeof(float), "comb holds one value per thread and load");
#pragma unroll
    for (int j = 0; j < NLSE; ++j) lse_s[tid + j * 256] = tid + j * 256 < R ? lse_ld[j] : INFINITY;
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        lse_r[mt][i] = lse_s[rb * 32 * MT + mt * 32 + 8 * (i >> 2) + 4 * half + (i & 3)];
  };
  if (PASS == 2) {
    float2* const fold = reinterpret_cast<float2*>(&ktile[0][0]);   // (no key has been stored yet)
#pragma unroll
    for (int j = 0; j < NLSE; ++j)
      lse_ld[j] = fold_rows(part, se.chunk0, se.chunk1, Rpad, j * 256, ROWS, 256, fold);
  }
  float m_run[MT], s_run[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    m_run[mt] = -INFINITY;
    s_run[mt] = 0.f;
  }

  // importance of a key (the lanes of a wave have neighbouring ones) and, if asked for, of its group
  auto put_sum = [&](int key, float v) __attribute__((always_inline)) {
    if (FINISH) {
      if (key < key_end) __hip_atomic_store(imp + se.score_off + key, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    if (key < key_end) imp[se.score_off + key] = v;
    if (gm) {
      const uint32_t top = max_8_lanes(key < key_end ? score_key(v) : 0u);
      if (key < key_end && tid % kGroup == 0) gm[group_off(se.score_off, seg) + key / kGroup] = top;
    }
  };
  // one tile: registers -> LDS, refill the register slot, barrier, MFMAs + epilogue
  auto do_tile = [&](auto pass_c, int t, u32x4 (&pf)[LPT], auto masked_c, auto online_c, auto first_c) __attribute__((always_inline)) {
    constexpr int PS = decltype(pass_c)::value;        // (1 or 2: of which pass)
    constexpr bool MASKED = decltype(masked_c)::value;   // the tile may reach past key_end
    constexpr bool ONLINE = decltype(online_c)::value;   // pass 1: running maximum instead of a fixed reference
    constexpr bool FIRST = decltype(first_c)::value;     // pass 1: the chunk's first tile (fixes the reference)
    const int buf = t & 1;
    tile_priority(t);
    store_tile(pf, buf);
    if (!ONLINE) issue_tile(t + NPF, pf);   // past the chunk end every piece comes from one clamped row
    __syncthreads();
    if (PS == 2 && t > 0 && tid < TK) {   // column sums of the previous tile
      float v = 0.f;
#pragma unroll
      for (int r = 0; r < RB; ++r) v += red[buf ^ 1][r][tid];
      put_sum(key_begin + (t - 1) * TK + tid, v);
    }
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) {
      __builtin_amdgcn_sched_barrier(0);   // keep one sub-tile's operands live at a time
      const int sub = ks + sb * KS;
      const int key0 = key_begin + t * TK + sub * 32;   // first key of this sub-tile
      bf16x8 kreg[KK];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        Pack16 p;
        p.u = *reinterpret_cast<const u32x4*>(&ktile[buf][(sub * 32 + l32) * ROWB + kk * 32 + half * 16]);
        kreg[kk] = p.b;
      }
      float colsum = 0.f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          if (PS == 1)
            acc = mfma16<KIND == 1>(kreg[kk], qreg[mt][kk], acc);
          else
            acc = mfma16<KIND == 1>(qreg[mt][kk], kreg[kk], acc);
        }
        if (PS == 1) {
          // lane: query row mt*32 + l32, keys key0 + 8*(i/4) + 4*half + i%4
          if (MASKED && key0 + 32 > key_end) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (key0 + 8 * (i >> 2) + 4 * half + (i & 3) >= key_end) acc[i] = -INFINITY;
          }
          if (ONLINE) {
            float mx = fmaxf(acc[0], acc[1]);
#pragma unroll
            for (int i = 2; i < 16; i += 2) mx = fmaxf(mx, fmaxf(acc[i], acc[i + 1]));
            const float mn = fmaxf(m_run[mt], mx * c_log2);
            const float mu = mn == -INFINITY ? 0.f : mn;
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += fast_exp2(fmaf(acc[i], c_log2, -mu));
            s_run[mt] = s_run[mt] * fast_exp2(m_run[mt] - mu) + sum;
            m_run[mt] = mn;
          } else {
            // The reference of the exponentials is fixed by the lane's first 16 logits of the chunk
            // (any finite reference gives the same log-sum-exp); later logits may exceed it by up to
            // ~2^100 before the sum overflows, which the caller detects and repeats ONLINE.
            if (FIRST && sb == 0) {
              float mx = fmaxf(acc[0], acc[1]);
#pragma unroll
              for (int i = 2; i < 16; i += 2) mx = fmaxf(mx, fmaxf(acc[i], acc[i + 1]));
              const float mn = mx * c_log2;
              m_run[mt] = mn == -INFINITY ? 0.f : mn;
            }
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += fast_exp2(fmaf(acc[i], c_log2, -m_run[mt]));
            s_run[mt] += sum;
          }
        } else {
          // lane: key key0 + l32, query rows mt*32 + 8*(i/4) + 4*half + i%4
#pragma unroll
          for (int i = 0; i < 16; ++i) colsum += fast_exp2(fmaf(acc[i], c_log2, -lse_r[mt][i]));
        }
      }
      if (PS == 2) {
        colsum += __shfl_xor(colsum, 32, 64);
        if (half == 0) red[buf][rb][sub * 32 + l32] = colsum;
      }
    }
  };

  // The first tile, Q and lse have to be complete here (loads return in order; the LPT loads of
  // the second tile, issued last, may still be in flight); inside the loop only the two tile slots
  // stay in flight, so the waits there can be partial.
  __builtin_amdgcn_sched_barrier(0);          // keep every earlier load ahead of the second tile's
  issue_tile(1, pf1);
  __builtin_amdgcn_s_waitcnt(0x0F70 | LPT);   // vmcnt(LPT)
  __builtin_amdgcn_sched_barrier(0);
  if (PASS == 2) share_lse();
  using T = std::true_type;
  using F = std::false_type;
  using P1 = std::integral_constant<int, 1>;
  using P2 = std::integral_constant<int, 2>;
  // Pass 1 with both sub-tiles of a tile in one wave (RB == 4; up to 64 rows per wave): software pipeline over sub-tiles.
  // The MFMAs of sub-tile s (two interleaved chains, one per row tile) are issued one per slot,
  // each slot also carrying the exponentials of two logits of sub-tile s-1 (read from the other
  // accumulator set), so the matrix pipe works in the shadow of the exponentials; the key operand
  // of the tile's second sub-tile is read from LDS during the first one's MFMAs.
  if constexpr (STATS && NSUB == 2 && MT <= 2) {
    constexpr int NSLOT = KK * MT, EPS = (16 * MT + NSLOT - 1) / NSLOT;
    f32x16 accA[MT], accB[MT];
    bf16x8 kA[KK], kB[KK];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) accA[mt][i] = accB[mt][i] = -INFINITY;   // exp2 of "the sub-tile before the first" is 0
    auto lds_read = [&](bf16x8& dst, int buf, int sub, int kk) __attribute__((always_inline)) {
      Pack16 pk;
      pk.u = *reinterpret_cast<const u32x4*>(&ktile[buf][(sub * 32 + l32) * ROWB + kk * 32 + half * 16]);
      dst = pk.b;
    };
    // keys past the chunk end count as -inf (pkey0 = first key of the accumulators' sub-tile)
    auto mask_tail = [&](f32x16 (&a)[MT], int pkey0) __attribute__((always_inline)) {
      if (pkey0 + 32 > key_end) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (pkey0 + 8 * (i >> 2) + 4 * half + (i & 3) >= key_end) a[mt][i] = -INFINITY;
      }
    };
    // one sub-tile: MFMAs into cur from operand kc, exponentials of prev; kn is filled for sub-tile nsub
    auto step = [&](f32x16 (&cur)[MT], f32x16 (&prev)[MT], bf16x8 (&kc)[KK], bf16x8 (&kn)[KK], auto prefetch_c, int buf,
                    int nsub) __attribute__((always_inline)) {
      constexpr bool PREFETCH = decltype(prefetch_c)::value;
#pragma unroll
      for (int sl = 0; sl < NSLOT; ++sl) {
        const int kk = sl / MT, mt = sl % MT;
#pragma unroll
        for (int j = 0; j < EPS; ++j) {
          const int e = sl * EPS + j;
          if (e < 16 * MT) s_run[e / 16] += fast_exp2(fmaf(prev[e / 16][e % 16], c_log2, -m_run[e / 16]));
        }
        if (kk == 0) {
          f32x16 z;
#pragma unroll
          for (int i = 0; i < 16; ++i) z[i] = 0.f;
          cur[mt] = mfma16<KIND == 1>(kc[kk], qreg[mt][kk], z);
        } else {
          cur[mt] = mfma16<KIND == 1>(kc[kk], qreg[mt][kk], cur[mt]);
        }
        if (PREFETCH && mt == MT - 1) lds_read(kn[kk], buf, nsub, kk);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto pipe_tile = [&](int t, u32x4 (&pf)[LPT], auto masked_c, auto first_c) __attribute__((always_inline)) {
      constexpr bool MASKED = decltype(masked_c)::value;   // this tile or the one before may reach past key_end
      constexpr bool FIRST = decltype(first_c)::value;
      const int buf = t & 1;
      const int key0 = key_begin + t * TK;
      tile_priority(t);
      store_tile(pf, buf);
      issue_tile(t + NPF, pf);
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) lds_read(kA[kk], buf, 0, kk);
      if (MASKED) mask_tail(accB, key0 - 32);            // second sub-tile of the tile before
      step(accA, accB, kA, kB, T{}, buf, 1);
      if (FIRST || MASKED) mask_tail(accA, key0);
      if (FIRST) {
        // The reference of the exponentials is fixed by the lane's first 16 logits of the chunk (any
        // finite reference gives the same log-sum-exp); later logits may exceed it by up to ~2^100
        // before the sum overflows, which is detected below and repeated with a running maximum.
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          float mx = fmaxf(accA[mt][0], accA[mt][1]);
#pragma unroll
          for (int i = 2; i < 16; i += 2) mx = fmaxf(mx, fmaxf(accA[mt][i], accA[mt][i + 1]));
          const float mn = mx * c_log2;
          m_run[mt] = mn == -INFINITY ? 0.f : mn;
        }
      }
      step(accB, accA, kB, kA, F{}, buf, 0);
    };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) m_run[mt] = 0.f;
    if (ntiles > NPF) {
      pipe_tile(0, pf0, F{}, T{});
      pipe_tile(1, pf1, F{}, F{});
      for (int t0 = NPF; t0 < ntiles - NPF; t0 += NPF) {
        pipe_tile(t0, pf0, F{}, F{});
        pipe_tile(t0 + 1, pf1, F{}, F{});
      }
      pipe_tile(ntiles - 2, pf0, T{}, F{});
      pipe_tile(ntiles - 1, pf1, T{}, F{});
    } else {
      pipe_tile(0, pf0, T{}, T{});
      pipe_tile(1, pf1, T{}, F{});
    }
    // the exponentials of the last sub-tile
    mask_tail(accB, key_begin + (ntiles - 1) * TK + 32);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) sum += fast_exp2(fmaf(accB[mt][i], c_log2, -m_run[mt]));
      s_run[mt] += sum;
    }
  } else if (STATS) {
    // the first tile fixes the reference of the exponentials; only the last pair can reach past the chunk end
    if (ntiles > NPF) {
      do_tile(P1{}, 0, pf0, F{}, F{}, T{});
      do_tile(P1{}, 1, pf1, F{}, F{}, F{});
      for (int t0 = NPF; t0 < ntiles - NPF; t0 += NPF) {
        do_tile(P1{}, t0, pf0, F{}, F{}, F{});
        do_tile(P1{}, t0 + 1, pf1, F{}, F{}, F{});
      }
      do_tile(P1{}, ntiles - 2, pf0, T{}, F{}, F{});
      do_tile(P1{}, ntiles - 1, pf1, T{}, F{}, F{});
    } else {
      do_tile(P1{}, 0, pf0, T{}, F{}, T{});
      do_tile(P1{}, 1, pf1, T{}, F{}, F{});
    }
  }
  // importance of the chunk's keys, whose first two tiles are on their way
  auto accumulate = [&]() __attribute__((always_inline)) {
    for (int t0 = 0; t0 < ntiles - NPF; t0 += NPF) {
      do_tile(P2{}, t0, pf0, F{}, F{}, F{});
      do_tile(P2{}, t0 + 1, pf1, F{}, F{}, F{});
    }
    do_tile(P2{}, ntiles - 2, pf0, T{}, F{}, F{});
    do_tile(P2{}, ntiles - 1, pf1, T{}, F{}, F{});
    __syncthreads();
    if (tid < TK) {
      const int t = ntiles - 1;
      float v = 0.f;
#pragma unroll
      for (int r = 0; r < RB; ++r) v += red[t & 1][r][tid];
      put_sum(key_begin + t * TK + tid, v);
    }
  };

  if (STATS) SLKV_STAMP(256 + bid, 1);
  if (PASS == 2) {
    accumulate();
    return;
  }
  // A sum that left the fp32 range (logits far above the chunk's first ones): the whole
  // workgroup repeats the chunk with the running maximum.  Not taken for ordinary inputs.
  bool bad = false;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) bad = bad || !(s_run[mt] < INFINITY);
  if (__syncthreads_or(bad ? 1 : 0)) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      m_run[mt] = -INFINITY;
      s_run[mt] = 0.f;
    }
    for (int t = 0; t < ntiles; ++t) {          // plain loop, one tile in flight: this path is rare
      issue_tile(t, pf0);
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
      do_tile(P1{}, t, pf0, T{}, T{}, F{});
    }
  }

#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    // (reference, sum) -> (log-sum-exp, 1): a sum referenced to early logits can be very large
    // or small, and merging such pairs directly could lose it to an underflowing factor
    m_run[mt] = s_run[mt] > 0.f ? m_run[mt] + __builtin_amdgcn_logf(s_run[mt]) : -INFINITY;
    s_run[mt] = 1.f;
    float m2 = __shfl_xor(m_run[mt], 32, 64);
    float s2 = __shfl_xor(s_run[mt], 32, 64);
    merge_stats(m_run[mt], s_run[mt], m2, s2);
    if (half == 0) comb[ks][rb * 32 * MT + mt * 32 + l32] = make_float2(m_run[mt], s_run[mt]);
  }
  __syncthreads();
  const int nchunks = se.chunk1 - se.chunk0;
#pragma unroll
  for (int j = 0; j < NLSE; ++j) {
    const int row = tid + j * 256;
    if (row < ROWS) {
      float mm = comb[0][row].x, ss = comb[0][row].y;
#pragma unroll
      for (int k2 = 1; k2 < KS; ++k2) merge_stats(mm, ss, comb[k2][row].x, comb[k2][row].y);
      // the chunk's log-sum-exp of the row (-inf: no key)
      const float l = ss > 0.f ? mm + __builtin_amdgcn_logf(ss) : -INFINITY;
      float* const p = part + ((int64_t)bid * Rpad + row);
      if (!BOTH) {
        if (row < Rpad) *p = l;
      } else if (nchunks == 1) {
        lse_ld[j] = l > -INFINITY ? l : INFINITY;
      } else if (row < Rpad) {
        __hip_atomic_store(p, l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  SLKV_STAMP(256 + bid, 2);
  if constexpr (BOTH) {
    // The second pass, its first keys on their way while the others' statistics are waited for.  As a rule over this
    // chunk alone; `left`, in thread 0: those whose workgroups have left.
    __shared__ int sh_next;
    meet_t* const word = meet + (int64_t)seg * kMeetWords;
    meet_t left = 0;
    bool met = false;
    int scored = 0;
    for (;;) {
      if (met || nchunks == 1) {
        issue_tile(0, pf0);
        issue_tile(1, pf1);
        __syncthreads();                                 // (every thread has read comb and sh_next)
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // the statistics are in memory
        __syncthreads();
        if (tid == 0) {
          left = meet_chunks(word, nchunks, chunk, limit);
          sh_next = left != kMeetLeft;
          if (FINISH && left == kMeetLeft) meet_leave(word, nchunks);
        }
        __syncthreads();
        if (!sh_next) return;
        issue_tile(0, pf0);                              // (before the wait they would delay what thread 0 reads)
        issue_tile(1, pf1);
        float2* const fold = reinterpret_cast<float2*>(&ktile[0][0]);
#pragma unroll
        for (int j = 0; j < NLSE; ++j)
          lse_ld[j] = fold_rows<true>(part, se.chunk0, se.chunk1, Rpad, j * 256, ROWS, 256, fold);
      }
      if (!met) share_lse();
      met = true;
      accumulate();
      ++scored;
      if (nchunks == 1) break;
      if (tid == 0) sh_next = meet_take(word, left);
      __syncthreads();
      if (sh_next < 0) break;
      set_chunk(sh_next);
    }
    if constexpr (FINISH) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the scores are in memory
      __syncthreads();
      if (nchunks > 1) {
        if (tid == 0) {
          const bool all = meet_scores(word, nchunks, scored, limit);
          if (!all) meet_leave(word, nchunks);
          sh_next = all;
        }
        __syncthreads();
        if (!sh_next) return;
      }
      finish_segment<256>(reinterpret_cast<uint32_t*>(ktile_s), tab, fin, seg, w, imp, word, nchunks);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Long histories of 16-bit keys: one pass over the keys instead of two, where no importance or pooled score is asked for
// (which calls: plan_q_resident).
//   score_sample_kernel     log-sum-exp of the rows over a sample of the keys: an estimate lse' of theirs
//   score_both_kernel       over all keys e = e^(x - lse'[row]), added up along the keys (the rows' log-sum-exp, exact) and down the
//                           rows (an approximate importance of every key)
//   approx_hist_kernel      histograms of the approximate importance; the range of rho
//   select_chosen_kernel    which keys can decide the selection; a probe, where that would be too many (first launch); their exact importance (second)
// and the selection as otherwise, from its exact values.
//
// The approximate importance of a key is I' = sum over the rows of e^(x - lse'[row]), the exact one
// I = sum of rho[row] * e^(x - lse'[row]) with rho = e^(lse' - lse), so rho_min I' <= I <= rho_max I', and the same
// holds for window maxima (averages: not built).  With tau' the k-th largest pooled I', known to a histogram bin [bin_lo, bin_hi),
// the k-th largest pooled I, tau, lies in [rho_min bin_lo, rho_max bin_hi].  Hence
//   a key with I' > bin_hi * rho_max / rho_min has I > tau: whatever its value, it only has to stay above tau;
//   a key with I' < bin_lo * rho_min / rho_max has I < tau: it may keep an I' below rho_min bin_lo, or stand at 0;
//   the keys between get their exact importance, computed as PASS 2 does.
// The selection on the array that holds these values keeps the same positions as on the exact importance.
//
// That asks for every rho near 1, and one row that gives half its weight to one key that the sample does not hold has rho = 0.5: the keys between are then
// up to all.  But such rows are few, or all alike, and I / I' is nearly the same for all keys.  So, where the range is wide, a probe comes first: the
// exact importance of the keys that are the largest by I', and with them, however they were chosen, a lower bound t of tau, the k-th largest score of the
// windows that they lie in.  Keys with I' < t / rho_max have I < tau; the others get their exact importance.  rho_max is kept near 1 by
// fold_sample.  Whatever the sample misses, the selection is exact; it only costs time, at worst that of all keys one by one.
//
// Of 131072 keys, 256 rows, 2 per cent of the keys pulled towards a query, 170 (3395) positions kept: 2300 (8400) keys are sampled, 40 to 70
// (1000) computed again.  With 1 row, or 16, that give half (0.9) of their weight to one key in the middle: 40 to 60 (800) in the probe and 30 to 60
// (1000 to 2100) behind it, where all of them were computed again without a probe.
// 32 segments of 20 K to 128 K keys, 256 rows, us: the two passes 160 + 176, their selection 52; sample 24, scan 184, histograms 13, bounds 7 (with a
// probe 20), chosen keys 20 (30), selection 22 (33).  The call, two passes / this: 407 / 278; one row at 0.9 404 / 307 (531 without the
// probe); 16 rows at 0.9 404 / 307 (528); 256 rows, a random share each 413 / 368; the queries 3 times as large 405 / 304 (481).  The worst found: the queries 5 times as
// large, where the sample says nothing, 404 / 498; a tenth of the positions kept and 256 rows with a random share each 470 / 570.
constexpr int kDenseKeys = 128;      // so many of a history's first and last keys are all in the sample (attention sinks, recent tokens);
// of those between, groups of neighbours (sample_step).
constexpr int kHists = 4, kHistPooled = 0, kHistKeys = 1;   // of I': pooled, and of a sample of the keys, not pooled;
constexpr int kHistProbe = 2, kHistExact = 3;               // of pooled exact scores: after a probe, and at the end
struct OneScan {
  float* part0;        // log-sum-exp of the sample in every range, [range][Rpad],
  float* dense;        // of all keys at either end, [segment][2][Rpad]
  uint32_t* hist;      // histograms, [segment][kHists][kHistBins]
  float* lse;          // log-sum-exp of the rows, [segment][2][256]: exact; of the sample
  uint32_t* bounds;    // [segment][kBoundWords]
  uint32_t* lists;     // [segment][kSelCandidates]
};

// 16 bytes per lane from base + off into LDS at lds (the same for the whole wave) + 16 * lane.  The caller waits for it (vmcnt);
// the compiler does not know of it.
__device__ __forceinline__ void load_to_lds16(const unsigned char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory", "m0");
}

// v of this lane and of the lane 32 away, added up, in both.
__device__ __forceinline__ float sum_halves(float v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Log-sum-exp of every query row over a sample of a range's keys: an online softmax, 8 waves of 32 rows (wave (rb, ks) takes
// the sub-tiles ks, ks + KS, .. of 32 keys of a tile).  Bound by round trips: a range has two to ten tiles.  (With the tile loop of
// score_q_resident_kernel, 4 waves of 64 rows at 256 registers, 41 us where this takes 25.)
template <int DK, int RB, int KIND>
__global__ __launch_bounds__(512, 4) void score_sample_kernel(const SegTable tab, const uint16_t* __restrict__ q, const void* __restrict__ kmat_v,
                                                              int64_t k_stride_tok, int64_t k_stride_head, int R, int Rpad, int w, int sampled_keys,
                                                              float c_log2, const OneScan one) {
  constexpr int NT = 512, KS = 8 / RB, TK = KS == 4 ? 128 : 64, NSUB = TK / 32 / KS, KK = DK / 16, ROWB = DK * 2 + 16, CPR = DK * 2 / 16;
  constexpr int LPT = TK * CPR / NT;
  __shared__ __attribute__((aligned(16))) unsigned char ktile[2][TK * ROWB];
  __shared__ float2 comb[2][KS][RB * 32];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int rb = wv % RB, ks = wv / RB, l32 = lane & 31, half = lane >> 5;
  const int bid = blockIdx.x;
  const int seg = find_segment_wave(tab.nseg, bid, [&](int s) { return tab.range_begin(s); });
  const SegShape sg = tab.shape(seg);
  const int m = sg.n - w, len = range_len(m, sg.kk, sampled_keys), r0 = tab.range_begin(seg), begin = (bid - r0) * len, keys = min(len, m - begin);
  // key u of the sample: the range's first `head` keys, its last `tail`, then, of those between, kSampleGroup neighbours every `stride` keys, which
  // stand for e^log_weight keys each
  int head = keys, tail = 0, stride = 1, total = keys;
  float log_weight = 0.f;
  if (keys > 2 * kDenseKeys) {
    head = bid == r0 ? kDenseKeys : 0;
    tail = begin + keys == m ? kDenseKeys : 0;
    const int between = keys - head - tail, groups = max(between / (kSampleGroup * sample_step(m, sg.kk)), 1);
    stride = between / groups;
    const int sampled = min(groups * kSampleGroup, between);
    total = head + tail + sampled;
    log_weight = sampled > 0 ? __builtin_amdgcn_logf((float)between / (float)sampled) : 0.f;
  }
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(kmat_v) +
      ((int64_t)sg.head * k_stride_head + (int64_t)(sg.tok_begin + begin) * k_stride_tok) * 2;
  const uint32_t row_bytes = (uint32_t)k_stride_tok * 2u, piece_off = (uint32_t)(tid % CPR) * 16u;
  u32x4 pf0[LPT], pf1[LPT];
  auto issue_tile = [&](int t, u32x4 (&pf)[LPT]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int u = min(t * TK + tid / CPR + i * (NT / CPR), total - 1);
      const int x = u - head - tail;
      const int key = u < head ? u : x < 0 ? x + keys : head + x / kSampleGroup * stride + x % kSampleGroup;
      pf[i] = *reinterpret_cast<const u32x4*>(kbase + ((uint32_t)key * row_bytes + piece_off));
    }
  };
  issue_tile(0, pf0);
  bf16x8 qreg[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    Pack16 p;
    p.u = *reinterpret_cast<const u32x4*>(q + ((int64_t)seg * R + min(rb * 32 + l32, R - 1)) * DK + kk * 16 + half * 8);
    qreg[kk] = p.b;
  }
  issue_tile(1, pf1);
  if (bid == r0)
    for (int i = tid; i < kHists * kHistBins; i += NT) one.hist[(size_t)seg * kHists * kHistBins + i] = 0;
  float m_run[2] = {-INFINITY, -INFINITY}, s_run[2] = {0.f, 0.f};   // the keys of head and tail; the others
  auto tile = [&](int t, u32x4 (&pf)[LPT], int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int idx = i * NT + tid;
      *reinterpret_cast<u32x4*>(&ktile[buf][(idx / CPR) * ROWB + (idx % CPR) * 16]) = pf[i];
    }
    issue_tile(t + 2, pf);
    __syncthreads();
#pragma unroll
    for (int sb = 0; sb < NSUB; ++sb) {
      const int sub = ks + sb * KS, u0 = t * TK + sub * 32;
      f32x16 acc;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        Pack16 p;
        p.u = *reinterpret_cast<const u32x4*>(&ktile[buf][(sub * 32 + l32) * ROWB + kk * 32 + half * 16]);
        acc = mfma16<KIND == 1>(p.b, qreg[kk], acc);
      }
      if (u0 + 32 > total) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (u0 + 8 * (i >> 2) + 4 * half + (i & 3) >= total) acc[i] = -INFINITY;
      }
      const bool sampled = u0 >= head + tail;            // (head and tail are multiples of 32 where other keys follow)
      const float lw = sampled ? log_weight : 0.f, m_old = sampled ? m_run[1] : m_run[0];
      float mx = acc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, acc[i]);
      const float mn = fmaxf(m_old, fmaf(mx, c_log2, lw));
      const float mu = mn == -INFINITY ? 0.f : mn;
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) sum += fast_exp2(fmaf(acc[i], c_log2, lw - mu));
      sum += (sampled ? s_run[1] : s_run[0]) * fast_exp2(m_old - mu);
      m_run[0] = sampled ? m_run[0] : mn;
      s_run[0] = sampled ? s_run[0] : sum;
      m_run[1] = sampled ? mn : m_run[1];
      s_run[1] = sampled ? sum : s_run[1];
    }
  };
  const int ntiles = (total + TK - 1) / TK;
  for (int t = 0; t < ntiles; t += 2) {
    tile(t, pf0, 0);
    if (t + 1 < ntiles) tile(t + 1, pf1, 1);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float m2 = __shfl_xor(m_run[i], 32, 64), s2 = __shfl_xor(s_run[i], 32, 64);
    merge_stats(m_run[i], s_run[i], m2, s2);
    if (half == 0) comb[i][ks][rb * 32 + l32] = make_float2(m_run[i], s_run[i]);
  }
  __syncthreads();
  const bool first = bid == r0, last = begin + keys == m;
  for (int i = tid; i < 2 * RB * 32; i += NT) {
    const int which = i / (RB * 32), row = i % (RB * 32);
    float mm = comb[which][0][row].x, ss = comb[which][0][row].y;
#pragma unroll
    for (int k2 = 1; k2 < KS; ++k2) merge_stats(mm, ss, comb[which][k2][row].x, comb[which][k2][row].y);
    const float l = ss > 0.f ? mm + __builtin_amdgcn_logf(ss) : -INFINITY;
    if (row >= Rpad) continue;
    float* const ends = one.dense + (int64_t)seg * 2 * Rpad + row;
    if (which == 1) one.part0[(int64_t)bid * Rpad + row] = l;
    else if (first) ends[0] = l;
    else if (last) ends[Rpad] = l;
    if (which == 0 && first && last) ends[Rpad] = -INFINITY;
  }
}

// One workgroup (4 waves) per chunk of keys, wave (rb, ks) with 32*MT query rows in registers, as in score_q_resident_kernel.
// D[row][key]: a lane owns one key and 16 rows per product, and adds every exponential to its row's running sum and to its key's.
//
// Bound by the matrix cores and the vector units, which do 32 cycles of MFMA and 44 of fma, exp2 and two adds per 32x32x16 product, and by the
// power both take (2.0 GHz under this load): the register-only loop takes 48 cycles a product, this one 72 of 2.5 M keys x 256 rows, 184 us = 0.9 PFLOP/s of products.
//  - The unit of the software pipeline is one 32x32 product of 8 chained MFMAs: among them go the exponentials of the unit before, so
//    two accumulators of 16 registers suffice, and the operand registers of the keys are refilled from LDS during their last use.  (16x16x32 MFMAs halve
//    the registers of lse' and sums, but overlap worse with the vector units: 15.6 against 11.2 ns for the same work in a register-only loop; 215 us.)
//  - Keys go from memory into LDS without passing registers, two tiles on their way: with them staged in registers
//    the loop spilled, and a reload waits for every load in flight (249 us).
//  - The tail mask is a second copy of the tile, not a branch between the units (20 us).
template <int DK, int MT, int RB, int KIND>
__global__ __launch_bounds__(256, 2) void score_both_kernel(const SegTable tab, const uint16_t* __restrict__ q, const void* __restrict__ kmat_v,
                                                            int64_t k_stride_tok, int64_t k_stride_head, int R, int Rpad, int w, int CH,
                                                            float c_log2, float* __restrict__ part, float* __restrict__ imp, int grid2d,
                                                            const OneScan one) {
  constexpr int KS = 4 / RB, TK = kTileKeys, NS = TK / 32 / KS, KK = DK / 16, ROWB = DK * 2, CPR = ROWB / 16;
  constexpr int LPT = TK * CPR / 256, RW = 32 * MT, ROWS = RB * RW;   // RW: rows of a wave
  constexpr int NB = 4;                                  // tiles in LDS: the one at work, the next, two on their way
  __shared__ __attribute__((aligned(16))) unsigned char ktile[NB][TK * ROWB];
  __shared__ float red[NB][RB][TK];
  __shared__ __attribute__((aligned(16))) float lse_s[256];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rb = wv % RB, ks = wv / RB, l32 = lane & 31, half = lane >> 5;

  struct SegEntry {
    int32_t n, tok_begin, head, score_off, chunk0, chunk1;
  };
  auto entry_of = [&](int s) {
    const SegShape sg = tab.shape(s);
    return SegEntry{sg.n, sg.tok_begin, sg.head, sg.score_off, tab.chunk_begin(s), tab.chunk_begin(s + 1)};
  };
  int seg = (int)blockIdx.y, bid;
  SegEntry se = entry_of(seg);
  if (grid2d) {
    bid = se.chunk0 + (int)blockIdx.x;
    if (bid >= se.chunk1) return;
  } else {
    bid = blockIdx.x;
    seg = find_segment_wave(tab.nseg, bid, [&](int s) { return tab.chunk_begin(s); });
    se = entry_of(seg);
  }
  const int key_begin = (bid - se.chunk0) * CH;
  const int key_end = min(se.n - w, key_begin + CH);
  const int ntiles = (key_end - key_begin + TK - 1) / TK;
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(kmat_v) +
      ((int64_t)se.head * k_stride_head + (int64_t)se.tok_begin * k_stride_tok) * 2;
  const uint32_t row_bytes = (uint32_t)k_stride_tok * 2u;
  // Keys go straight from memory into LDS, 1 KiB (64 / CPR rows) per wave and instruction, no registers in between.  The 16-byte pieces of a
  // row are permuted so that the lanes of an operand read, consecutive rows, meet different banks: piece p of row r lies in slot
  // p ^ swz(r).
  auto swz = [](int r) { return CPR == 16 ? r & 15 : (r >> 1) & 7; };
  const int ld_row = wv * (64 / CPR) + lane / CPR;       // + 256 / CPR for each further instruction, which swz does not see
  const uint32_t ld_piece = (uint32_t)((lane % CPR) ^ swz(ld_row)) * 16u;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)&ktile[0][0];
  const uint32_t ld_first = (uint32_t)(key_begin + ld_row) * row_bytes + ld_piece, ld_last = (uint32_t)(key_end - 1) * row_bytes + ld_piece;
  auto issue_tile = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i)                        // (past the end: the last key)
      load_to_lds16(kbase, min(ld_first + (uint32_t)(t * TK + i * (256 / CPR)) * row_bytes, ld_last),
                    lds_base + (uint32_t)((t % NB) * TK * ROWB + (i * 4 + wv) * 1024));
  };
  {
    const float l = fold_sample(one.part0, one.dense + (int64_t)seg * 2 * Rpad, tab.range_begin(seg), tab.range_begin(seg + 1), Rpad, ROWS);
    lse_s[tid] = tid < R ? l : INFINITY;
    if (bid == se.chunk0) one.lse[(size_t)seg * 512 + 256 + tid] = l;   // (for approx_hist_kernel)
  }
  __builtin_amdgcn_sched_barrier(0);                     // (the fold's loads and the queries together do not fit the registers)
  bf16x8 qreg[MT][KK];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row = min(rb * RW + mt * 32 + l32, R - 1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      Pack16 p;
      p.u = *reinterpret_cast<const u32x4*>(q + ((int64_t)seg * R + row) * DK + kk * 16 + half * 8);
      qreg[mt][kk] = p.b;
    }
  }
  __syncthreads();
  issue_tile(0);
  issue_tile(1);
  issue_tile(2);
  float lse_r[MT][16], row_sum[MT][16];
  f32x16 accA, accB;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    accA[i] = accB[i] = -INFINITY;                       // (exp2 of "the products before the first" is 0)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      lse_r[mt][i] = lse_s[rb * RW + mt * 32 + 8 * (i >> 2) + 4 * half + (i & 3)];
      row_sum[mt][i] = 0.f;
    }
  }
  bf16x8 kreg[KK];
  uint32_t rd[KK];                                       // where in LDS they come from (first sub-tile of a tile)
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) rd[kk] = (uint32_t)((ks * NS * 32 + l32) * ROWB + ((kk * 2 + half) ^ swz(l32)) * 16);
  auto lds_read = [&](int sub, int kk) __attribute__((always_inline)) {
    Pack16 pk;
    pk.u = *reinterpret_cast<const u32x4*>(&ktile[0][0] + (rd[kk] + (uint32_t)(sub * 32 * ROWB)));
    kreg[kk] = pk.b;
  };
  // exponential of product i of row tile mt
  auto one_exp = [&](const f32x16& a, int mt, int i, float& cs) __attribute__((always_inline)) {
    const float x = fast_exp2(fmaf(a[i], c_log2, -lse_r[mt][i]));
    row_sum[mt][i] += x;
    cs += x;
    asm volatile("" : "+v"(row_sum[mt][i]), "+v"(cs));   // here and not behind the next branch, where 16 exponentials would wait in registers
  };
  // The products of one row tile and 32 keys (kreg) into cur, a chain of MFMAs, and among them the exponentials of prev, the
  // products before them, of row tile PM.  RELOAD: the last use of these keys, the operands of the next (sub-tile nsub of the tile
  // that lies `ahead` bytes on) follow.
  auto unit = [&](f32x16& cur, const f32x16& prev, auto mt_c, auto pm_c, auto reload_c, int ahead, int nsub, float& cs) __attribute__((always_inline)) {
    constexpr int M = decltype(mt_c)::value, PM = decltype(pm_c)::value, EPS = 16 / KK;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk == 0) {
        f32x16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        cur = mfma16<KIND == 1>(qreg[M][kk], kreg[kk], z);
      } else {
        cur = mfma16<KIND == 1>(qreg[M][kk], kreg[kk], cur);
      }
      if (decltype(reload_c)::value) {
        if (nsub == 0) rd[kk] += (uint32_t)ahead;
        lds_read(nsub, kk);
      }
#pragma unroll
      for (int j = 0; j < EPS; ++j) one_exp(prev, PM, kk * EPS + j, cs);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto put = [&](float cs, int rbuf, int sub) __attribute__((always_inline)) {
    red[rbuf][rb][ks * NS * 32 + sub * 32 + l32] = sum_halves(cs);   // (both halves write the same value)
  };
  // the sums of tile t's keys over the RB row blocks: a wave looks after 16 keys, RB neighbouring lanes after one
  static_assert(16 * RB <= 64, "RB lanes per key");
  auto read_sums = [&](int rbuf) __attribute__((always_inline)) { return red[rbuf][lane % RB][(wv * 16 + lane / RB) % TK]; };
  auto store_sums = [&](float v, int t) __attribute__((always_inline)) {
    v += dpp_move_f<0xb1>(v);                            // quad_perm: the neighbour
    if (RB == 4) v += dpp_move_f<0x4e>(v);               // and the pair next to them
    const int key = wv * 16 + lane / RB;
    if (lane < 16 * RB && lane % RB == 0 && key < key_end - key_begin - t * TK) (imp + se.score_off + key_begin + t * TK)[(uint32_t)key] = v;
  };
  auto mask_keys = [&](f32x16& a, int t, int sub) __attribute__((always_inline)) {
    if (key_begin + t * TK + (ks * NS + sub) * 32 + l32 >= key_end) {
#pragma unroll
      for (int i = 0; i < 16; ++i) a[i] = -INFINITY;
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  float cs = 0.f;                                        // of the keys whose products are in the accumulators
  __builtin_amdgcn_s_waitcnt(0x0F70 | LPT);
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) lds_read(0, kk);
  // tile t, in LDS since the barrier like tile t + 1; MASKED: it may reach past key_end
  auto tile = [&](int t, auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int buf = t % NB, before = (t + NB - 1) % NB;
    const int ahead = buf == NB - 1 ? -(NB - 1) * TK * ROWB : TK * ROWB;
    tile_priority(t);
    issue_tile(t + 3);                                   // into the buffer of tile t - 1, which every wave has read; past the end: the last key again
    const float sums = read_sums((t + NB - 2) % NB);     // (complete since the barrier)
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int nsub = s + 1 < NS ? s + 1 : 0;
      unit(accA, accB, I0{}, std::integral_constant<int, MT - 1>{}, std::integral_constant<bool, MT == 1>{}, ahead, nsub, cs);
      if (MASKED) mask_keys(accA, t, s);
      put(cs, s > 0 ? buf : before, s > 0 ? s - 1 : NS - 1);
      cs = 0.f;
      if constexpr (MT == 2) {
        unit(accB, accA, I1{}, I0{}, std::true_type{}, ahead, nsub, cs);
        if (MASKED) mask_keys(accB, t, s);
      } else {
        accB = accA;
      }
    }
    if (t > 1) store_sums(sums, t - 2);
    __builtin_amdgcn_s_waitcnt(0x0F70 | LPT);            // vmcnt: all but the tile issued above
    __syncthreads();
  };
#pragma unroll 1
  for (int t = 0; t < ntiles - 1; ++t) tile(t, std::false_type{});
  tile(ntiles - 1, std::true_type{});
  {
    const int last = (ntiles - 1) % NB;
#pragma unroll
    for (int i = 0; i < 16; ++i) one_exp(accB, MT - 1, i, cs);
    put(cs, last, NS - 1);
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // nothing is on its way into LDS any more
    __syncthreads();
    if (ntiles > 1) store_sums(read_sums((last + NB - 1) % NB), ntiles - 2);
    store_sums(read_sums(last), ntiles - 1);
  }
  // the rows' sums over the 32 lanes that hold a row's keys, by row moves, into the last of them
  bool bad = false;
  float* const sums = reinterpret_cast<float*>(&ktile[0][0]);   // [KS][ROWS] (every wave is past its last read)
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float v = row_sum[mt][i];
      v += dpp_move_f<kDppRowShr + 1>(v);
      v += dpp_move_f<kDppRowShr + 2>(v);
      v += dpp_move_f<kDppRowShr + 4>(v);
      v += dpp_move_f<kDppRowShr + 8>(v);
      v += dpp_move_f<kDppRowBcast15, 0xa>(v);
      // (a row beyond R has lse' = inf and the sum 0; lse' = inf below R: no estimate, a sample of NaNs)
      const int row = rb * RW + mt * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
      bad = bad || (l32 == 31 && (!(v < INFINITY) || (row < R && lse_r[mt][i] == INFINITY)));
      if (l32 == 31) sums[ks * ROWS + row] = v;
    }
  if (__syncthreads_or(bad ? 1 : 0)) {
    // A sum that left the fp32 range (logits far above the sample's) or is none: the chunk once more, with a running maximum, a tile at a time.
    // Not taken for ordinary inputs.
    int ln = l32;
    asm volatile("" : "+v"(ln));                         // (no address of here is computed, and kept, before the loop above)
    float m_run[MT], s_run[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      m_run[mt] = -INFINITY;
      s_run[mt] = 0.f;
    }
    for (int t = 0; t < ntiles; ++t) {
      __syncthreads();
      for (int i = tid; i < TK * CPR; i += 256) {
        const int r = i / CPR, key = min(key_begin + t * TK + r, key_end - 1);
        *reinterpret_cast<u32x4*>(&ktile[0][r * ROWB + ((i % CPR) ^ swz(r)) * 16]) =
            *reinterpret_cast<const u32x4*>(kbase + ((uint32_t)key * row_bytes + (uint32_t)(i % CPR) * 16u));
      }
      __syncthreads();
      for (int s = 0; s < NS; ++s) {
        const int r0 = (ks * NS + s) * 32, key0 = key_begin + t * TK + r0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          f32x16 a;
#pragma unroll
          for (int i = 0; i < 16; ++i) a[i] = 0.f;
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            Pack16 pk;
            pk.u = *reinterpret_cast<const u32x4*>(&ktile[0][(r0 + ln) * ROWB + ((kk * 2 + half) ^ swz(ln)) * 16]);
            a = mfma16<KIND == 1>(pk.b, qreg[mt][kk], a);
          }
          // lane: query row mt*32 + l32, keys key0 + 8*(i/4) + 4*half + i%4
          float mx = -INFINITY;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            if (key0 + 8 * (i >> 2) + 4 * half + (i & 3) >= key_end) a[i] = -INFINITY;
            mx = fmaxf(mx, a[i]);
          }
          const float mn = fmaxf(m_run[mt], mx * c_log2), mu = mn == -INFINITY ? 0.f : mn;
          float sum = 0.f;
#pragma unroll
          for (int i = 0; i < 16; ++i) sum += fast_exp2(fmaf(a[i], c_log2, -mu));
          s_run[mt] = s_run[mt] * fast_exp2(m_run[mt] - mu) + sum;
          m_run[mt] = mn;
        }
      }
    }
    float2* const comb = reinterpret_cast<float2*>(&ktile[1][0]);   // [KS][ROWS]
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float m2 = __shfl_xor(m_run[mt], 32, 64), s2 = __shfl_xor(s_run[mt], 32, 64);
      merge_stats(m_run[mt], s_run[mt], m2, s2);
      if (half == 0) comb[ks * ROWS + rb * RW + mt * 32 + l32] = make_float2(m_run[mt], s_run[mt]);
    }
    __syncthreads();
    for (int row = tid; row < ROWS; row += 256) {
      float mm = comb[row].x, ss = comb[row].y;
#pragma unroll
      for (int k2 = 1; k2 < KS; ++k2) merge_stats(mm, ss, comb[k2 * ROWS + row].x, comb[k2 * ROWS + row].y);
      if (row < Rpad) part[(int64_t)bid * Rpad + row] = ss > 0.f ? mm + __builtin_amdgcn_logf(ss) : -INFINITY;
    }
    return;
  }
  for (int row = tid; row < ROWS; row += 256) {
    float v = sums[row];
#pragma unroll
    for (int k2 = 1; k2 < KS; ++k2) v += sums[k2 * ROWS + row];
    if (row < Rpad) part[(int64_t)bid * Rpad + row] = v > 0.f ? lse_s[row] + __builtin_amdgcn_logf(v) : -INFINITY;
  }
}

constexpr int kBinShift = 17;                        // 64 bins per octave,
constexpr uint32_t kBinBase = 106u << (23 - kBinShift);   // from 2^-21 to 2^11; what lies outside counts in the first and last bin
constexpr int kSelCandidates = 12288;                // scores that select_rank_kernel's list in LDS can hold
constexpr float kAboveAll = 0x1p120f;                // stands for the importance of a key above tau
constexpr float kProbeGain = 0.05f;                  // a probe has to save this share of a history's keys: it takes 10 us more than the bounds alone, all keys 220 us
constexpr float kSlack = 1.f / 1024.f;               // of the bounds: far above the rounding of either side

__device__ __forceinline__ uint32_t score_bin(uint32_t u) {
  const uint32_t b = u >> kBinShift;
  return b <= kBinBase ? 0u : min(b - kBinBase, (uint32_t)kHistBins - 1u);
}

// Histogram of the pooled approximate importance, and of that of every eighth run of 256 keys itself: a workgroup per block of 4096 positions
// (x - 1) of a segment (y).  A block's two counts of a bin share a word.  Workgroup x == 0: the segment's rows, their log-sum-exp and the range of rho.
constexpr int kApproxBlock = 4096;
__global__ __launch_bounds__(256) void approx_hist_kernel(const SegTable tab, int w, int radius, int R, int Rpad, const float* __restrict__ part,
                                                          const float* __restrict__ imp, const OneScan one) {
  __shared__ uint32_t bins[kHistBins];
  __shared__ uint32_t stage[kApproxBlock + kMaxPool];
  const int tid = threadIdx.x, seg = blockIdx.y;
  const SegShape sg = tab.shape(seg);
  const int m = sg.n - w, p0 = ((int)blockIdx.x - 1) * kApproxBlock;
  if (!(sg.kk > 0 && sg.kk < m) || p0 >= m) return;
  if (p0 < 0) {
    const int lane = tid & 63, wv = tid >> 6;
    const float lse0 = one.lse[(size_t)seg * 512 + 256 + tid];
    const int rows = Rpad <= 64 ? 64 : Rpad <= 128 ? 128 : 256;
    const float lse = fold_rows(part, tab.chunk_begin(seg), tab.chunk_begin(seg + 1), Rpad, 0, rows, 256, reinterpret_cast<float2*>(stage));
    one.lse[(size_t)seg * 512 + tid] = tid < R ? lse : INFINITY;
    // anything that is not a positive number ends as 0 or inf
    const float rho = fast_exp2(lse0 - lse);
    float rmin = tid < R ? (rho > 0.f ? rho : 0.f) : INFINITY, rmax = tid < R ? (rho < INFINITY ? rho : INFINITY) : 0.f;
    float rsum = rmax;
#pragma unroll
    for (int dlt = 32; dlt > 0; dlt >>= 1) {
      rmin = fminf(rmin, __shfl_xor(rmin, dlt, 64));
      rmax = fmaxf(rmax, __shfl_xor(rmax, dlt, 64));
      rsum += __shfl_xor(rsum, dlt, 64);
    }
    float* const sh = reinterpret_cast<float*>(bins);
    if (lane == 0) {
      sh[wv] = rmin;
      sh[4 + wv] = rmax;
      sh[8 + wv] = rsum;
    }
    __syncthreads();
    if (tid == 0) {
      float* const out = reinterpret_cast<float*>(one.bounds + seg * kBoundWords + kBoundRho);
      out[0] = fminf(fminf(sh[0], sh[1]), fminf(sh[2], sh[3]));
      out[1] = fmaxf(fmaxf(sh[4], sh[5]), fmaxf(sh[6], sh[7]));
      out[2] = (sh[8] + sh[9] + sh[10] + sh[11]) / (float)R;
    }
    return;
  }
  const float* I = imp + sg.score_off;
  const int cnt = min(kApproxBlock, m - p0);
  constexpr int PER = kApproxBlock / 256;
  float v[PER + 1];
#pragma unroll
  for (int e = 0; e <= PER; ++e) {
    const int j = p0 - radius + e * 256 + tid;
    v[e] = I[min(max(j, 0), m - 1)];                 // (positions beyond either end: a neighbour inside the window or none)
  }
  for (int i = tid; i < kHistBins; i += 256) bins[i] = 0;
#pragma unroll
  for (int e = 0; e <= PER; ++e)
    if (e * 256 + tid < kApproxBlock + 2 * radius) stage[e * 256 + tid] = score_key(v[e]);
  __syncthreads();
#pragma unroll 4
  for (int e = 0; e < PER; ++e) {
    const int s = e * 256 + tid;
    if (s < cnt) {
      uint32_t a = stage[s];
      for (int t = 1; t <= 2 * radius; ++t) a = max(a, stage[s + t]);
      atomicAdd(&bins[score_bin(a)], 1u);
      if (e % 8 == 0) atomicAdd(&bins[score_bin(stage[s + radius])], 1u << 16);
    }
  }
  __syncthreads();
  uint32_t* const H = one.hist + (size_t)seg * kHists * kHistBins;
  for (int i = tid; i < kHistBins; i += 256) {
    const uint32_t c = bins[i];
    if (c & 0xffffu) atomicAdd(&H[kHistPooled * kHistBins + i], c & 0xffffu);
    if (c >> 16) atomicAdd(&H[kHistKeys * kHistBins + i], c >> 16);
  }
}

// What follows from the histograms and the range of rho, as every workgroup of a segment finds it (NT threads; ends with a barrier):
//   word[0], [1]: keys whose I' lies between (bit patterns, inclusive) need their exact importance; above: kAboveAll stands for it;
//   word[2], [3]: the k-th largest pooled score lies between;
//   probe: the range of rho is too wide to tell much, a probe comes first.  word[0]: it computes the keys from here on;
//   wide: the pooled scores between word[2] and [3] may be more than a list holds.
struct OneScanBounds {
  uint32_t word[4];
  bool probe, wide;
};
template <int NT>
__device__ __forceinline__ OneScanBounds one_scan_bounds(const uint32_t* __restrict__ H, const float* __restrict__ rho, int m, int kk,
                                                         uint32_t* bins, uint32_t* sh_scan, uint32_t* res, uint32_t (*sh_count)[NT / 64]) {
  constexpr int PER = kHistBins / NT;
  const int tid = threadIdx.x;
  uint32_t keys_in[PER];                                 // sampled keys of the bins
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    bins[i * NT + tid] = H[kHistPooled * kHistBins + i * NT + tid];
    keys_in[i] = H[kHistKeys * kHistBins + i * NT + tid];
  }
  const float rmin = rho[0], rmax = rho[1], rmean = rho[2];
  __syncthreads();
  select_bin<NT>(bins, (uint32_t)kk, sh_scan, res);
  const uint32_t b = res[0];
  const float ratio = rmax / rmin;
  const bool usable = b > 0u && rmin > 0.f && ratio < 1e6f;     // (false for NaN, too)
  const float bin_lo = __uint_as_float((b + kBinBase) << kBinShift);
  const float bin_hi = b == (uint32_t)kHistBins - 1u ? INFINITY : __uint_as_float((b + 1u + kBinBase) << kBinShift);
  OneScanBounds r{{0u, 0x7f800000u, 0u, 0x7f800000u}, false, false};   // not usable: every key, any score
  uint32_t guess = 0;                                           // about where the keys begin that follow a probe: I = rmean I' for most keys
  if (usable) {
    r.word[0] = __float_as_uint(bin_lo * (rmin / rmax) * (1.f - kSlack));
    r.word[1] = min(__float_as_uint(bin_hi * ratio * (1.f + kSlack)), 0x7f800000u);
    r.word[2] = __float_as_uint(bin_lo * rmin * (1.f - kSlack));
    r.word[3] = min(__float_as_uint(bin_hi * rmax * (1.f + kSlack)), 0x7f800000u);
    guess = __float_as_uint(bin_lo * (0.9f * rmean / rmax));
  }
  // positions whose pooled score probably lies between word[2] and [3], and sampled keys: between word[0] and [1], from the guess on, all
  uint32_t count[4] = {0, 0, 0, 0};
  const uint32_t lo_bin = score_bin(r.word[0]), hi_bin = score_bin(r.word[1]), guess_bin = score_bin(guess);
  const uint32_t lo2_bin = usable ? score_bin(__float_as_uint(__uint_as_float(r.word[2]) / rmean * 0.95f)) : 0u;
  const uint32_t hi2_bin = usable ? score_bin(__float_as_uint(__uint_as_float(r.word[3]) / rmean * 1.05f)) : (uint32_t)kHistBins - 1u;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const uint32_t at = (uint32_t)(i * NT + tid);
    if (at >= lo2_bin && at <= hi2_bin) count[0] += bins[at];
    if (at >= lo_bin && at <= hi_bin) count[1] += keys_in[i];
    if (at >= guess_bin) count[2] += keys_in[i];
    count[3] += keys_in[i];
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    count[c] = wave_sum(count[c]);
    if ((tid & 63) == 0) sh_count[c][tid >> 6] = count[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    count[c] = 0;
#pragma unroll
    for (int v = 0; v < NT / 64; ++v) count[c] += sh_count[c][v];
  }
  r.probe = usable && (float)count[2] + kProbeGain * (float)count[3] < (float)count[1];
  r.wide = r.probe || count[0] > (uint32_t)kSelCandidates;
  if (r.probe) {
    // The keys that put half as many positions again as are wanted into this bin or above: the exact order differs, and from no more than
    // kk positions their kk-th largest score would be a poor bound.
    select_bin<NT>(bins, (uint32_t)min(kk + kk / 2, m), sh_scan, res);
    r.word[0] = (max(res[0], 1u) + kBinBase) << kBinShift;
  }
  __syncthreads();
  return r;
}

// The exact importance of the keys that can decide the selection.  A workgroup (8 waves) per range of positions lists them
// and takes them TK at a time through the loop of PASS 2; wave (rb, ks) holds 32 query rows.  Two launches:
//   probe: the bounds of the segment, which the second one finds in memory; where they ask for a probe, the exact pooled scores that it gives, in a histogram;
//   otherwise, blockhist == NULL: the importance array is made fit for select_resident_kernel;
//   or the positions are pooled here (the keys of the neighbours' edges are done twice) and their scores between word[2] and [3] listed, or (wide) all of
//   them counted in a histogram, so that the block-wise selection starts at phase 1 of select_rank_kernel.
template <int DK, int RB, int KIND>
__global__ __launch_bounds__(512, 4) void select_chosen_kernel(const SegTable tab, const uint16_t* __restrict__ q, const void* __restrict__ kmat_v,
                                                               int64_t k_stride_tok, int64_t k_stride_head, int R, int w, int sampled_keys, int radius,
                                                               float c_log2, const OneScan one, float* __restrict__ imp,
                                                               float* __restrict__ pooled, uint32_t* __restrict__ blockhist, int probe) {
  constexpr int NT = 512, KS = 8 / RB, TK = KS == 4 ? 128 : 64, NSUB = TK / 32 / KS, KK = DK / 16, ROWB = DK * 2 + 16, CPR = DK * 2 / 16;
  constexpr int LPT = TK * CPR / NT, MOST = kRangeMost + kMaxPool - 1, PER = (MOST + NT - 1) / NT;
  constexpr int NB = KS == 4 ? 1 : 2;                    // up to 64 rows: one tile in LDS, or a CU would hold one workgroup only (32 heads x 58 K keys of 16 rows, two launches: 26 us instead of 17)
  __shared__ __attribute__((aligned(16))) unsigned char ktile[NB][TK * ROWB];
  __shared__ float red[2][RB][TK];
  __shared__ uint32_t val[MOST];                         // pooled scores (dense: the keys' own); 0 where no key that matters is near
  __shared__ uint16_t list[MOST];
  __shared__ float lse_s[256];
  __shared__ uint32_t nlist, nsure, nabove, nband, band0;
  __shared__ uint32_t sh_scan[NT / 64], res[2], sh_count[4][NT / 64];
  uint32_t* const bins = reinterpret_cast<uint32_t*>(&ktile[0][0]);   // before and after the tiles
  static_assert(sizeof(ktile) >= kHistBins * sizeof(uint32_t), "the bins fit the tiles' place");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int rb = wv % RB, ks = wv / RB, l32 = lane & 31, half = lane >> 5;
  const int bid = (int)(gridDim.x - 1 - blockIdx.x);     // (the last segments' first: short ones have the most to do)
  const int seg = find_segment_wave(tab.nseg, bid, [&](int s) { return tab.range_begin(s); });
  const SegShape sg = tab.shape(seg);
  const int m = sg.n - w, len = range_len(m, sg.kk, sampled_keys), begin = (bid - tab.range_begin(seg)) * len;
  const bool pools = blockhist || probe;
  const int reach = pools ? radius : 0;
  uint32_t* const H = one.hist + (size_t)seg * kHists * kHistBins;
  uint32_t* const bd = one.bounds + seg * kBoundWords;
  const float* const rho = reinterpret_cast<const float*>(bd + kBoundRho);
  float* const I = imp + sg.score_off;
  const int first = begin, end = min(begin + len, m);
  const int p0 = max(first - reach, 0), cnt = min(end + reach, m) - p0;   // positions looked at here
  uint32_t lo, hi, lo2, hi2;
  bool probed, wide;
  if (probe) {
    const OneScanBounds b = one_scan_bounds<NT>(H, rho, m, sg.kk, bins, sh_scan, res, sh_count);
    if (begin == 0 && tid == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) bd[i] = b.word[i];
      bd[kBoundProbe] = b.probe ? 1u : 0u;
      bd[kBoundWide] = b.wide ? 1u : 0u;
      if (blockhist) {                                   // the words that select_rank_kernel, phase 1, expects
        uint32_t* const hdr = blockhist + (size_t)tab.blk_begin(seg) * kHistBins;
        hdr[4] = b.word[2];
        hdr[5] = b.word[3];
        hdr[6] = 0;                                      // pooled scores above the range
        hdr[7] = 0;                                      // scores listed (or counted, where they are more than a list holds)
      }
    }
    if (!b.probe) return;
    probed = true;
    wide = b.wide;
    lo = b.word[0];
    hi = hi2 = 0x7f800000u;
    lo2 = 0;
  } else {
    probed = bd[kBoundProbe] != 0u;
    wide = bd[kBoundWide] != 0u;
    lo = bd[0];
    hi = bd[1];
    lo2 = bd[2];
    hi2 = bd[3];
  }
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) v[e] = I[p0 + min(e * NT + tid, cnt - 1)];
  if (tid < 256) lse_s[tid] = one.lse[(size_t)seg * 512 + tid];
  if (tid == 0) nlist = nsure = nabove = nband = 0;
  if (pools)
    for (int i = tid; i < cnt; i += NT) val[i] = 0;
  // A key's score enters the windows that it lies in, or, where the list holds much of the range, its own place: the windows' maxima follow at the end
  // (lists of all keys, call of 2.5 M: windows of 7 the same, of 13 467 -> 440 us, of 63 620 -> 480).
  bool dense = false;
  auto pool = [&](int i, uint32_t u) __attribute__((always_inline)) {
    if (dense) val[i] = u;
    else for (int j = max(i - radius, 0); j <= min(i + radius, cnt - 1); ++j) atomicMax(&val[j], u);
  };
  bf16x8 qreg[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    Pack16 p;
    p.u = *reinterpret_cast<const u32x4*>(q + ((int64_t)seg * R + min(rb * 32 + l32, R - 1)) * DK + kk * 16 + half * 8);
    qreg[kk] = p.b;
  }
  if (probed && !probe) {
    // the probe's kk-th largest pooled score: what tau reaches at least
    for (int i = tid; i < kHistBins; i += NT) bins[i] = H[kHistProbe * kHistBins + i];
    __syncthreads();
    select_bin<NT>(bins, (uint32_t)sg.kk, sh_scan, res);
    lo2 = res[0] ? (res[0] + kBinBase) << kBinShift : 0u;
    lo = __float_as_uint(__uint_as_float(lo2) / rho[1] * (1.f - kSlack));
    hi = hi2 = 0x7f800000u;
  }
  const uint32_t span2 = hi2 - lo2;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int i = e * NT + tid;
    const uint32_t u = score_key(v[e]);
    const bool valid = i < cnt, in = valid && u >= lo && u <= hi;
    const unsigned long long mask = __ballot(in);
    if (mask) {
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&nlist, (uint32_t)__popcll(mask));
      base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
      if (in) list[base + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = (uint16_t)i;
    }
    if (valid && u > hi) {
      if (blockhist) list[MOST - 1 - (int)atomicAdd(&nsure, 1u)] = (uint16_t)i;   // (few; the two lists together hold at most cnt entries)
      else I[p0 + i] = kAboveAll;
    }
    if (!pools && valid && u >= lo2 && u < lo) I[p0 + i] = 0.f;   // (below tau, where its I' may be above)
  }
  __syncthreads();
  dense = (int)nlist > cnt / 4;
  for (int i = tid; i < (int)nsure; i += NT) pool(list[MOST - 1 - i], __float_as_uint(kAboveAll));
  const int nl = (int)nlist, ntiles = (nl + TK - 1) / TK;
  if (nl > 0) {
    const unsigned char* kbase = reinterpret_cast<const unsigned char*>(kmat_v) +
        ((int64_t)sg.head * k_stride_head + (int64_t)(sg.tok_begin + p0) * k_stride_tok) * 2;
    const uint32_t row_bytes = (uint32_t)k_stride_tok * 2u, piece_off = (uint32_t)(tid % CPR) * 16u;
    const int piece_row = tid / CPR;
    u32x4 pf0[LPT], pf1[LPT];
    auto issue_tile = [&](int t, u32x4 (&pf)[LPT]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        const int key = list[min(t * TK + piece_row + i * (NT / CPR), nl - 1)];
        pf[i] = *reinterpret_cast<const u32x4*>(kbase + ((uint32_t)key * row_bytes + piece_off));
      }
    };
    issue_tile(0, pf0);
    issue_tile(1, pf1);
    float lse_r[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) lse_r[i] = lse_s[rb * 32 + 8 * (i >> 2) + 4 * half + (i & 3)];
    auto tile = [&](int t, u32x4 (&pf)[LPT], int buf) __attribute__((always_inline)) {   // t == ntiles: only the sums of the tile before
      if (NB == 1) __syncthreads();                      // (every wave has read the tile before)
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        const int idx = i * NT + tid;
        *reinterpret_cast<u32x4*>(&ktile[buf % NB][(idx / CPR) * ROWB + (idx % CPR) * 16]) = pf[i];
      }
      issue_tile(t + 2, pf);
      __syncthreads();
      if (t > 0 && tid < TK) {                           // column sums of the previous tile
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < RB; ++r) sum += red[buf ^ 1][r][tid];
        const int li = (t - 1) * TK + tid;
        if (li < nl) {
          if (!pools) I[p0 + list[li]] = sum;
          else if (score_key(sum) >= lo2) pool(list[li], max(score_key(sum), 1u));   // (1: not "no key that matters")
        }
      }
      if (t == ntiles) return;
#pragma unroll
      for (int sb = 0; sb < NSUB; ++sb) {
        const int sub = ks + sb * KS;
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          Pack16 p;
          p.u = *reinterpret_cast<const u32x4*>(&ktile[buf % NB][(sub * 32 + l32) * ROWB + kk * 32 + half * 16]);
          acc = mfma16<KIND == 1>(qreg[kk], p.b, acc);
        }
        float colsum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) colsum += fast_exp2(fmaf(acc[i], c_log2, -lse_r[i]));
        colsum += __shfl_xor(colsum, 32, 64);
        if (half == 0) red[buf][rb][sub * 32 + l32] = colsum;
      }
    };
    for (int t = 0; t <= ntiles; t += 2) {
      tile(t, pf0, 0);
      if (t < ntiles) tile(t + 1, pf1, 1);
    }
  }
  if (!pools) return;
  __syncthreads();
  // pooled scores (exact from lo2 on) of positions first .. end - 1, those above the range counted, those in it listed
  constexpr int OWN = kRangeMost / NT;
  uint32_t key[OWN];
  uint32_t above = 0, in_band = 0;
#pragma unroll
  for (int e = 0; e < OWN; ++e) {
    const int j = first + e * NT + tid;
    const bool real = j < end;
    key[e] = 0;
    if (real) {
      key[e] = val[j - p0];
      if (dense)
        for (int t = max(j - radius, p0); t <= min(j + radius, p0 + cnt - 1); ++t) key[e] = max(key[e], val[t - p0]);
      if (!probe) pooled[sg.score_off + j] = __uint_as_float(key[e]);
    }
    above += (uint32_t)__popcll(__ballot(real && key[e] > lo2 + span2));
    in_band += (uint32_t)__popcll(__ballot(real && key[e] - lo2 <= span2));
  }
  if (probe || wide) {
    for (int i = tid; i < kHistBins; i += NT) bins[i] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < OWN; ++e)
      if (first + e * NT + tid < end && (key[e] || !probe)) atomicAdd(&bins[score_bin(key[e])], 1u);
    __syncthreads();
    for (int i = tid; i < kHistBins; i += NT)
      if (bins[i]) atomicAdd(&H[(probe ? kHistProbe : kHistExact) * kHistBins + i], bins[i]);
    return;
  }
  uint32_t base = 0;
  if (lane == 0) {
    if (above) atomicAdd(&nabove, above);
    if (in_band) base = atomicAdd(&nband, in_band);
  }
  base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
  __syncthreads();
  if (tid == 0) {
    uint32_t* const hdr = blockhist + (size_t)tab.blk_begin(seg) * kHistBins;
    if (nabove) atomicAdd(&hdr[6], nabove);
    band0 = nband ? atomicAdd(&hdr[7], nband) : 0u;
  }
  __syncthreads();
  if (in_band) {
    base += band0;
    uint32_t* const L = one.lists + (size_t)seg * kSelCandidates;
#pragma unroll
    for (int e = 0; e < OWN; ++e) {
      const bool in = first + e * NT + tid < end && key[e] - lo2 <= span2;
      const unsigned long long mask = __ballot(in);
      const uint32_t at = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if (in && at < (uint32_t)kSelCandidates) L[at] = key[e];
      base += (uint32_t)__popcll(mask);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Scoring of E4M3 keys (bf16 queries) and of fp32 inputs, on the matrix cores.
//
// A workgroup (4 or 8 waves) owns one chunk of history keys of one segment.  The query rows of the segment
// (in blocks of RBT 32-row tiles) sit in LDS, staged once; a wave holds a group of GK keys in registers as
// MFMA operands, loaded straight from memory (16 bytes of one key row per lane and load), and walks the query
// tiles over it while the loads of its next group are in flight.  Nothing is shared between the waves inside
// the loop, so there is no barrier in it and no key passes through LDS; E4M3 keys are widened to bf16 once, in
// registers.
//   PASS 1: D[key][row]: a lane owns one query row per tile -> sum of exp2(x - reference), kept per lane in
//           LDS between the groups; at the end the chunk's log-sum-exp of every row goes to `part`.
//   PASS 2: the segment's chunks are folded into the rows' log-sum-exp while the first keys are on their way;
//           D[row][key]: a lane owns one key per tile -> sum over all rows of exp2(x - lse[row]).
// A segment of a single chunk needs nobody else's rows: PASS 1 runs both passes over it.
// rsplit waves may share a key group and take its query tiles in turn (one group per wave then); the second pass adds
// their sums up in LDS.
//
// fp32 products run on the 32x32x2 fp32 MFMA: twice the rate of plain FMAs, and an operand is read from LDS once
// for 32 products instead of once for each (4 heads x 1024 keys, d 64: 16.4 + 12.1 us with FMAs, 8.6 + 7.8 us).
// E4M3, 8 heads x 32704 keys x 256 rows: 29.0 + 25.5 -> 26.5 + 23.2 us against score_q_resident_kernel's layout,
// which widened every key on its way into LDS.  For 16-bit keys that layout is the better one (see there): at
// these sizes both are bound by the power that the MFMAs and exponentials take, and it takes less.
//
// The 32x32x16 MFMA takes, per lane, 8 consecutive k-elements of row (lane%32) at k offset 8*(lane/32) for both
// operands (the 32x32x2 fp32 MFMA: one element, k offset lane/32) and returns in result register i the element
// at row 8*(i/4) + 4*(lane/32) + i%4, column lane%32.  Which 16-byte pieces of the rows meet in which MFMA is
// free as long as keys and queries agree: piece i of a key row is bytes 32*i + 16*(lane/32) of it.
// Rows beyond R and keys beyond the chunk are loaded from a clamped (valid) address and masked.
template <int DK, int KIND>   // KIND: 2 bf16 queries with E4M3 keys, 3 fp32
struct ScoreCfg {
  static constexpr bool F32 = KIND == 3, F8 = KIND == 2;
  static constexpr int QB = F32 ? 4 : 2;              // bytes of a query element
  static constexpr int KB = F32 ? 4 : 1;              // bytes of a key element in memory
  static constexpr int ROWB = DK * QB + 16;           // padded LDS row: conflict-free 16-byte reads down a column
  static constexpr int PPR = DK * QB / 16;            // 16-byte pieces of a query row
  static constexpr int KK = PPR / 2;                  // operand pieces per lane and row
  static constexpr int RAW = DK * KB / 32;            // pieces per lane and key as they come from memory
  static constexpr int KT = F32 ? 1 : 2;              // 32-key tiles of a group
  static constexpr int GK = 32 * KT;
  static constexpr int RBT = F32 && DK == 128 ? 4 : 8;   // query tiles per row block
};

// LDS of a scoring workgroup: query tiles of a row block, {reference, sum} per (wave, tile, lane) or the
// merge buffer of the prologue, log-sum-exp of the block's rows.
template <int DK, int KIND>
constexpr size_t score_lds_bytes(int tiles, int waves) {
  return (size_t)tiles * 32 * ScoreCfg<DK, KIND>::ROWB + (size_t)waves * tiles * 64 * sizeof(float2) + (size_t)tiles * 32 * sizeof(float);
}

template <int DK, int KIND, int PASS, class TAB>
__global__ __launch_bounds__(512, 2) void score_k_resident_kernel(const TAB tab, const void* __restrict__ qmat, const void* __restrict__ kmat,
                                                       int64_t k_stride_tok, int64_t k_stride_head, int R, int Rpad, int w,
                                                       int CH, float c_log2, float* __restrict__ part, float* __restrict__ imp,
                                                       int grid2d, int rsplit, uint32_t* __restrict__ gm,
                                                       meet_t* __restrict__ meet, int limit) {
  using C = ScoreCfg<DK, KIND>;
  constexpr int KK = C::KK, KT = C::KT, RAW = C::RAW, GK = C::GK, RBT = C::RBT, ROWB = C::ROWB, PPR = C::PPR;
  extern __shared__ __attribute__((aligned(16))) unsigned char score_smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthr = blockDim.x, NW = nthr >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  // wave: key groups kw, kw + KW, ..., query tiles rsub, rsub + rsplit, ...
  const int KW = NW / rsplit, kw = wv % KW, rsub = wv / KW;

  // Which chunk of which segment.  With a two-dimensional grid (grid2d; the host chooses it when the
  // segments' chunk counts are alike enough) blockIdx.y is the segment and blockIdx.x the chunk, and
  // workgroups past a segment's last chunk leave at once; otherwise blockIdx.x counts the chunks of
  // all segments and the segment is searched in the table.  The table is read through the scalar
  // cache, cold at every launch, so each dependent lookup costs a memory round trip before the
  // first key can be requested: the entries of segment blockIdx.y are therefore fetched before it
  // is known which case applies (y is 0 with a one-dimensional grid: a valid entry either way).
  struct SegEntry {
    int32_t n, tok_begin, head, qrow_off, score_off, chunk0, chunk1;
  };
  auto entry_of = [&](int s) {
    const SegShape sg = tab.shape(s);
    return SegEntry{sg.n, sg.tok_begin, sg.head, s * R, sg.score_off, tab.chunk_begin(s), tab.chunk_begin(s + 1)};
  };
  int seg = (int)blockIdx.y;
  SegEntry se = entry_of(seg);
  asm volatile("" :: "s"(se.n), "s"(se.tok_begin), "s"(se.head), "s"(se.qrow_off), "s"(se.chunk0), "s"(se.chunk1));   // fetched here, not behind the branch
  int bid;
  if (grid2d) {
    bid = se.chunk0 + (int)blockIdx.x;
    if (bid >= se.chunk1) return;
  } else {
    bid = blockIdx.x;
    seg = find_segment_wave(tab.nseg, bid, [&](int s) { return tab.chunk_begin(s); });
    se = entry_of(seg);
  }
  const int nchunks = se.chunk1 - se.chunk0;
  if (PASS == 2 && nchunks == 1) return;               // done by pass 1
  const int chunk = bid - se.chunk0;
  int key_begin, key_end, ngroups;
  auto set_chunk = [&](int c) __attribute__((always_inline)) {
    key_begin = c * CH;
    key_end = min(se.n - w, key_begin + CH);
    ngroups = (key_end - key_begin + GK - 1) / GK;
  };
  set_chunk(chunk);
  // uniform 64-bit base of the segment's keys + 32-bit byte offsets (the host checks the range)
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(kmat) +
      ((int64_t)se.head * k_stride_head + (int64_t)se.tok_begin * k_stride_tok) * C::KB;
  const uint32_t row_bytes = (uint32_t)k_stride_tok * (uint32_t)C::KB;

  // ---- the keys: group g of the chunk as this wave's operand registers
  u32x4 rawA[KT][RAW], rawB[KT][RAW];
  auto load = [&](u32x4 (&raw)[KT][RAW], int g) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const int key = min(key_begin + g * GK + kt * 32 + l32, key_end - 1);
      const unsigned char* row = kbase + ((uint32_t)key * row_bytes + (uint32_t)half * 16u);
#pragma unroll
      for (int i = 0; i < RAW; ++i) raw[kt][i] = *reinterpret_cast<const u32x4*>(row + i * 32);
    }
  };
  // f(registers, group) over this wave's groups kw, kw + KW, ..., two in registers in turn.  The loads past
  // the last group are issued too (of the chunk's last key; PASS 3: of the first two groups, for the sweep to come): only so
  // does the compiler know how many loads follow those it waits for.  preloaded: the first two groups are on their way already.
  auto sweep = [&](bool preloaded, auto f) __attribute__((always_inline)) {
    int g = kw;
    if (g >= ngroups) return;
    if (!preloaded) {
      load(rawA, g);
      load(rawB, g + KW);
    }
    for (;;) {
      f(rawA, g);
      load(rawA, PASS == 3 && g + 2 * KW >= ngroups ? kw : g + 2 * KW);
      g += KW;
      if (g >= ngroups) break;
      f(rawB, g);
      load(rawB, PASS == 3 && g + 2 * KW >= ngroups ? kw + KW : g + 2 * KW);
      g += KW;
      if (g >= ngroups) break;
    }
  };
  // pieces of a group as MFMA operands: what came from memory, or E4M3 bytes widened to bf16 (the hardware
  // converter gives exact fp32 values, checked against the format's definition for all 256 codes, whose upper
  // halves are the bf16 patterns; memory piece p becomes operand pieces 2p and 2p + 1)
  auto widen = [&](const u32x4 (&raw)[KT][RAW], u32x4 (&op)[KT][KK]) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int p = 0; p < RAW; ++p) {
        if constexpr (C::F8) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8((int)raw[kt][p][j], false);
            const f32x2 b = __builtin_amdgcn_cvt_pk_f32_fp8((int)raw[kt][p][j], true);
            op[kt][2 * p + (j >> 1)][2 * (j & 1)] = __builtin_amdgcn_perm(__float_as_uint(a[1]), __float_as_uint(a[0]), 0x07060302u);
            op[kt][2 * p + (j >> 1)][2 * (j & 1) + 1] = __builtin_amdgcn_perm(__float_as_uint(b[1]), __float_as_uint(b[0]), 0x07060302u);
          }
        } else {
          op[kt][p] = raw[kt][p];
        }
      }
  };
  // ---- the queries: LDS address of this lane's piece kk of its row of tile rt
  unsigned char* const qs = score_smem;
  auto q_piece = [&](int rt, int kk) __attribute__((always_inline)) {
    // E4M3 keys: memory piece p holds elements 32p + 16*half .. + 15, in operand pieces 2p, 2p + 1
    const int off = C::F8 ? (kk >> 1) * 64 + half * 32 + (kk & 1) * 16 : kk * 32 + half * 16;
    return *reinterpret_cast<const u32x4*>(qs + (rt * 32 + l32) * ROWB + off);
  };
  // logits of a group's keys and query tile rt (unscaled): keys x rows (pass 1) or rows x keys (pass 2)
  auto logits = [&](const u32x4 (&op)[KT][KK], int rt, auto keys_first_c, f32x16 (&acc)[KT]) __attribute__((always_inline)) {
    constexpr bool KEYS_FIRST = decltype(keys_first_c)::value;
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const u32x4 qp = q_piece(rt, kk);
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        if constexpr (C::F32) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float kf = __uint_as_float(op[kt][kk][e]), qf = __uint_as_float(qp[e]);
            acc[kt] = __builtin_amdgcn_mfma_f32_32x32x2f32(KEYS_FIRST ? kf : qf, KEYS_FIRST ? qf : kf, kk + e ? acc[kt] : z, 0, 0, 0);
          }
        } else {
          Pack16 kp, qq;
          kp.u = op[kt][kk];
          qq.u = qp;
          acc[kt] = mfma16<false>(KEYS_FIRST ? kp.b : qq.b, KEYS_FIRST ? qq.b : kp.b, kk ? acc[kt] : z);
        }
      }
    }
  };

  // ---- LDS behind the queries (sized for the first row block, the largest)
  const int tiles0 = min((R + 31) >> 5, RBT);
  float2* const stat = reinterpret_cast<float2*>(score_smem + (size_t)tiles0 * 32 * ROWB);   // [wave][tile][lane]
  float* const lse_s = reinterpret_cast<float*>(stat + (size_t)NW * tiles0 * 64);             // [row of the block]

  bool preloaded = true;
  load(rawA, kw);
  int rb0 = 0, rows, rts;                                // the row block at hand
  // queries of the block: memory -> LDS
  auto stage_queries = [&]() __attribute__((always_inline)) {
    rows = min(R - rb0, RBT * 32);
    rts = (rows + 31) >> 5;
      const unsigned char* qsrc = reinterpret_cast<const unsigned char*>(qmat) + ((int64_t)se.qrow_off + rb0) * (DK * C::QB);
      const int pieces = rts * 32 * PPR;
      for (int i0 = tid; i0 < pieces; i0 += 8 * nthr) {
        u32x4 t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = min(i0 + u * nthr, pieces - 1);
          t[u] = *reinterpret_cast<const u32x4*>(qsrc + (size_t)min(i / PPR, rows - 1) * (DK * C::QB) + (i % PPR) * 16);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = min(i0 + u * nthr, pieces - 1);
          *reinterpret_cast<u32x4*>(qs + (i / PPR) * ROWB + (i % PPR) * 16) = t[u];
        }
      }
  };
  // row statistics of the chunk: to memory, or (a segment of one chunk) the rows' log-sum-exp to LDS
  auto statistics = [&]() __attribute__((always_inline)) {
      float2* const mine = stat + (size_t)wv * tiles0 * 64 + lane;
      for (int rt = 0; rt < rts; ++rt) mine[rt * 64] = make_float2(0.f, 0.f);
      __syncthreads();
      // ONLINE: running maximum instead of a fixed reference
      auto stats_group = [&](const u32x4 (&raw)[KT][RAW], int g, auto online_c) __attribute__((always_inline)) {
        constexpr bool ONLINE = decltype(online_c)::value;
        u32x4 op[KT][KK];
        widen(raw, op);
        const int key0 = key_begin + g * GK;
        const bool first = g == kw, tail = key0 + GK > key_end;
#pragma unroll 1
        for (int rt = rsub; rt < rts; rt += rsplit) {
          float2 st = mine[rt * 64];
          f32x16 acc[KT];
          logits(op, rt, std::true_type{}, acc);
          // lane: query row l32 of the tile, keys key0 + kt*32 + 8*(i/4) + 4*half + i%4
          if (tail) {
            int left = key_end - key0 - 4 * half;
            asm volatile("" : "+v"(left));               // the comparisons stay here (hoisted out of the loop they would spill)
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
              for (int i = 0; i < 16; ++i)
                if (kt * 32 + 8 * (i >> 2) + (i & 3) >= left) acc[kt][i] = -INFINITY;
          }
          if (first || ONLINE) {
            // The reference of the exponentials is fixed by the lane's first logits of the chunk (any finite
            // reference gives the same log-sum-exp); later logits may exceed it by up to ~2^100 before the
            // sum overflows, which is detected below and repeated ONLINE.
            float mx = acc[0][0];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
              for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[kt][i]);
            const float ref = mx == -INFINITY ? (first ? 0.f : st.x) : mx * c_log2;
            if (first) {
              st = make_float2(ref, 0.f);
            } else if (ref > st.x) {
              st.y *= fast_exp2(st.x - ref);
              st.x = ref;
            }
          }
          float sum[KT];
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            sum[kt] = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum[kt] += fast_exp2(fmaf(acc[kt][i], c_log2, -st.x));
          }
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) st.y += sum[kt];
          mine[rt * 64] = st;
        }
      };
      sweep(preloaded, [&](const u32x4 (&raw)[KT][RAW], int g) __attribute__((always_inline)) { stats_group(raw, g, std::false_type{}); });
      bool bad = false;
      for (int rt = 0; rt < rts; ++rt) bad = bad || !(mine[rt * 64].y < INFINITY);
      if (__syncthreads_or(bad ? 1 : 0)) {
        // a sum that left the fp32 range (logits far above the chunk's first ones); not taken for ordinary inputs
        for (int g = kw; g < ngroups; g += KW) {
          load(rawA, g);
          stats_group(rawA, g, std::true_type{});
        }
        preloaded = false;
        __syncthreads();
      } else {
        preloaded = PASS == 3;
      }
      // the chunk's log-sum-exp of every row of the block (-inf: no key)
      for (int row = tid; row < rts * 32; row += nthr) {
        const float2* p = stat + (row >> 5) * 64 + (row & 31);
        float mm = -INFINITY, ss = 0.f;
        for (int v = 0; v < NW; ++v) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            // (reference, sum) -> (log-sum-exp, 1): a sum referenced to early logits can be very large or
            // small, and merging such pairs directly could lose it to an underflowing factor
            const float2 s = p[(size_t)v * tiles0 * 64 + h * 32];
            if (s.y > 0.f) merge_stats(mm, ss, s.x + __builtin_amdgcn_logf(s.y), 1.f);
          }
        }
        const float l = ss > 0.f ? mm + __builtin_amdgcn_logf(ss) : -INFINITY;
        if (nchunks == 1) lse_s[row] = row < rows && ss > 0.f ? l : INFINITY;
        else if (PASS == 3) __hip_atomic_store(part + ((int64_t)bid * Rpad + rb0 + row), l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else part[(int64_t)bid * Rpad + rb0 + row] = l;
      }
  };
  auto fold = [&]() __attribute__((always_inline)) {
    const float l = fold_rows<PASS == 3>(part, se.chunk0, se.chunk1, Rpad, rb0, rts * 32, nthr, stat);
    if (tid < rts * 32) lse_s[tid] = tid < rows ? l : INFINITY;
    __syncthreads();
  };
  // ---- importance of the chunk's keys: sum over the rows of exp2(x - lse)
  auto importance = [&]() __attribute__((always_inline)) {
    float* const dst = imp + se.score_off;
    float* const col = reinterpret_cast<float*>(stat);   // [wave][lane]
    if (rsplit > 1) col[tid] = 0.f;                      // (of a wave without keys)
    auto put = [&](int g, float v) __attribute__((always_inline)) {
      const int key = key_begin + g * GK + (KT == 2 ? lane : l32);
      const bool mine = key < key_end && (KT == 2 || half == 0);
      if (mine && rb0) v += dst[key];                    // (a later row block adds to what this lane wrote)
      if (mine) dst[key] = v;
      if (C::F8 && gm && rb0 + RBT * 32 >= R) {          // (the last row block; fp32: not asked for)
        const uint32_t top = max_8_lanes(key < key_end ? score_key(v) : 0u);
        if (mine && lane % kGroup == 0) gm[group_off(se.score_off, seg) + key / kGroup] = top;
      }
    };
    sweep(preloaded, [&](const u32x4 (&raw)[KT][RAW], int g) __attribute__((always_inline)) {
      u32x4 op[KT][KK];
      widen(raw, op);
      float colsum[KT];
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) colsum[kt] = 0.f;
#pragma unroll 1
      for (int rt = rsub; rt < rts; rt += rsplit) {
        // lane: key l32 of tile kt, query rows rt*32 + 8*(i/4) + 4*half + i%4
        f32x16 acc[KT];
        logits(op, rt, std::false_type{}, acc);
        f32x4v l[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) l[j] = *reinterpret_cast<const f32x4v*>(&lse_s[rt * 32 + 8 * j + 4 * half]);
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) colsum[kt] += fast_exp2(fmaf(acc[kt][i], c_log2, -l[i >> 2][i & 3]));
      }
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) colsum[kt] += __shfl_xor(colsum[kt], 32, 64);
      const float v = KT == 2 && half ? colsum[KT - 1] : colsum[0];
      if (rsplit > 1) col[tid] = v;
      else put(g, v);
    });
    if (rsplit > 1) {                                    // one group per wave: the sums of its query tiles
      __syncthreads();
      if (rsub == 0 && kw < ngroups) {
        float v = 0.f;
        for (int r = 0; r < rsplit; ++r) v += col[(r * KW + kw) * 64 + lane];
        put(kw, v);
      }
    }
    preloaded = PASS == 3;
  };

  for (; rb0 < R; rb0 += RBT * 32) {
    if (rb0 > 0) __syncthreads();
    stage_queries();
    if (rb0 == 0) load(rawB, kw + KW);                 // behind the queries: the first group does not wait for it
    if (PASS == 2) {
      fold();
    } else {
      statistics();
      if (nchunks > 1) continue;
      __syncthreads();
    }
    importance();
  }
  if constexpr (PASS == 3) {
    if (nchunks == 1) return;
    // The second pass, with the first keys on their way and (one row block) the queries where they are.  As a rule over this chunk
    // alone; `left`, in thread 0: those whose workgroups have left.
    __shared__ int sh_next;
    meet_t* const word = meet + (int64_t)seg * kMeetWords;
    meet_t left = 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the statistics are in memory
    __syncthreads();
    if (tid == 0) {
      left = meet_chunks(word, nchunks, chunk, limit);
      sh_next = left != kMeetLeft ? chunk : -1;
    }
    for (;;) {
      __syncthreads();
      const int next = sh_next;
      if (next < 0) return;
      if (next != chunk) {
        set_chunk(next);
        preloaded = false;
      }
      for (rb0 = 0; rb0 < R; rb0 += RBT * 32) {
        if (R > RBT * 32) {
          if (rb0 > 0) __syncthreads();
          stage_queries();
        }
        fold();
        importance();
      }
      __syncthreads();                                   // (every thread has read sh_next, and the sums in LDS)
      if (tid == 0) sh_next = meet_take(word, left);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Pooling + top-k (Algorithm 3, steps 7-8).  Writes the kept positions: history positions
// ascending, then the window.
//
// Histories longer than one round of kSelRound positions take six launches; whatever touches every
// position runs with one workgroup per block of kSelBlock positions, only the digit searches run
// per segment (the block-wise kernels are described where they are defined):
//   select_pool_kernel: pool the block's importance scores (halo from the neighbours), write the
//     pooled scores, histogram their leading 11 key bits, write the block's histogram;
//   select_rank_kernel, phase 0: one workgroup per segment adds the block histograms and picks
//     the digit that holds the k-th largest score;
//   select_collect_kernel: the blocks copy their scores of that digit to the segment's list;
//   select_rank_kernel, phase 1: narrows the list down to the exact k-th largest value tau and
//     the number of scores equal to tau that belong to the top k (ties go to lower positions);
//     it also writes the window's positions and those of segments that are not ranked;
//   select_count_kernel, select_emit_kernel: the kept history positions, block by block: those
//     with score > tau, or == tau among the first `need_eq`.
// (One kernel with a per-segment ticket, the last block doing the ranking, was measured and
// dropped: with 1024-thread workgroups at one per CU, the blocks of later segments queue behind
// ranking workgroups and start tens of microseconds late.)
// Keys are the bit patterns of the pooled scores (>= 0, so monotone).  While ranking, a wave owns
// 2048 consecutive positions of a round, lane l the positions 64*j + l (j < 32).
// Slices: where the chip has CUs to spare, further workgroups of select_resident_kernel select again for a segment that keeps more than 64 rows (128
// where only so few fit), each to write and copy that many of them.  The selection of a segment is a chain of phases that takes as
// long on one CU as on ten; the copies, a few us where one workgroup holds 128 to 256 rows, and the gather launch (4 us) for those with more, are what
// it saves.  us a call, without / slices of 32 / 64 / 128 / 256 rows: 8 x 32 K, 107 to 1834 kept 57.7 / - / 56.3 / 57.4 / 59.3; 8 x 21 K, 397 to 7655 kept
// 59.6 / - / 55.3 / 56.6 / 58.7; 16 short prompts 45.4 / - / 45.0 / 43.4 / 44.7; one sequence's cache, 58 to 865 kept 20.7 / 18.9 / 19.1 / 19.5 / 20.5;
// 8 x 8 K, 91 to 155 kept 25.5 / 24.6 / 24.8 / 25.5; 8 x 16 K, 220 kept 30.6 / 28.9 / 29.1 / 29.8; 4 x 1 K fp32, 105 to 137 kept 19.9 / - / 20.1: not
// where the shortest form selects and nothing would be left to the gather.  Two workgroups to a CU (a decode cache of 256 segments, 480 slices
// of 256) 60.8 / 60.5: not worth their LDS.
constexpr int kSliceLog2Least = 6, kSliceLog2Most = 7;
constexpr int kInlineGatherRows = 256;    // without slices: segments up to this many kept rows are gathered by the selection kernel

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelBlock = 4096;           // history positions per phase-A block
constexpr int kSelEmitThreads = 256;      // workgroup of the block-wise count / emit kernels (16 positions per thread)
constexpr int kSelEPT = 32;
constexpr int kSelEPTLong = 24, kSelEPTMore = 16, kSelEPTMid = 8, kSelEPTLess = 4, kSelEPTSmall = 2;   // shorter histories: fewer positions per thread in the one-workgroup kernel
constexpr int kSelRound = kSelThreads * kSelEPT;
constexpr int kSelRankMax = 256;          // lists up to this length are ranked by direct counting
constexpr int kSelTieGroups = 512;        // this many group maxima in the bound's digit switch the histograms to the pile-aware step
constexpr int kSelTrackMax = 512;         // up to this many wanted keys the first level also tracks the largest and smallest key of every digit
constexpr int kDigitShift = 20;           // first-level digit = key >> 20: sign (0), 8 exponent and 3 mantissa bits
static_assert((0x7f800000u >> kDigitShift) < (uint32_t)kHistBins, "every key has a first-level digit inside the histogram");

__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

template <int RADIUS, class TAB>   // pooling radius known at compile time (0..3), or -1: any radius
__global__ __launch_bounds__(kSelThreads) void select_pool_kernel(const TAB tab, int w, int pool_kernel, int pool_mode,
                                                                  const float* __restrict__ imp, float* __restrict__ pooled,
                                                                  uint32_t* __restrict__ blockhist) {
  constexpr int NT = kSelThreads;
  __shared__ uint32_t hist[kHistBins];
  __shared__ float stage[kSelBlock + 2 * kSelHaloMax];
  const int tid = threadIdx.x;
  const int bid = blockIdx.x;
  const int seg = find_segment_wave(tab.nseg, bid, [&](int s) { return tab.blk_begin(s); });
  const int blk = bid - tab.blk_begin(seg);
  const SegShape sg = tab.shape(seg);
  const int n = sg.n;
  const int kk = sg.kk;
  const int m = n - w;
  if (!(kk > 0 && kk < m)) return;                    // not ranked: nothing to pool (such segments have no block)
  SLKV_STAMP(bid, 0);
  const float* I = imp + sg.score_off;
  float* P = pooled + sg.score_off;
  const int radius = RADIUS >= 0 ? RADIUS : pool_kernel / 2;
  const bool is_max = pool_mode != SLKV_POOL_AVG;
  const float fill = is_max ? -INFINITY : 0.f;
  const float inv_p = 1.f / (float)pool_kernel;
  const int p0 = blk * kSelBlock;
  const int cnt = min(kSelBlock, m - p0);
  for (int s = tid; s < cnt + 2 * radius; s += NT) {   // stage[s] = importance at position p0 - radius + s
    const int j = p0 - radius + s;
    stage[s] = (j >= 0 && j < m) ? I[j] : fill;
  }
  for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kSelBlock / NT; ++e) {
    const int s = e * NT + tid;
    if (s < cnt) {
      float a = stage[s];
      if (RADIUS >= 0) {
#pragma unroll
        for (int t = 1; t <= 2 * (RADIUS >= 0 ? RADIUS : 0); ++t) a = is_max ? fmaxf(a, stage[s + t]) : a + stage[s + t];
      } else {
        for (int t = 1; t <= 2 * radius; ++t) a = is_max ? fmaxf(a, stage[s + t]) : a + stage[s + t];
      }
      if (!is_max) a *= inv_p;
      P[p0 + s] = a;
      atomicAdd(&hist[score_key(a) >> kDigitShift], 1u);
    }
  }
  __syncthreads();
  uint32_t* bh = blockhist + (size_t)(tab.blk_begin(seg) + blk) * kHistBins;
  for (int i = tid; i < kHistBins; i += NT) bh[i] = hist[i];
  SLKV_STAMP(bid, 1);
}

// Phase B: one workgroup per segment (unranked segments only write their positions).
template <class TAB>
__global__ __launch_bounds__(kSelThreads) void select_rank_kernel(const TAB tab, int w, const float* __restrict__ pooled,
                                                                  uint32_t* __restrict__ blockhist,
                                                                  int32_t* __restrict__ kept_idx, int64_t* __restrict__ d_out_offsets,
                                                                  const GatherArgs ga, int split_emit,
                                                                  const uint32_t* __restrict__ lists, int phase, const OneScan one) {
  constexpr int NT = kSelThreads, NW = kSelWaves, EPT = kSelEPT, ROUND = kSelRound;
  __shared__ uint32_t hist[kHistBins];
  __shared__ uint32_t cand[kSelCandidates];
  __shared__ uint32_t small_list[kSelRankMax];
  __shared__ int32_t sh_pos[kInlineGatherRows];
  __shared__ uint32_t sh_scan[NW];
  __shared__ uint32_t res[4];

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int seg = blockIdx.x;
  const int bid = seg;
  (void)bid;                                           // (only the development stamps use it)
  const int nblk = tab.blk_begin(seg + 1) - tab.blk_begin(seg);
  const SegShape sg = tab.shape(seg);
  const int n = sg.n;
  const int kk = sg.kk;
  const int m = n - w;
  const int kept = tab.out_off(seg + 1) - tab.out_off(seg);
  const bool small_seg = !split_emit && kept <= kInlineGatherRows;   // (split_emit: the launch has ranked segments, and gather_kernel copies every row)
  int32_t* out = kept_idx + tab.out_off(seg);
  if (d_out_offsets && tid == 0 && phase != 0) {
    d_out_offsets[seg] = tab.out_off(seg);
    if (seg == tab.nseg - 1) d_out_offsets[seg + 1] = tab.out_off(tab.nseg);
  }
  auto emit = [&](int pos, int j) __attribute__((always_inline)) {   // kept position j goes to output slot pos
    if ((uint32_t)pos < (uint32_t)kept) {
      out[pos] = j;
      if (small_seg) sh_pos[pos] = j;
    }
  };
  SLKV_STAMP(bid, 2);
  if (small_seg)
    for (int i = tid; i < kInlineGatherRows; i += NT) sh_pos[i] = 0;
  __syncthreads();
  const bool ranked = kk > 0 && kk < m;
  // Ranked segments take two launches of this kernel with select_collect_kernel between them
  // (words 4.. of the segment's first histogram row carry the state across):
  //   phase 0: add up the block histograms, find the first-level digit of the k-th largest score;
  //   (collect: the blocks copy their scores of that digit to the segment's list in memory)
  //   phase 1: rank the list, or, if the digit holds more scores than the LDS list, narrow it by
  //            sweeps over the pooled array; write the window's positions.
  if (phase == 0 && !ranked) return;
  uint32_t* const hdr = blockhist + (size_t)tab.blk_begin(seg) * kHistBins;   // (used for ranked segments only)
  if (!ranked) {
    if (kk < 0) {
      for (int j = tid; j < n; j += NT) emit(j, j);
    } else {
      for (int j = tid; j < w; j += NT) emit(j, m + j);   // kk == 0: the window alone
    }
  } else {
    const float* P = pooled + sg.score_off;
    if (phase == 0) {
      // first-level histogram of the segment: the sum of its blocks' histograms
      static_assert(kHistBins == 2 * NT, "a thread adds up two bins");
      const uint32_t* bh0 = blockhist + (size_t)tab.blk_begin(seg) * kHistBins;
      uint32_t a0 = 0, a1 = 0;
      for (int b0 = 0; b0 < nblk; b0 += 24) {             // 48 loads in flight
        uint32_t v0[24], v1[24];
#pragma unroll
        for (int u = 0; u < 24; ++u) {
          const int b = min(b0 + u, nblk - 1);
          v0[u] = bh0[(size_t)b * kHistBins + tid];
          v1[u] = bh0[(size_t)b * kHistBins + NT + tid];
        }
#pragma unroll
        for (int u = 0; u < 24; ++u)
          if (b0 + u < nblk) {
            a0 += v0[u];
            a1 += v1[u];
          }
      }
      hist[tid] = a0;
      hist[NT + tid] = a1;
      __syncthreads();
      SLKV_STAMP(bid, 3);
      select_bin<NT>(hist, (uint32_t)kk, sh_scan, res);
      if (tid == 0) {
        const uint32_t in_range = hist[res[0]];
        hdr[4] = res[0] << kDigitShift;                    // [lo, hi]: the keys of the chosen digit
        hdr[5] = (res[0] << kDigitShift) + ((1u << kDigitShift) - 1u);
        hdr[6] = res[1];                                  // rank of the wanted key inside the digit
        hdr[7] = 0;                                       // length of the list (filled by the blocks)
        hdr[8] = in_range;
        hdr[9] = in_range <= (uint32_t)kSelCandidates ? 1u : 0u;   // 1: the blocks list the digit's scores
      }
      SLKV_STAMP(bid, 5);
      return;
    }
    // ---------------- the k-th largest pooled score of the segment
    const int rounds = (m + ROUND - 1) / ROUND;
    const bool multi = rounds > 1;
    uint32_t key[EPT];
    auto load_round = [&](int r) __attribute__((always_inline)) {
      const int base = r * ROUND + wv * (64 * EPT) + lane;
      float ld[EPT];
#pragma unroll
      for (int j = 0; j < EPT; ++j) ld[j] = P[min(base + j * 64, m - 1)];
#pragma unroll
      for (int j = 0; j < EPT; ++j) key[j] = base + j * 64 < m ? score_key(ld[j]) : kKeyNone;
    };
    // f(key) over every score of the segment (rounds beyond the first re-read the pooled array)
    auto sweep = [&](auto f) __attribute__((always_inline)) {
      for (int r = 0; r < rounds; ++r) {
        if (multi) load_round(r);
#pragma unroll
        for (int j = 0; j < EPT; ++j) f(key[j]);
      }
    };
    // (chosen: after select_chosen_kernel, word 6 counts the scores above the range instead)
    const bool chosen = one.hist != nullptr;
    uint32_t lo = hdr[4], hi = hdr[5], k = chosen ? (uint32_t)kk - hdr[6] : hdr[6], in_range = chosen ? hdr[7] : hdr[8];
    bool use_list = chosen ? in_range <= (uint32_t)kSelCandidates : hdr[9] != 0u;
    uint32_t ncand = min(hdr[7], (uint32_t)kSelCandidates);   // (== in_range when the list is used)
    if (chosen && one.bounds[seg * kBoundWords + kBoundWide]) {
      // select_chosen_kernel has counted the scores per bin instead: those of the k-th largest one's bin, from the pooled array into the list
      for (int i = tid; i < kHistBins; i += NT) hist[i] = one.hist[((size_t)seg * kHists + kHistExact) * kHistBins + i];
      if (tid == 0) res[2] = 0;
      __syncthreads();
      select_bin<NT>(hist, (uint32_t)kk, sh_scan, res);
      const uint32_t b = res[0];
      k = res[1];
      in_range = hist[b];
      lo = b ? (b + kBinBase) << kBinShift : 0u;
      hi = b == (uint32_t)kHistBins - 1u ? 0x7f800000u : ((b + 1u + kBinBase) << kBinShift) - 1u;
      use_list = in_range <= (uint32_t)kSelCandidates;
      ncand = in_range;
      if (use_list || !multi)
        for (int r = 0; r < rounds; ++r) {
          load_round(r);
          if (use_list)
#pragma unroll
            for (int j = 0; j < EPT; ++j)
              if (key[j] >= lo && key[j] <= hi) {
                const uint32_t slot = atomicAdd(&res[2], 1u);
                if (slot < (uint32_t)kSelCandidates) cand[slot] = key[j];
              }
        }
      __syncthreads();
    } else if (use_list) {
      // the scores of the chosen digit, listed by the blocks: into LDS
      const uint32_t* L = lists + (chosen ? (int64_t)seg * kSelCandidates : (int64_t)sg.score_off);
      for (uint32_t i = tid; i < ncand; i += NT) cand[i] = L[i];
      __syncthreads();
    } else if (!multi) {
      load_round(0);
    }
    SLKV_STAMP(bid, 4);
    SLKV_STAMP(bid, 6);
    // narrow [lo, hi] down to one value: 11 bits per level over what is left of the range
    for (;;) {
      if (in_range <= (uint32_t)kSelRankMax && (use_list || lo == hi)) {
        if (lo == hi) break;                              // every score left equals lo
        // short list: gather the scores still in range, then the k-th largest by counting
        if (tid == 0) res[3] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < ncand; i += NT) {
          const uint32_t kv = cand[i];
          if (kv >= lo && kv <= hi) {
            const uint32_t slot = atomicAdd(&res[3], 1u);
            if (slot < (uint32_t)kSelRankMax) small_list[slot] = kv;
          }
        }
        __syncthreads();
        const uint32_t ns = min(res[3], (uint32_t)kSelRankMax);
        if ((uint32_t)tid < ns) {
          const uint32_t kv = small_list[tid];
          uint32_t gt = 0, ge = 0;
          for (uint32_t i = 0; i < ns; ++i) {
            const uint32_t o = small_list[i];
            gt += o > kv ? 1u : 0u;
            ge += o >= kv ? 1u : 0u;
          }
          if (gt < k && k <= ge) {   // every thread holding the k-th largest value writes the same pair
            res[0] = kv;
            res[1] = k - gt;
          }
        }
        __syncthreads();
        lo = hi = res[0];
        k = res[1];
        __syncthreads();
        break;
      }
      const uint32_t span1 = hi - lo;
      const int nbits = span1 ? 32 - __clz(span1) : 0;
      const int shift = nbits > 11 ? nbits - 11 : 0;
      for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
      __syncthreads();
      if (use_list) {
        for (uint32_t i = tid; i < ncand; i += NT) {
          const uint32_t kv = cand[i];
          if (kv >= lo && kv <= hi) atomicAdd(&hist[(kv - lo) >> shift], 1u);
        }
      } else {
        sweep([&](uint32_t kv) {
          if (kv >= lo && kv <= hi) atomicAdd(&hist[(kv - lo) >> shift], 1u);
        });
      }
      __syncthreads();
      select_bin<NT>(hist, k, sh_scan, res);
      in_range = hist[res[0]];
      k = res[1];
      lo = lo + (res[0] << shift);
      hi = min(hi, lo + ((1u << shift) - 1u));
      __syncthreads();
      if (shift == 0) break;
    }
    const uint32_t tau = lo, need_eq = k;
    SLKV_STAMP(bid, 7);

    // The kept history positions are written by select_count_kernel + select_emit_kernel, one
    // workgroup per block of the history: they find the threshold in words 2 and 3 of the segment's
    // first block histogram (read in full above, not needed again in this call).
    if (tid == 0) {
      hdr[2] = tau;
      hdr[3] = need_eq;
    }
    for (int j = tid; j < w; j += NT) emit(kk + j, m + j);
    SLKV_STAMP(bid, 8);
  }

  // Small segments copy their K/V rows here (saves the gather launch); larger ones are left
  // to gather_kernel, which skips the segments handled here.
  if (kept > 0 && small_seg) {
    __syncthreads();                                // sh_pos is complete
    const int64_t tok0 = sg.tok_begin, h = sg.head, row0 = tab.out_off(seg);
    const int pieces = kept * ga.lanes_per_row;
    for (int idx = tid; idx < pieces; idx += NT) {
      const int row = idx / ga.lanes_per_row, c = idx % ga.lanes_per_row;
      const int64_t tok = tok0 + sh_pos[row];
      const uint4 kv = *reinterpret_cast<const uint4*>(ga.k + (h * ga.k_stride_head + tok * ga.k_stride_tok) * ga.elt_bytes + c * 16);
      const uint4 vv = *reinterpret_cast<const uint4*>(ga.v + (h * ga.v_stride_head + tok * ga.v_stride_tok) * ga.elt_bytes + c * 16);
      const int64_t o = ((row0 + row) * ga.lanes_per_row + c) * 16;
      *reinterpret_cast<uint4*>(ga.k_out + o) = kv;
      *reinterpret_cast<uint4*>(ga.v_out + o) = vv;
      if (ga.pos_out && c == 0) ga.pos_out[row0 + row] = ga.pos_in[tok];
    }
  }
  SLKV_STAMP(bid, 9);
}

// Between the two phases of select_rank_kernel: every block copies its scores of the digit chosen
// for its segment (keys in [lo, hi], words 4 and 5 of the segment's first histogram row) to the
// segment's list in memory, in any order: one atomic on the list's length (word 7) per wave.
// Nothing is listed when the digit holds more scores than the ranking workgroup's LDS list (word 9).
template <class TAB>
__global__ __launch_bounds__(kSelEmitThreads) void select_collect_kernel(const TAB tab, int w, const float* __restrict__ pooled,
                                                                     uint32_t* __restrict__ blockhist,
                                                                     uint32_t* __restrict__ lists, int seg0) {
  constexpr int NT = kSelEmitThreads, PER = kSelBlock / NT;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int seg, blk;
  if (seg0 >= 0) {
    seg = seg0 + (int)blockIdx.y;
    blk = blockIdx.x;
    if (blk >= tab.blk_begin(seg + 1) - tab.blk_begin(seg)) return;
  } else {
    seg = find_segment_wave(tab.nseg, (int)blockIdx.x, [&](int s) { return tab.blk_begin(s); });
    blk = (int)blockIdx.x - tab.blk_begin(seg);
  }
  const SegShape sg = tab.shape(seg);
  const int m = sg.n - w;
  const int kk = sg.kk;
  if (!(kk > 0 && kk < m)) return;
  uint32_t* hdr = blockhist + (size_t)tab.blk_begin(seg) * kHistBins;
  const float* P = pooled + sg.score_off;
  const int p0 = blk * kSelBlock + wv * (64 * PER) + lane;
  float pv[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) pv[j] = P[min(p0 + j * 64, m - 1)];
  if (hdr[9] == 0u) return;
  const uint32_t lo = hdr[4], span = hdr[5] - lo;
  uint32_t* L = lists + sg.score_off;         // as long as the history: every list fits
  uint32_t key[PER];
  uint32_t c = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    key[j] = p0 + j * 64 < m ? score_key(pv[j]) : kKeyNone;
    c += (uint32_t)__popcll(__ballot(key[j] - lo <= span));   // (kKeyNone - lo exceeds every span)
  }
  if (c) {
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&hdr[7], c);
    base = (uint32_t)__shfl((int)base, 0, 64);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool in = key[j] - lo <= span;
      const unsigned long long mask = __ballot(in);
      if (in) L[base + lanes_below(mask)] = key[j];
      base += (uint32_t)__popcll(mask);
    }
  }
}

// Ordered compaction of long histories, spread over the blocks of select_pool_kernel (one
// workgroup per kSelBlock positions) once select_rank_kernel has left the threshold tau and the
// number need_eq of positions equal to tau that are kept (the first ones in position order):
//   select_count_kernel: positions of the block above tau / equal to tau -> words 0, 1 of the
//     block's histogram row (free by now);
//   select_emit_kernel: sums the counts of the segment's earlier blocks, scans its own positions
//     (a wave owns 1024 consecutive ones) and writes the kept ones to their output slots:
//     slot = (#greater before) + min(#equal before, need_eq).
template <class TAB>
__global__ __launch_bounds__(kSelEmitThreads) void select_count_kernel(const TAB tab, int w, const float* __restrict__ pooled,
                                                                   uint32_t* __restrict__ blockhist, int seg0) {
  constexpr int NT = kSelEmitThreads, PER = kSelBlock / NT;
  __shared__ uint32_t sh[NT / 64];
  const int tid = threadIdx.x;
  // seg0 >= 0: one grid row per segment (no search in the table; blocks past the segment's last
  // one leave at once); seg0 < 0: one row over all blocks
  int seg, blk;
  if (seg0 >= 0) {
    seg = seg0 + (int)blockIdx.y;
    blk = blockIdx.x;
    if (blk >= tab.blk_begin(seg + 1) - tab.blk_begin(seg)) return;
  } else {
    seg = find_segment_wave(tab.nseg, (int)blockIdx.x, [&](int s) { return tab.blk_begin(s); });
    blk = (int)blockIdx.x - tab.blk_begin(seg);
  }
  const SegShape sg = tab.shape(seg);
  const int m = sg.n - w;
  const int kk = sg.kk;
  if (!(kk > 0 && kk < m)) return;                    // (such segments have no block)
  uint32_t* row0 = blockhist + (size_t)tab.blk_begin(seg) * kHistBins;
  const uint32_t tau = row0[2];
  const float* P = pooled + sg.score_off;
  const int p0 = blk * kSelBlock + tid;               // (which thread counts which position does not matter here)
  uint32_t cg = 0, ce = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = p0 + e * NT;
    const uint32_t kv = score_key(P[min(j, m - 1)]);
    if (j < m) {
      cg += kv > tau ? 1u : 0u;
      ce += kv == tau ? 1u : 0u;
    }
  }
  const uint32_t tot = block_sum<NT, uint32_t>((ce << 16) | cg, sh);   // a block holds 4096 positions: 13 bits each
  if (tid == 0) {
    uint32_t* row = row0 + (size_t)blk * kHistBins;
    row[0] = tot & 0xffffu;
    row[1] = tot >> 16;
  }
}

template <class TAB>
__global__ __launch_bounds__(kSelEmitThreads) void select_emit_kernel(const TAB tab, int w, const float* __restrict__ pooled,
                                                                  const uint32_t* __restrict__ blockhist,
                                                                  int32_t* __restrict__ kept_idx, int seg0) {
  constexpr int NT = kSelEmitThreads, PER = kSelBlock / NT;
  __shared__ uint32_t sh[NT / 64];
  const int tid = threadIdx.x;
  // seg0 >= 0: one grid row per segment (no search in the table; blocks past the segment's last
  // one leave at once); seg0 < 0: one row over all blocks
  int seg, blk;
  if (seg0 >= 0) {
    seg = seg0 + (int)blockIdx.y;
    blk = blockIdx.x;
    if (blk >= tab.blk_begin(seg + 1) - tab.blk_begin(seg)) return;
  } else {
    seg = find_segment_wave(tab.nseg, (int)blockIdx.x, [&](int s) { return tab.blk_begin(s); });
    blk = (int)blockIdx.x - tab.blk_begin(seg);
  }
  const SegShape sg = tab.shape(seg);
  const int m = sg.n - w;
  const int kk = sg.kk;
  if (!(kk > 0 && kk < m)) return;
  const uint32_t* row0 = blockhist + (size_t)tab.blk_begin(seg) * kHistBins;
  const uint32_t tau = row0[2], need_eq = row0[3];
  const int kept = tab.out_off(seg + 1) - tab.out_off(seg);
  int32_t* out = kept_idx + tab.out_off(seg);
  const float* P = pooled + sg.score_off;
  // this block's own positions first (the loads fly while the earlier blocks are added up): a wave
  // owns 64 * PER consecutive positions, lane l the positions 64 j + l, so that loads are coalesced
  // and ballots are in position order
  const int lane = tid & 63, wv = tid >> 6;
  const int p0 = blk * kSelBlock + wv * (64 * PER) + lane;
  float pv[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) pv[j] = P[min(p0 + j * 64, m - 1)];
  // kept positions before this block: greater, and equal (capped at need_eq when they are used)
  uint32_t pg = 0, pe = 0;
  for (int b = tid; b < blk; b += NT) {
    pg += row0[(size_t)b * kHistBins];
    pe += row0[(size_t)b * kHistBins + 1];
  }
  // (a segment has at most 2^31 / kSelBlock blocks of at most 4096 positions: the sums fit 32 bits each)
  const uint32_t g0 = block_sum<NT, uint32_t>(pg, sh);
  const uint32_t e0 = block_sum<NT, uint32_t>(pe, sh);
  uint32_t key[PER];
  uint32_t wg = 0, we = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    key[j] = p0 + j * 64 < m ? score_key(pv[j]) : kKeyNone;
    wg += (uint32_t)__popcll(__ballot(key[j] > tau && key[j] != kKeyNone));
    we += (uint32_t)__popcll(__ballot(key[j] == tau));
  }
  __shared__ uint32_t sh_wg[NT / 64], sh_we[NT / 64];
  if (lane == 0) {
    sh_wg[wv] = wg;
    sh_we[wv] = we;
  }
  __syncthreads();
  uint32_t g = g0, q = e0;                            // greater / equal before this wave's positions
#pragma unroll
  for (int v2 = 0; v2 < NT / 64; ++v2)
    if (v2 < wv) {
      g += sh_wg[v2];
      q += sh_we[v2];
    }
  if (wg + we) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool isg = key[j] > tau && key[j] != kKeyNone;
      const bool ise = key[j] == tau;
      const unsigned long long mg = __ballot(isg), me = __ballot(ise);
      if (mg | me) {
        const uint32_t my_g = g + lanes_below(mg);
        const uint32_t my_e = q + lanes_below(me);    // ties are taken in position order
        uint32_t pos = 0xffffffffu;
        if (isg) pos = my_g + min(my_e, need_eq);
        else if (ise && my_e < need_eq) pos = my_g + my_e;
        if (pos < (uint32_t)kept) out[pos] = p0 + j * 64;
        g += (uint32_t)__popcll(mg);
        q += (uint32_t)__popcll(me);
      }
    }
  }
}

// The same selection for launches whose histories all fit one round of kSelRound positions: one
// workgroup per segment does everything, and the scores never leave its registers between the
// first load and the last store (no second workgroup to wait for, no re-read).  Thread t owns 32
// consecutive positions (values reach it through an LDS transposition of coalesced loads), so
// pooling is a sliding window in registers and the ordered compaction is one block scan of
// packed (greater, equal) counts plus per-thread bit masks.  The radix levels take their 11-bit
// digits relative to the range of keys still in question, which spreads the LDS histogram over
// nearly all bins and leaves few scores in the chosen one; where k allows, the range is first cut
// from below by the k-th largest of per-group maxima (see the search in the kernel).
constexpr int kResStageFloats = kSelRound + 2 * kSelHaloMax + ((kSelRound + 2 * kSelHaloMax) >> 5) + 8;
constexpr int kResCandidates = 3072;   // keys that the list behind the staging array can hold
constexpr int kResAuxWords = 3 * kHistBins;   // second histogram, largest and smallest key per digit: the start of the staging array, once the scores are in registers
// For every EPT, although the shorter forms need less: a workgroup has its CU to itself, and more than 256 segments run in rounds.
constexpr size_t kResLdsBytes = (size_t)(kResStageFloats + kResCandidates) * sizeof(float);

// index into the staging array: one word of padding per thread's positions, so that the threads
// of a wave read their consecutive positions from different banks
template <int EPT>
__device__ __forceinline__ int pad_idx(int i) { return i + i / EPT; }

template <int RADIUS, int EPT_, class TAB>   // pooling radius known at compile time (0..3), or -1: any radius, window read from LDS;
                                             // EPT_: positions per thread (the history is at most 1024 * EPT_ positions)
__global__ __launch_bounds__(kSelThreads) void select_resident_kernel(const TAB tab, int w, int pool_kernel, int pool_mode,
                                                                      int write_pooled, const float* __restrict__ imp, const uint32_t* __restrict__ gm,
                                                                      float* __restrict__ pooled, int32_t* __restrict__ kept_idx,
                                                                      int64_t* __restrict__ d_out_offsets, const GatherArgs ga,
                                                                      meet_t* __restrict__ meet, int slice_log2) {
  constexpr int NT = kSelThreads, EPT = EPT_, ROUND = NT * EPT_;   // the history is at most ROUND positions
  extern __shared__ float stage[];
  __shared__ uint32_t hist[kHistBins];
  __shared__ int32_t sh_pos[kInlineGatherRows];
  __shared__ uint32_t sh_scan[NT / 64];
  __shared__ uint32_t res[4];                      // [0], [1]: digit search and ranking results; [2], [3]: list lengths, in turn
  __shared__ uint32_t sh_mm[2 * (NT / 64)];

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // Slices (slice_log2 > 0): the workgroups beyond the segments select once more for a segment that keeps more than a slice,
  // each to write and copy the next 2^slice_log2 of its rows.
  int seg = blockIdx.x, slice = 0;
  if (seg >= tab.nseg) {
    int more = seg - tab.nseg;
    for (int s0 = 0; s0 < tab.nseg; s0 += 64) {
      const int s = min(s0 + lane, tab.nseg - 1), rows = s0 + lane < tab.nseg ? tab.out_off(s + 1) - tab.out_off(s) : 0;
      const int extra = max(rows - 1, 0) >> slice_log2, incl = (int)wave_incl_scan((uint32_t)extra);
      const unsigned long long past = __builtin_amdgcn_ballot_w64(incl > more);
      if (past) {
        const int l = __builtin_ctzll(past);
        seg = s0 + l;
        slice = 1 + more - __builtin_amdgcn_readlane(incl - extra, l);
        break;
      }
      more -= __builtin_amdgcn_readlane(incl, 63);
    }
    if (!slice) return;
  }
  const SegShape sg = tab.shape(seg);
  const int n = sg.n;
  const int kk = sg.kk;
  const int m = n - w;
  const int seg_kept = tab.out_off(seg + 1) - tab.out_off(seg);
  const int first = slice << slice_log2, kept = slice_log2 ? min(seg_kept - first, 1 << slice_log2) : seg_kept;   // this workgroup's part of them
  const int64_t row0 = tab.out_off(seg) + first;
  const bool small_seg = kept <= kInlineGatherRows;
  int32_t* out = kept_idx + row0;
  if (slice == 0 && tid == 0) {
    if (d_out_offsets) {
      d_out_offsets[seg] = tab.out_off(seg);
      if (seg == tab.nseg - 1) d_out_offsets[seg + 1] = tab.out_off(tab.nseg);
    }
    if (meet) __hip_atomic_store(meet + (int64_t)seg * kMeetWords, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  auto emit = [&](int pos, int j) __attribute__((always_inline)) {   // kept position j goes to output slot pos of the segment
    const int p = pos - first;
    if ((uint32_t)p < (uint32_t)kept) {
      out[p] = j;
      if (small_seg) sh_pos[p] = j;
    }
  };
  SLKV_STAMP(128 + seg, 0);
  if (small_seg)
    for (int i = tid; i < kInlineGatherRows; i += NT) sh_pos[i] = 0;
  __syncthreads();
  // The observation window is kept whatever the scores say: where this workgroup also copies its rows
  // and the window is one 16-byte piece per thread at most, the pieces are
  // fetched right behind the scores and stored at the end, off the critical path.
  const int lpr = ga.lanes_per_row;
  const int win0 = kk - first;                                   // the window's place among this workgroup's rows
  const bool win_early = small_seg && w * lpr <= NT && win0 >= 0 && win0 + w <= kept;
  const bool win_mine = win_early && tid < w * lpr;
  const int win_piece = min(tid, max(w * lpr - 1, 0));           // (threads past the window's pieces fetch its last one again: a load
  const int win_row = win_piece / lpr, win_c = win_piece % lpr;  //  under a condition would have to be waited for where the branches meet)
  u32x4 win_k, win_v;
  const bool ranked = kk > 0 && kk < m;
  if (!ranked) {
    if (kk < 0) {
      for (int j = tid; j < n; j += NT) emit(j, j);
    } else {
      for (int j = tid; j < w; j += NT) emit(j, m + j);   // kk == 0: the window alone
    }
  }
  if (ranked) {
  const float* I = imp + sg.score_off;
  float* P = pooled + sg.score_off;
  if (slice) write_pooled = 0;
  const int radius = RADIUS >= 0 ? RADIUS : pool_kernel / 2;
  auto fetch_window = [&]() __attribute__((always_inline)) {
    const int64_t tok = (int64_t)sg.tok_begin + m + win_row, h = sg.head;
    win_k = *reinterpret_cast<const u32x4*>(ga.k + (h * ga.k_stride_head + tok * ga.k_stride_tok) * ga.elt_bytes + win_c * 16);
    win_v = *reinterpret_cast<const u32x4*>(ga.v + (h * ga.v_stride_head + tok * ga.v_stride_tok) * ga.elt_bytes + win_c * 16);
  };

  // Window maxima (or no pooling), with the largest score of every group of 8 positions at hand: the k-th largest pooled score is found, and the kept
  // positions written, from the few positions whose own score reaches a bound below it.
  //   A score reaches the windows of min(radius + 1, 8) positions at least, of which no two groups' largest scores share more than
  //   `slack` in all, so `need` groups whose largest score is >= L put the k-th largest pooled score at or above L.
  //   Of the groups with a score >= L the scores >= L are listed in position order (others lie below every kept score).  The largest score
  //   of a window (of equal ones the first) owns its position; the positions that a score owns are neighbours: right of the next score
  //   before it that is at least as large, by more than the radius, left of the next one after it that is larger.
  //   The k-th largest pooled score is then that of the listed scores, each counted as often as it owns a position.
  // Returns false, in all threads, where the lists would not hold them; the positions are then ranked one by one below.
  // 8 segments of 32704 positions, k from 43 to 1770: 15.3 -> 9 us (the call 68.2 -> 61.9); the passes over 32 positions a thread are what it saves.
  auto select_by_groups = [&]() -> bool {
    if (!gm) return false;
    constexpr int kMostGroups = NT, kMostScores = 4 * NT;
    const int cover = min(radius + 1, kGroup), slack = min(radius, kGroup - 1), need = (kk + slack + cover - 1) / cover;
    const int ngroups = (m + kGroup - 1) / kGroup;
    if (need > min(ngroups, kMostGroups) || ngroups > 4 * NT) return false;
    uint32_t* const base = reinterpret_cast<uint32_t*>(stage);
    uint32_t* const glist = base;                              // groups, in order
    int32_t* const spos = (int32_t*)(base + kMostGroups);      // listed scores: position,
    uint32_t* const skey = base + kMostGroups + kMostScores;   // key
    uint32_t* const dhist = base + kMostGroups + 2 * kMostScores;   // of the positions owned, per digit; and the
    uint32_t* const dmax = dhist + kHistBins;                  // largest and
    uint32_t* const dmin = dmax + kHistBins;                   // smallest key of every digit
    static_assert(kMostGroups + 2 * kMostScores + 3 * kHistBins <= (int)(kResLdsBytes / sizeof(uint32_t)), "the lists fit the staging area");
    constexpr int kShift = 17;                                 // 64 bins per octave from 2^-21 on
    constexpr uint32_t kFirst = 106u << (23 - kShift);
    auto bin = [&](uint32_t u) { return (u >> kShift) <= kFirst ? 0u : min((u >> kShift) - kFirst, (uint32_t)kHistBins - 1u); };
    uint32_t gk[4];
    const uint32_t* const G = gm + group_off(sg.score_off, seg);
#pragma unroll
    for (int c = 0; c < 4; ++c) gk[c] = G[min(4 * tid + c, ngroups - 1)];
    for (int i = tid; i < kHistBins; i += NT) {
      hist[i] = 0;
      dhist[i] = 0;
      dmax[i] = 0;
      dmin[i] = 0xffffffffu;
    }
    if (tid == 0) res[2] = 0;
    __syncthreads();
    uint32_t top = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (4 * tid + c >= ngroups) gk[c] = 0;
      else atomicAdd(&hist[bin(gk[c])], 1u);
      top = max(top, gk[c]);
    }
    top = wave_reduce_to_last(top, [](uint32_t a, uint32_t b) { return max(a, b); });
    if (lane == 63) atomicMax(&res[2], top);
    __syncthreads();
    select_bin<NT>(hist, (uint32_t)need, sh_scan, res);
    const uint32_t b = res[0], kmax = res[2];
    if (b == 0u) return false;
    const uint32_t L = (b + kFirst) << kShift;
    // the groups that reach L
    uint32_t cnt = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) cnt += gk[c] >= L ? 1u : 0u;
    uint32_t at = block_incl_scan<NT>(cnt, sh_scan);
    if (tid == NT - 1) res[3] = at;
    at -= cnt;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (gk[c] >= L) {
        if (at < (uint32_t)kMostGroups) glist[at] = (uint32_t)(4 * tid + c);
        ++at;
      }
    __syncthreads();
    const uint32_t ng = res[3];
    if (ng > (uint32_t)kMostGroups) return false;
    // their scores that do
    uint32_t u[kGroup];
    cnt = 0;
    int p0 = 0;
    if (tid < (int)ng) {
      p0 = (int)glist[tid] * kGroup;
      float v[kGroup];
#pragma unroll
      for (int e = 0; e < kGroup; ++e) v[e] = I[min(p0 + e, m - 1)];
#pragma unroll
      for (int e = 0; e < kGroup; ++e) {
        u[e] = p0 + e < m ? score_key(v[e]) : 0u;
        cnt += u[e] >= L ? 1u : 0u;
      }
    }
    fetch_window();                                            // (behind the last loads that somebody waits for before the end)
    at = block_incl_scan<NT>(cnt, sh_scan);
    if (tid == NT - 1) res[3] = at;                            // (read by all before the barriers of the scan above)
    at -= cnt;
    if (tid < (int)ng) {
#pragma unroll
      for (int e = 0; e < kGroup; ++e)
        if (u[e] >= L) {
          if (at < (uint32_t)kMostScores) {
            spos[at] = p0 + e;
            skey[at] = u[e];
          }
          ++at;
        }
    }
    __syncthreads();
    const int ns = (int)res[3];
    if (ns > kMostScores) return false;
    // what each score owns: `per` consecutive ones per thread
    const int per = (ns + NT - 1) / NT;
    int from[4], own[4];
    uint32_t sk[4];
    const uint32_t span0 = kmax - L;
    auto shift_of = [](uint32_t span) {
      const int nbits = span ? 32 - __clz(span) : 0;
      return nbits > 11 ? nbits - 11 : 0;
    };
    int shift = shift_of(span0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = tid * per + c;
      own[c] = 0;
      sk[c] = 0;
      if (c < per && i < ns) {
        const int p = spos[i];
        const uint32_t k0 = skey[i];
        int lo = max(p - radius, 0), hi = min(p + radius, m - 1);
        for (int q = i - 1; q >= 0 && spos[q] >= p - 2 * radius; --q)
          if (skey[q] >= k0) {
            lo = max(lo, spos[q] + radius + 1);
            break;
          }
        for (int q = i + 1; q < ns && spos[q] <= p + 2 * radius; ++q)
          if (skey[q] > k0) {
            hi = min(hi, spos[q] - radius - 1);
            break;
          }
        from[c] = lo;
        own[c] = max(hi - lo + 1, 0);
        sk[c] = k0;
        if (own[c]) {
          const uint32_t d = (k0 - L) >> shift;
          atomicAdd(&dhist[d], (uint32_t)own[c]);
          atomicMax(&dmax[d], k0);
          atomicMin(&dmin[d], k0);
        }
      }
    }
    // the k-th largest, 11 bits of the range at a time; as a rule the first digit holds one score
    uint32_t lo = L, hi = kmax, k = (uint32_t)kk;
    for (;;) {
      __syncthreads();
      select_bin<NT>(dhist, k, sh_scan, res);
      const uint32_t d = res[0], big = dmax[d], small = dmin[d];
      k = res[1];
      lo += d << shift;
      hi = min(hi, lo + ((1u << shift) - 1u));
      if (big == small || shift == 0) {
        lo = big;
        break;
      }
      shift = shift_of(hi - lo);
      __syncthreads();                                         // every thread has read the digit's keys
      for (int i = tid; i < kHistBins; i += NT) {
        dhist[i] = 0;
        dmax[i] = 0;
        dmin[i] = 0xffffffffu;
      }
      __syncthreads();
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (own[c] && sk[c] >= lo && sk[c] <= hi) {
          const uint32_t dd = (sk[c] - lo) >> shift;
          atomicAdd(&dhist[dd], (uint32_t)own[c]);
          atomicMax(&dmax[dd], sk[c]);
          atomicMin(&dmin[dd], sk[c]);
        }
    }
    // kept positions in order: slot = (#greater before) + min(#equal before, wanted)
    uint32_t packed = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) packed += own[c] && sk[c] >= lo ? (uint32_t)own[c] << (sk[c] > lo ? 0 : 16) : 0u;
    const uint32_t excl = block_incl_scan<NT, false>(packed, sh_scan) - packed;
    uint32_t greater = excl & 0xffffu, equal = excl >> 16;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (own[c] && sk[c] >= lo) {
        int take = own[c];
        if (sk[c] == lo) take = equal < k ? min(take, (int)(k - equal)) : 0;
        const int slot = (int)(greater + min(equal, k));
        for (int e = 0; e < take; ++e) emit(slot + e, from[c] + e);
        if (sk[c] > lo) greater += (uint32_t)own[c];
        else equal += (uint32_t)own[c];
      }
    return true;
  };
  const bool is_max = pool_mode != SLKV_POOL_AVG;
  const float fill = 0.f;                          // scores are >= 0, so zero padding leaves window maxima as they are
  const float inv_p = 1.f / (float)pool_kernel;

  bool selected = false;
  if constexpr (EPT > kSelEPTMid) selected = select_by_groups();
  if (!selected) {
  // Keys: bit patterns of the pooled scores (>= 0, so monotone as unsigned integers); positions
  // past the end of the history get a key above every score.
  uint32_t key[EPT];
  const int j0 = EPT * tid;

  // keys of the pooled scores from the importance array.  Window maxima are taken on the keys
  // themselves (integer maxima, three operands at a time); averages in floating point.
  auto pool_all = [&]() {
    const int base = 0;
    // all loads first (clamped addresses, so none depends on a branch), then the LDS writes
    float ld[EPT + 1];
#pragma unroll
    for (int c = 0; c <= EPT; ++c) {
      const int j = base - radius + (c < EPT ? c * NT + tid : ROUND + min(tid, 2 * radius));
      ld[c] = I[min(max(j, 0), m - 1)];
    }
#pragma unroll
    for (int c = 0; c < EPT; ++c) {
      const int s = c * NT + tid, j = base - radius + s;
      stage[pad_idx<EPT>(s)] = (j >= 0 && j < m) ? ld[c] : fill;
    }
    if (tid < 2 * radius) {
      const int s = ROUND + tid, j = base - radius + s;
      stage[pad_idx<EPT>(s)] = (j >= 0 && j < m) ? ld[EPT] : fill;
    }
    __syncthreads();
    fetch_window();                                // (behind the barrier: every score has arrived, and nothing waits for these loads before the end)
    if (RADIUS >= 0) {
      constexpr int RR = RADIUS >= 0 ? RADIUS : 0;
      float v[EPT + 2 * RR];
#pragma unroll
      for (int e = 0; e < EPT + 2 * RR; ++e) v[e] = stage[pad_idx<EPT>(EPT * tid + e)];
      if (is_max) {
        uint32_t kv[EPT + 2 * RR], t3[EPT + 3];
#pragma unroll
        for (int e = 0; e < EPT + 2 * RR; ++e) kv[e] = score_key(v[e]);
        if (RR >= 2) {
#pragma unroll
          for (int e = 0; e < EPT + RR; ++e) t3[e] = max(max(kv[e], kv[e + 1]), kv[e + 2]);   // RR == 2 reads t3 up to EPT + 1, RR == 3 up to EPT + 2
        }
#pragma unroll
        for (int e = 0; e < EPT; ++e)
          key[e] = RR == 0 ? kv[e] : RR == 1 ? max(max(kv[e], kv[e + 1]), kv[e + 2]) : RR == 2 ? max(t3[e], t3[e + 2]) : max(max(t3[e], t3[e + 3]), kv[e + 6]);
      } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          float a = v[e];
#pragma unroll
          for (int t = 1; t <= 2 * RR; ++t) a += v[e + t];
          key[e] = score_key(a * inv_p);
        }
      }
    } else {
#pragma unroll 1
      for (int e = 0; e < EPT; ++e) {
        float a = stage[pad_idx<EPT>(EPT * tid + e)];
        for (int t = 1; t <= 2 * radius; ++t) {
          const float x = stage[pad_idx<EPT>(EPT * tid + e + t)];
          a = is_max ? fmaxf(a, x) : a + x;
        }
        key[e] = score_key(is_max ? a : a * inv_p);
      }
    }
    __syncthreads();
  };

  // pass 1: keys of the pooled scores, the largest key of each group of GS consecutive positions
  // (NQ groups per thread), the range of the keys over the segment, and (if asked) the pooled array
  constexpr int NQ = EPT < 4 ? EPT : 4, GS = EPT / NQ;
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  uint32_t gmax[NQ];
  pool_all();
  SLKV_STAMP(128 + seg, 1);
#pragma unroll
  for (int q = 0; q < NQ; ++q) gmax[q] = 0u;
  if (j0 + EPT <= m) {                             // every thread but the last ones with positions
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      kmin = min(kmin, key[e]);
      gmax[e / GS] = max(gmax[e / GS], key[e]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      if (j0 + e < m) {
        kmin = min(kmin, key[e]);
        gmax[e / GS] = max(gmax[e / GS], key[e]);
      } else {
        key[e] = kKeyNone;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) kmax = max(kmax, gmax[q]);
  if (write_pooled) {
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (j0 + e < m) P[j0 + e] = __uint_as_float(key[e]);
  }
  kmin = wave_reduce_to_last(kmin, [](uint32_t a, uint32_t b) { return min(a, b); });
  kmax = wave_reduce_to_last(kmax, [](uint32_t a, uint32_t b) { return max(a, b); });
  if (lane == 63) {
    sh_mm[wv] = kmin;
    sh_mm[NT / 64 + wv] = kmax;
  }
  // histograms for the levels below, cleared here under the same barrier; the second one and the
  // digits' largest and smallest keys live at the start of the staging array, which is free now
  uint32_t* const aux_hist = reinterpret_cast<uint32_t*>(stage);
  uint32_t* const aux_max = aux_hist + kHistBins;
  uint32_t* const aux_min = aux_max + kHistBins;
  for (int i = tid; i < kHistBins; i += NT) {
    hist[i] = 0;
    aux_hist[i] = 0;
    aux_max[i] = 0;
    aux_min[i] = 0xffffffffu;
  }
  if (tid == 0) res[2] = 0;                        // counter of the first list (see below)
  __syncthreads();
  kmin = sh_mm[0];
  kmax = sh_mm[NT / 64];
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) {
    kmin = min(kmin, sh_mm[i]);
    kmax = max(kmax, sh_mm[NT / 64 + i]);
  }

  SLKV_STAMP(128 + seg, 2);
  // The k-th largest key: radix select on (key - lo) >> shift with 11-bit digits taken relative to
  // the range [lo, hi] still in question.  After a digit search the keys of the chosen digit are
  // copied to a list in LDS (two areas in turn), the next level histograms that list, and a list of
  // at most kSelRankMax keys is ranked by direct counting.
  // Where at least k groups hold positions, two shortcuts come first.  The k-th largest of the
  // groups' maxima bounds the k-th largest key from below: its digit is found from a histogram of
  // one key per group, and the first level over all keys then counts only those from that digit's
  // lower edge upwards (a few times k, as a rule), in finer digits.  That level also keeps the
  // largest and smallest key of every digit: if the chosen digit holds one value only (with max
  // pooling a run of equal scores, as a rule), or its largest key is the one wanted, the search
  // ends there.
  uint32_t lo = kmin, hi = kmax, k = (uint32_t)kk;
  auto list_at = [&](int i) { return reinterpret_cast<uint32_t*>(stage) + (i ? kResStageFloats : kResAuxWords); };
  auto list_cap = [](int i) { return (uint32_t)(i ? kResCandidates : kSelRound - kResAuxWords); };
  int cur = -1;                                    // the list that holds the candidates; -1: the keys in registers
  uint32_t nlist = 0;
  int ncollect = 0;                                // lists made so far; list i counts its entries in res[2 + (i & 1)]
  bool hist_clean = true, unsynced = false;        // unsynced: results of a digit search read, no barrier since
  bool pending = false;                            // a digit has been chosen whose keys are not listed yet
  bool found = false;
  uint32_t cnt_sel = 0;
  const bool full = j0 + EPT <= m;                 // this thread holds no key of a position past the end
  auto shift_of = [](uint32_t span) {
    const int nbits = span ? 32 - __clz(span) : 0;
    return nbits > 11 ? nbits - 11 : 0;
  };
  // a list is made between two barriers: the counter of the one after it is cleared meanwhile
  auto begin_list = [&]() {
    if (tid == 0) res[2 + ((ncollect + 1) & 1)] = 0;
  };
  auto push = [&](int dst, uint32_t kv) __attribute__((always_inline)) {
    const uint32_t slot = atomicAdd(&res[2 + (ncollect & 1)], 1u);
    if (slot < list_cap(dst)) list_at(dst)[slot] = kv;
  };
  auto end_list = [&](int dst) {
    __syncthreads();
    nlist = min(res[2 + (ncollect & 1)], list_cap(dst));
    ++ncollect;
    cur = dst;
    unsynced = false;
  };
  // Histogram step for segments with piles of equal keys (thousands of LDS atomics on one address
  // would serialise): the lanes of the wave whose key equals that of the first counted lane are
  // added by that lane in one atomic, likewise those equal to the first counted lane left over;
  // the other counted lanes add themselves.
  bool ties = false;
  auto count_pile = [&](bool in, uint32_t kv, uint32_t d, uint32_t* h, bool with_range) __attribute__((always_inline)) {
    const unsigned long long act = __builtin_amdgcn_ballot_w64(in);
    if (act) {                                     // (the same for the whole wave, like `rest` below)
      const int first = __builtin_ctzll(act);
      const bool same = in && kv == (uint32_t)__builtin_amdgcn_readlane((int)kv, first);
      const unsigned long long sm = __builtin_amdgcn_ballot_w64(same);
      bool mine = in;
      uint32_t add = 1u;
      if (same) {
        mine = lane == first;
        add = (uint32_t)__popcll(sm);
      }
      const unsigned long long rest = act & ~sm;
      if (rest) {
        const int second = __builtin_ctzll(rest);
        const bool same2 = in && kv == (uint32_t)__builtin_amdgcn_readlane((int)kv, second);
        if (same2) {
          mine = lane == second;
          add = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(same2));
        }
      }
      if (mine) {
        atomicAdd(&h[d], add);
        if (with_range) {
          atomicMax(&aux_max[d], kv);
          atomicMin(&aux_min[d], kv);
        }
      }
    }
  };
  const uint32_t groups = (uint32_t)((m + GS - 1) / GS);     // groups that hold at least one position
  if (k <= groups) {
    {
      const int shift = shift_of(hi - lo);
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (j0 + q * GS < m) atomicAdd(&hist[(gmax[q] - lo) >> shift], 1u);
      __syncthreads();
      SLKV_STAMP(128 + seg, 3);
      select_bin<NT>(hist, k, sh_scan, res);
      SLKV_STAMP(128 + seg, 4);
      ties = hist[res[0]] >= (uint32_t)kSelTieGroups;   // many groups share one digit: expect piles of equal keys
      lo += res[0] << shift;                       // k groups hold a key >= lo, so the k-th largest key is >= lo
      hist_clean = false;
    }
    const uint32_t span1 = hi - lo;
    const int shift = shift_of(span1);
    if (span1 == 0u) {
      found = true;                                // k groups or more hold the largest key (all scores equal, for one): it is the threshold
    } else {
    const bool track = ties || k <= (uint32_t)kSelTrackMax;   // (with many keys wanted the two extra atomics per counted key cost more than they save)
    if (ties) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t dk = key[e] - lo;
        count_pile(dk <= span1, key[e], dk >> shift, aux_hist, true);
      }
    } else if (track) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t dk = key[e] - lo;             // (a key below lo wraps to a difference above any span)
        if (dk <= span1) {
          const uint32_t d = dk >> shift;
          atomicAdd(&aux_hist[d], 1u);
          atomicMax(&aux_max[d], key[e]);
          atomicMin(&aux_min[d], key[e]);
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t dk = key[e] - lo;
        if (dk <= span1) atomicAdd(&aux_hist[dk >> shift], 1u);
      }
    }
    __syncthreads();
    select_bin<NT>(aux_hist, k, sh_scan, res);
    const uint32_t bsel = res[0];
    const uint32_t top = aux_max[bsel], bottom = aux_min[bsel];
    cnt_sel = aux_hist[bsel];
    k = res[1];
    unsynced = true;
    lo = lo + (bsel << shift);
    hi = min(hi, lo + ((1u << shift) - 1u));
    if (track && (top == bottom || k == 1u)) {
      lo = top;                                    // one value in the digit, or the largest of the digit is wanted
      found = true;
    } else if (shift == 0) {
      found = true;                                // the digit is the key
    } else {
      pending = true;
    }
    }
  }
  while (!found) {
    if (pending) {
      // the keys of the chosen digit go to the other list (their order does not matter for counting)
      pending = false;
      const int dst = cur == 0 ? 1 : 0;
      if (cnt_sel <= (cur >= 0 ? list_cap(dst) : (uint32_t)kResCandidates)) {   // (from registers every copied key costs an LDS atomic with its latency)
        begin_list();
        const uint32_t span2 = hi - lo;
        if (cur >= 0) {
          const uint32_t* cand = list_at(cur);
          for (uint32_t i = tid; i < nlist; i += NT) {
            const uint32_t kv = cand[i];
            if (kv - lo <= span2) push(dst, kv);
          }
        } else {
#pragma unroll
          for (int e = 0; e < EPT; ++e)
            if (key[e] - lo <= span2) push(dst, key[e]);
        }
        end_list(dst);
      }
    }
    const uint32_t span1 = hi - lo;
    const int shift = shift_of(span1);
    if (cur >= 0 && nlist <= (uint32_t)kSelRankMax) {
      // short list: the k-th largest by counting, for each entry, the entries above it (four
      // entries a step; both list areas are longer than any index read here)
      const uint32_t* cand = list_at(cur);
      if ((uint32_t)tid < nlist) {
        const uint32_t kv = cand[tid];
        uint32_t gt = 0, ge = 0;
        for (uint32_t i = 0; i < nlist; i += 4) {
#pragma unroll
          for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t o = cand[i + u];
            const bool live = i + u < nlist;
            gt += (live && o > kv) ? 1u : 0u;
            ge += (live && o >= kv) ? 1u : 0u;
          }
        }
        if (gt < k && k <= ge) {   // every thread holding the k-th largest value writes the same pair
          res[0] = kv;
          res[1] = k - gt;
        }
      }
      __syncthreads();
      lo = res[0];
      k = res[1];
      break;
    }
    if (!hist_clean) {
      if (unsynced) __syncthreads();               // every thread has read the counts and results of the level before
      for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
      __syncthreads();
    }
    if (cur >= 0) {
      const uint32_t* cand = list_at(cur);
      for (uint32_t i = tid; i < nlist; i += NT) {
        const uint32_t dk = cand[i] - lo;
        if (dk <= span1) atomicAdd(&hist[dk >> shift], 1u);
      }
    } else if (ties) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t dk = key[e] - lo;
        count_pile(dk <= span1, key[e], dk >> shift, hist, false);
      }
    } else if (hist_clean && full) {
      // lo and hi are the smallest and largest key of the segment: nothing to test
#pragma unroll
      for (int e = 0; e < EPT; ++e) atomicAdd(&hist[(key[e] - lo) >> shift], 1u);
    } else {
      // in [lo, hi] <=> key - lo <= hi - lo: a key below lo wraps to a difference above any span,
      // and kKeyNone lies above every hi
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t dk = key[e] - lo;
        if (dk <= span1) atomicAdd(&hist[dk >> shift], 1u);
      }
    }
    __syncthreads();
    if (hist_clean) SLKV_STAMP(128 + seg, 3);
    select_bin<NT>(hist, k, sh_scan, res);
    if (hist_clean) SLKV_STAMP(128 + seg, 4);
    const uint32_t bsel = res[0];
    cnt_sel = hist[bsel];
    k = res[1];
    hist_clean = false;
    unsynced = true;
    lo = lo + (bsel << shift);
    hi = min(hi, lo + ((1u << shift) - 1u));
    if (shift == 0) break;
    pending = true;
  }
  const uint32_t tau = lo, need_eq = k;
  SLKV_STAMP(128 + seg, 5);

  // ordered compaction: slot = (#greater before) + min(#equal before, need_eq)
  {
    uint32_t gmask = 0, emask = 0;                 // bit e: element e is above / equal to the threshold
    const uint32_t upto = kKeyNone - tau;           // tau <= key < kKeyNone <=> key - tau < upto
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const uint32_t dk = key[e] - tau;
      const bool in = dk < upto;
      if (__builtin_amdgcn_ballot_w64(in)) {        // few positions are kept: most waves skip most steps
        gmask |= (in && dk != 0u) ? (1u << e) : 0u;
        emask |= dk == 0u ? (1u << e) : 0u;
      }
    }
    const uint32_t cg = __popc(gmask), ce = __popc(emask);
    const uint32_t packed = (ce << 16) | cg;       // the round holds at most 32768 of either
    const uint32_t incl = block_incl_scan<NT, false>(packed, sh_scan);   // sh_scan is not used again
    const uint32_t excl = incl - packed;
    const uint32_t g_before = excl & 0xffffu, e_before = excl >> 16;
    // ties are taken in position order: this thread keeps its first `take` equal elements
    uint32_t take = 0;
    if (e_before < need_eq) take = (need_eq - e_before) < ce ? (need_eq - e_before) : ce;
    uint32_t sel = gmask;
    for (uint32_t em = emask; take > 0; --take) {
      sel |= em & (0u - em);                       // lowest set bit
      em &= em - 1u;
    }
    uint32_t pos = g_before + (e_before < need_eq ? e_before : need_eq);
    while (sel) {
      const int e = __ffs(sel) - 1;
      emit((int)pos++, j0 + e);
      sel &= sel - 1u;
    }
  }
  }  // by the scores of all positions
  for (int j = tid; j < w; j += NT) emit(kk + j, m + j);
  SLKV_STAMP(128 + seg, 6);
  }  // ranked

  // Small segments copy their K/V rows here (saves the gather launch); larger ones are left
  // to gather_kernel, which skips the segments handled here.  Four pieces per thread are in
  // flight at a time.
  if (kept > 0 && small_seg) {
    __syncthreads();                                // sh_pos is complete
    const int64_t tok0 = sg.tok_begin, h = sg.head;
    const bool win_done = ranked && win_early;      // the window's pieces are in registers
    const int pieces = (win_done ? win0 : kept) * lpr;
    const uint32_t magic = 0xffffffffu / (uint32_t)lpr + 1u;   // idx / lpr == umulhi(idx, magic) for idx < 2^16 (lpr > 1)
    struct Piece {
      u32x4 kq, vq;
      int row, c;
      int64_t tok;
    };
    auto fetch = [&](int idx, Piece& q) __attribute__((always_inline)) {
      q.row = lpr == 1 ? idx : (int)__umulhi((uint32_t)idx, magic);
      q.c = idx - q.row * lpr;
      if (idx < pieces) {
        q.tok = tok0 + sh_pos[q.row];
        q.kq = *reinterpret_cast<const u32x4*>(ga.k + (h * ga.k_stride_head + q.tok * ga.k_stride_tok) * ga.elt_bytes + q.c * 16);
        q.vq = *reinterpret_cast<const u32x4*>(ga.v + (h * ga.v_stride_head + q.tok * ga.v_stride_tok) * ga.elt_bytes + q.c * 16);
      }
    };
    auto put = [&](int idx, const Piece& q) __attribute__((always_inline)) {
      if (idx < pieces) {
        const int64_t o = ((row0 + q.row) * lpr + q.c) * 16;
        *reinterpret_cast<u32x4*>(ga.k_out + o) = q.kq;
        *reinterpret_cast<u32x4*>(ga.v_out + o) = q.vq;
        if (ga.pos_out && q.c == 0) ga.pos_out[row0 + q.row] = ga.pos_in[q.tok];
      }
    };
    for (int base = tid; base < pieces; base += 4 * NT) {
      Piece q0, q1, q2, q3;
      fetch(base, q0);
      fetch(base + NT, q1);
      fetch(base + 2 * NT, q2);
      fetch(base + 3 * NT, q3);
      put(base, q0);
      put(base + NT, q1);
      put(base + 2 * NT, q2);
      put(base + 3 * NT, q3);
    }
    if (win_done && win_mine) {
      const int64_t o = ((row0 + win0 + win_row) * lpr + win_c) * 16;
      *reinterpret_cast<u32x4*>(ga.k_out + o) = win_k;
      *reinterpret_cast<u32x4*>(ga.v_out + o) = win_v;
      if (ga.pos_out && win_c == 0) ga.pos_out[row0 + win0 + win_row] = ga.pos_in[tok0 + m + win_row];
    }
  }
  SLKV_STAMP(128 + seg, 7);
}

// Copies kept rows of K and V (bit copies) into the packed output; one 16-byte lane per piece.
// Bound by HBM, after a chain of three loads (segment, kept position, row); the segment is looked up once per workgroup.
// A call with more pieces than the chip has threads (kGatherThreads) gives each thread PIECES = 4, so that as many rows are in
// flight at the end of one chain: re-compression of 256 segments, 64 K rows, 70.4 -> 68.0 us a call.  With fewer, 4 pieces a
// thread only leave CUs idle (16 short prompts: 54.2 -> 58.5 us).
constexpr int64_t kGatherThreads = 256 * 2048;
template <int PIECES, class TAB>
__global__ __launch_bounds__(256) void gather_kernel(const TAB tab, const GatherArgs ga,
                                                     const int32_t* __restrict__ kept_idx, int all_segments) {
  const int shift = __builtin_ctz(ga.lanes_per_row);                  // 4 to 32 lanes per row: a power of two
  const int64_t first = (int64_t)blockIdx.x * (256 * PIECES);
  const int c = (int)threadIdx.x & (ga.lanes_per_row - 1);
  const int row0 = tab.out_off(0), row1 = tab.out_off(tab.nseg);
  // the segment of the workgroup's first row, and where the next three begin
  const int seg0 = find_segment_wave(tab.nseg, min(row0 + (int)(first >> shift), row1 - 1), [&](int s) { return tab.out_off(s); });
  int next[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) next[i] = tab.out_off(min(seg0 + 1 + i, tab.nseg));
  int64_t row[PIECES], tok[PIECES], head[PIECES];
  bool copy[PIECES];
  u32x4 kv[PIECES], vv[PIECES];
#pragma unroll
  for (int u = 0; u < PIECES; ++u) {
    row[u] = row0 + ((first + u * 256 + threadIdx.x) >> shift);
    copy[u] = row[u] < row1;
    const int r = (int)min(row[u], (int64_t)row1 - 1);
    int seg = seg0;
#pragma unroll
    for (int i = 0; i < 3; ++i) seg += r >= next[i] ? 1 : 0;
    while (r >= next[2] && tab.out_off(seg + 1) <= r) ++seg;
    if (!all_segments && tab.out_off(seg + 1) - tab.out_off(seg) <= kInlineGatherRows) copy[u] = false;   // done by the selection kernel
    // (a position outside the segment cannot come out of the selection; clamped all the same, so
    // that no input can turn into an out-of-bounds read here)
    const SegShape sg = tab.shape(seg);
    const int kept = copy[u] ? kept_idx[r] : 0;
    tok[u] = (int64_t)sg.tok_begin + min(max(kept, 0), max(sg.n - 1, 0));
    head[u] = sg.head;
  }
#pragma unroll
  for (int u = 0; u < PIECES; ++u)
    if (copy[u]) {
      kv[u] = *reinterpret_cast<const u32x4*>(ga.k + (head[u] * ga.k_stride_head + tok[u] * ga.k_stride_tok) * ga.elt_bytes + c * 16);
      vv[u] = *reinterpret_cast<const u32x4*>(ga.v + (head[u] * ga.v_stride_head + tok[u] * ga.v_stride_tok) * ga.elt_bytes + c * 16);
    } else {
      kv[u] = vv[u] = u32x4{0, 0, 0, 0};
    }
#pragma unroll
  for (int u = 0; u < PIECES; ++u)
    if (copy[u]) {
      const int64_t o = (row[u] * ga.lanes_per_row + c) * 16;
      *reinterpret_cast<u32x4*>(ga.k_out + o) = kv[u];
      *reinterpret_cast<u32x4*>(ga.v_out + o) = vv[u];
      if (ga.pos_out && c == 0) ga.pos_out[row[u]] = ga.pos_in[tok[u]];
    }
}

// Words of a segment table that does not fit a kernel argument, on their way into the workspace.
struct UploadWords {
  int32_t w[kArgWords];
};
__global__ void upload_kernel(const UploadWords part, int count, int32_t* __restrict__ dst) {
  const int i = threadIdx.x;
  if (i < count) dst[i] = part.w[i];
}

// ------------------------------------------------------------------------------------------
// Host side: planning, validation, launches.

// One (sequence, KV head) segment as the kernels see it.
struct Seg {
  int64_t row_begin;   // first token row of the segment (multiplied by the token stride)
  int64_t n;           // rows in the segment; the last w are the window
  int64_t cap;         // capacity C of its head
  int32_t head;        // multiplied by the head stride (0 for a ragged cache)
  int64_t qrow_off;    // first row of the segment's [G*w][d] query block
  int64_t score_off;   // offset of the segment in the importance / pooled arrays
};

// What both entry points reduce to: common shape parameters plus the list of segments.
struct Geometry {
  int dtype, Hq, Hkv, d, w, pool_kernel, pool;
  bool ragged;
  const int64_t* h_begin;   // B+1 token offsets, or (ragged) one row offset per segment and the end
  const int32_t* h_caps;    // capacities of the KV heads
  int64_t k_stride_tok, k_stride_head, v_stride_tok, v_stride_head;
  int64_t score_elems;   // length of the importance / pooled arrays
  std::vector<Seg> segs;
  int64_t longest;       // ranked history (0: none)
};

struct Plan {
  int R, Rpad, CH;
  int64_t hist_blocks;   // block histograms of the selection
  int waves;             // per workgroup of the scoring passes
  int rsplit;            // of these, that share a key group's query tiles (score_k_resident_kernel)
  size_t part_bytes, score_bytes, hist_bytes, table_bytes;
  size_t off_part, off_imp, off_pooled, off_hist, off_table, total_bytes;
  int per_cu;            // workgroups of a scoring launch that a CU holds at least
  int meet_most;         // chunks of a segment up to which both scoring passes take one launch (see meet_chunks), if its workgroups fit the chip
  double passes_us;      // estimate of both scoring passes together
  bool one_scan;         // the call may go over its keys once (see OneScan), if the workspace has these bytes as well
  int sampled;           // see range_len
  int64_t ranges;
  size_t off_part0, off_dense, off_bins, off_lse, off_bounds, off_lists, one_scan_bytes;
};

static bool seg_ranked(int64_t n, int64_t w, int64_t cap) { return n > w && n > cap && cap > w; }
// key chunks of the scoring passes and blocks of the selection for one segment
static int64_t seg_chunks(const Seg& s, int w, int64_t ch) { return seg_ranked(s.n, w, s.cap) ? (s.n - w + ch - 1) / ch : 0; }
static int64_t seg_ranges(const Seg& s, int w, int sampled) {
  if (!seg_ranked(s.n, w, s.cap)) return 0;
  const int m = (int)(s.n - w), len = range_len(m, (int)(s.cap - w), sampled);
  return (m + len - 1) / len;
}
static int64_t longest_ranked(const Geometry& g) {
  int64_t longest = 0;
  for (const Seg& s : g.segs)
    if (seg_ranked(s.n, g.w, s.cap)) longest = std::max(longest, s.n - g.w);
  return longest;
}
static int64_t seg_blocks(const Seg& s, int w) { return seg_ranked(s.n, w, s.cap) ? (s.n - w + kSelBlock - 1) / kSelBlock : 0; }

// f(head dimension, KIND) of a call, as integral constants.
template <class F>
static auto with_score_kind(int d, int dtype, F f) {
  const int kind = dtype == SLKV_BF16 ? 0 : dtype == SLKV_F16 ? 1 : dtype == SLKV_BF16_KV_FP8 ? 2 : 3;
  if (d == 128) {
    switch (kind) {
      case 0: return f(std::integral_constant<int, 128>{}, std::integral_constant<int, 0>{});
      case 1: return f(std::integral_constant<int, 128>{}, std::integral_constant<int, 1>{});
      case 2: return f(std::integral_constant<int, 128>{}, std::integral_constant<int, 2>{});
      default: return f(std::integral_constant<int, 128>{}, std::integral_constant<int, 3>{});
    }
  }
  switch (kind) {
    case 0: return f(std::integral_constant<int, 64>{}, std::integral_constant<int, 0>{});
    case 1: return f(std::integral_constant<int, 64>{}, std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 64>{}, std::integral_constant<int, 2>{});
    default: return f(std::integral_constant<int, 64>{}, std::integral_constant<int, 3>{});
  }
}

// The ranked history lengths of a call (less one; equal neighbours together) and how many chunks they make: in single
// precision, which a cost allows and which adds up 512 different ones in under a microsecond (this runs for every call).
struct RankedLengths {
  std::vector<float> len;
  std::vector<int> times;
  int64_t longest, ranked = 0;
  explicit RankedLengths(const Geometry& g) : longest(std::max<int64_t>(g.longest, 1)) {
    for (const Seg& s : g.segs)
      if (seg_ranked(s.n, g.w, s.cap)) {
        const float m1 = (float)(s.n - g.w - 1);
        if (!len.empty() && len.back() == m1) {
          times.back() += 1;
        } else {
          len.push_back(m1);
          times.push_back(1);
        }
        ++ranked;
      }
  }
  int64_t chunks(int64_t ch) const {
    const float per_chunk = 1.0f / (float)ch;
    int count = 0;
    for (size_t i = 0; i < len.size(); ++i) count += times[i] * ((int)(len[i] * per_chunk) + 1);
    return count;
  }
};

// Workgroup size, chunk length and split of the query tiles of score_k_resident_kernel: what takes the least time by the
// costs below, measured over calls of 2 to 56 segments of 104 to 16 K keys.
//   kStartUs: a workgroup's start and end (queries into LDS, first keys, row statistics); kLaunchUs: from one pass to the
//   next, saved where every segment is one chunk and the first pass completes it;
//   tile: a key group against 32 query rows by a wave that has its SIMD to itself; `shared` times as long with two on it
//   (8 waves on a CU, in one workgroup of 8 waves or in two of 4 where their LDS fits twice): fp32 MFMAs fill the
//   matrix pipe alone, E4M3 keys leave gaps;
//   kFoldUs: per chunk of a segment, its statistics read back by the second pass.
// Waves that share a key group (rsplit of them take its query tiles in turn) shorten the chain of tiles of calls that
// leave most SIMDs idle; with more keys than that they only repeat loads, so rsplit > 1 means one group per wave.
// fp32: 4 heads x 1 K keys, d 64, one query tile 24.2 -> 19.7 us (groups of 32 keys instead of 64); 2 x 700, d 128, four tiles
// 36.8 -> 25.3; 8 x 2 K, d 64, two tiles 28.0 -> 20.6; E4M3: 22 segments of 104 to 878 keys, four tiles 27.2 -> 19.9; 8 x 1.5 K 22.8 -> 19.4;
// 56 segments of one chunk 27.7 -> 22.6 (no second pass); 8 x 32 K as before.
//
// Both passes in one launch (PASS 3): the queries stay in LDS, up to two groups of keys a wave in registers (the second pass then waits for no key, though it requests them again).  Two launches
// / one, us a call: E4M3 8 x 32 K 57.8 / 55.1, 16 x 32 K 90.4 / 84.2, 128 x 3 K 64.0 / 58.0, 192 x 1.7 to 9 K of 64 rows 99.1 / 84.2, 4 x 20 K of 448 rows 62.9 / 58.3,
// 8 x 2 K 21.6 / 20.5, a decode cache of 256 segments 35.3 / 34.6, of 8 22.9 / 20.3; fp32 4 x 1 K 20.6 / 19.4, 32 x 0.6 K 23.9 / 22.7.  Not with many short
// chunks to a segment, for which everybody waits and which everybody reads back: E4M3 8 x 12 K in 47 each 27.8 / 28.5; fp32 8 x 4 K in 31 29.6 / 29.8, 8 x 2 K in 32
// 31.5 / 31.7.  (Planned for, by its lower cost, one launch takes fewer, longer chunks: 8 x 8 K fp32 46.3 -> 47.5.)  Long passes gain as well, unlike those of 16-bit keys (kTogetherUs): one
// workgroup has a CU to itself.  E4M3 32 x 32 K 159 / 152, 64 x 32 K 283 / 278, six prompts of 2 to 32 K 163 / 151 (on several streams: meet_limit).
static void plan_k_resident(const Geometry& g, Plan& p) {
  constexpr double kLaunchUs = 3.7, kFoldUs = 0.03;
  const bool f32 = g.dtype == SLKV_F32;
  const double tile_us = f32 ? (g.d == 128 ? 2.1 : 1.25) : (g.d == 128 ? 0.64 : 0.4), shared = f32 ? 2.0 : 1.6;
  int gk = 0, tiles = 0, max_tiles = 0;
  size_t lds4 = 0;
  with_score_kind(g.d, g.dtype, [&](auto dk, auto kind) {
    using C = ScoreCfg<decltype(dk)::value, decltype(kind)::value>;
    gk = C::GK;
    tiles = (p.R + 31) / 32;
    max_tiles = std::min(tiles, C::RBT);
    lds4 = score_lds_bytes<decltype(dk)::value, decltype(kind)::value>(max_tiles, 4);
  });
  const RankedLengths lens(g);
  const int64_t longest = lens.longest, ranked = lens.ranked;
  double best = 0;
  p.per_cu = 1;
  p.waves = 8;
  p.rsplit = 1;
  p.CH = 8 * gk;
  for (const int waves : {4, 8}) {
    const double kStartUs = waves == 4 ? 5 : 5.75;
    for (int rs = 1; rs <= waves && (rs == 1 || (rs < 2 * tiles && tiles == max_tiles)); rs *= 2) {
      const bool pairs = waves == 4 && 2 * (lds4 + 256) <= 160 * 1024;
      const int64_t unit = (int64_t)(waves / rs) * gk, most = (longest + unit - 1) / unit;
      // chunks of gpw groups a wave; returns whether longer ones can only idle workgroups
      auto consider = [&](int64_t gpw) {
        const int64_t count = lens.chunks(gpw * unit);
        const int64_t rounds = (count + (pairs ? 511 : 255)) / (pairs ? 512 : 256);
        const double tile = tile_us * (waves == 8 || (pairs && count > 256) ? shared : 1.0);
        const double sweep = (double)(std::min(gpw, most) * ((tiles + rs - 1) / rs)) * tile;
        const double us = gpw >= most ? (double)rounds * (kStartUs + 2 * sweep)
                                      : 2 * (double)rounds * (kStartUs + sweep) + kLaunchUs + kFoldUs * (double)((longest + gpw * unit - 1) / (gpw * unit));
        // (more chunks than run at once only where the segments alone are that many: their statistics take workspace)
        if (best == 0 || (us < best && (gpw >= most || count <= 512 + ranked))) {
          best = us;
          p.waves = waves;
          p.rsplit = rs;
          p.CH = (int)(gpw * unit);
          p.per_cu = pairs ? 2 : 1;
        }
        return rounds <= 1;
      };
      if (rs > 1) {
        consider(1);
        continue;
      }
      for (int64_t gpw = 1; gpw < most && !consider(gpw); gpw += std::max<int64_t>(1, gpw / 16)) {}
      consider(most);
    }
  }
  p.meet_most = f32 ? 16 : 32;
  p.passes_us = best;
}

// Chunk length of score_q_resident_kernel: what takes the least time, by a workgroup's start and end and the time of a
// 64-key tile for one workgroup on a CU (`alone`) and for two (`paired`; above 256 query rows its registers leave room
// for one).  For 65 to 256 rows the arithmetic bounds either, two workgroups gain 10 % in the loop and pay 2 us for their
// starts: 8 x 24 K keys of 256 rows 53.5 us with 504 chunks, 50.0 with 256; 32 K 62.6 and 59.8; 64 K 113 and 113; 128 K 183 and 187.
// Up to 64 rows one workgroup's loads in flight do not keep the memory busy: 32 x 16 K keys 57.4 us with 512, 61.3 with 256.
// 448 rows, 4 x 24 K: 88 us with 376 chunks, which run in two rounds, 60.7 with 252.  What does not fit at once runs in rounds.
// Small calls take chunks down to two tiles: 8 x 2 K keys of 128 rows 22.5 us with 256 keys a chunk, 19.6 with 128.
//
// Both passes in one launch (PASS 3) up to an estimated pass time of kTogetherUs: it saves a launch, and the second start of every
// workgroup: table, queries, first keys.  Two launches / one, us a call: 1 x 1.2 K 21.7 / 18.5, 1 x 2 K 23.9 / 20.6, 1 x 8 K 25.6 / 24.2, 16 prompts
// of 150 to 5 K 56.0 / 47.7, a decode cache of 256 segments 67.7 / 60.5, 1 x 32 K of 256 rows 62.2 / 61.1, 2 x 32 K 98.0 / 94.9.  Above the
// line the start is little of it, and the two workgroups of a CU, of which one is served first, wait for each other: 3 x 32 K 138.9 / 143.4.
// On 1 to 4 streams at once, 16 short prompts 59.0 43.5 38.8 37.8 / 47.8 37.8 36.6 36.4; a decode cache of 256 segments 70.2 50.4 55.9 45.5 / 55.2 40.8 46.5 41.2; 1 x 32 K 67.3 50.9 48.2 46.3 /
// 64.9 50.6 49.1 48.4, of E4M3 keys 70.7 58.7 50.8 48.7 / 65.4 56.7 49.9 52.3.  On four streams 256 workgroups of long chunks to a call lose what waits on CUs that another call could use; the line
// stays, since such calls gain as much where fewer run at once.  (The priority of the waves, first pass over second or second over first, changes nothing.)
//
// One pass over the keys instead of two (OneScan) where a pass takes this long by the costs above: it saves a pass, less a tenth, and
// costs the sample, the histograms, the bounds and the chosen keys; where histories above 32768 positions are selected by blocks it
// saves three of that selection's launches as well.  One pass / two, us, on keys as in OneScan, and (in brackets) with 16 rows of every segment that give half
// of their weight to one key each, for which the line has to leave room: 8 x 48 K keys of 256 rows 94 / 99 (110 / 99), 8 x 64 K 103 / 115 (118 / 116), 8 x 80 K
// 112 / 132 (132 / 131), 8 x 128 K 142 / 189 (166 / 189); of 128 rows 8 x 64 K 85 / 89 (97 / 89), 8 x 96 K 94 / 113 (118 / 111), 8 x 128 K 110 / 138 (131 / 141);
// of 64 rows 8 x 96 K 88 / 100 (93 / 100), 16 x 96 K 154 / 168 (159 / 170); of 16 rows 32 x 50 K 156 / 173, 32 x 75 K 201 / 245;
// histories of at most 32768, 256 rows: 32 x 20 K 136 / 115, 32 x 32 K 177 / 170, 64 x 20 K 191 / 211 (1024 kept on average 238 / 234), 48 x 30 K 212 / 236,
// 64 x 32 K 256 / 320, of 128 rows 64 x 32 K 200 / 216.  (More than 64 segments, before the probe: 128 x 16 K 329 / 323.)
constexpr double kTogetherUs = 50;
constexpr double kOneScanUs = 50, kOneScanFewRowsUs = 40, kOneScanResidentUs = 100;
static void plan_q_resident(const Geometry& g, Plan& p) {
  const int cfg = p.R <= 64 ? 0 : p.R <= 128 ? 1 : p.R <= 256 ? 2 : 3;
  const double dim = g.d == 128 ? 1.0 : 0.6;
  const double alone = dim * (cfg == 0 ? 0.6 : cfg == 1 ? 0.6 : cfg == 2 ? 1.2 : 2.4), paired = dim * (cfg == 0 ? 0.75 : cfg == 1 ? 1.09 : 2.18);
  constexpr double kStartUs = 6;
  const double second = cfg == 0 ? 1.0 : 2.2;            // two workgroups of a CU that start together
  const RankedLengths lens(g);
  double best = 0;
  p.CH = 128;
  for (int64_t ch = 128;; ch += std::max<int64_t>(128, ch / 32 / 128 * 128)) {   // pairs of 64-key tiles
    const int64_t count = lens.chunks(ch);
    const double tiles = (double)(std::min(ch, (lens.longest + 127) / 128 * 128) / 64);
    const double one = kStartUs + tiles * alone, two = kStartUs + second + tiles * paired;
    const int64_t full = cfg == 3 ? count / 256 : count / 512, rest = cfg == 3 ? count % 256 : count % 512;
    const double us = (double)full * (cfg == 3 ? one : two) + (rest == 0 ? 0 : rest <= 256 ? one : two);
    // (more chunks than run at once only where the segments alone are that many: their statistics take workspace)
    if (best == 0 || us < best || count > 512 + lens.ranked) {
      best = us;
      p.CH = (int)ch;
    }
    if (count <= 256 || ch >= lens.longest || ch >= (1 << 16)) break;
  }
  p.waves = 4;
  p.rsplit = 1;
  p.per_cu = cfg == 3 ? 1 : 2;
  p.meet_most = best <= kTogetherUs ? kMeetMost : 0;
  p.passes_us = 2 * best;
  const double worth = lens.longest <= kSelRound ? kOneScanResidentUs : cfg == 2 ? kOneScanUs : kOneScanFewRowsUs;
  p.one_scan = best >= worth && (cfg == 2 || lens.longest > kSelRound) && p.R <= 256 && g.pool != SLKV_POOL_AVG && g.segs.size() <= (size_t)kMaxSegPerLaunch;
}

// Ranges of a call in one pass: the shortest that run at once, two workgroups on a CU, and that fold_sample reads in one round trip.
// 32 segments of 20 K to 128 K keys: 511 ranges, chosen keys 20 us; 590 shorter ones, of which the last start when the first have ended, 28 us; 504, but those
// of the short segments 6144 positions long, 24 to 55 us, by how many keys these list.  8 x 128 K: 64 ranges a segment and not 32, score_both 89 us and not 82.
static void plan_ranges(const Geometry& g, Plan& p) {
  for (const int sampled : {64, 96, 128, 192, 256, 288, 320, 384, 512}) {
    p.sampled = sampled;
    p.ranges = 0;
    int64_t most = 0;
    for (const Seg& s : g.segs) {
      const int64_t n = seg_ranges(s, g.w, sampled);
      p.ranges += n;
      most = std::max(most, n);
    }
    if (p.ranges <= 512 && most <= 32) return;
  }
}

static void make_plan(const Geometry& g, Plan& p) {
  p.one_scan = false;
  p.R = (g.Hq / g.Hkv) * g.w;
  p.Rpad = (p.R + 31) / 32 * 32;
  if (g.dtype == SLKV_BF16 || g.dtype == SLKV_F16) plan_q_resident(g, p);
  else plan_k_resident(g, p);
  const int64_t ch = p.CH;
  int64_t chunks = 0;
  p.hist_blocks = 0;
  for (const Seg& s : g.segs) {
    const int64_t nc = seg_chunks(s, g.w, ch), nb = seg_blocks(s, g.w);
    chunks += nc;
    p.hist_blocks += nb;
  }
  auto align = [](size_t x) { return (x + 255) / 256 * 256; };
  p.part_bytes = align((size_t)std::max<int64_t>(chunks, 1) * p.Rpad * sizeof(float));
  p.score_bytes = align((size_t)std::max<int64_t>(1, g.score_elems) * sizeof(float));
  p.hist_bytes = align((size_t)p.hist_blocks * kHistBins * sizeof(uint32_t));
  p.off_part = SLKV_WORKSPACE_HEADER_BYTES;
  p.off_imp = p.off_part + p.part_bytes;
  p.off_pooled = p.off_imp + p.score_bytes;
  p.off_hist = p.off_pooled + p.score_bytes;
  p.off_table = p.off_hist + p.hist_bytes;
  // device-resident segment table: only for calls with more segments than one kernel argument holds
  const size_t S = g.segs.size();
  p.table_bytes = S > (size_t)kMaxSegPerLaunch ? align((4 * S + 4 + (size_t)g.Hkv) * sizeof(int32_t)) : 0;
  p.total_bytes = p.off_table + p.table_bytes;
  p.one_scan_bytes = 0;
  p.ranges = 0;
  if (p.one_scan) {
    plan_ranges(g, p);
    p.off_part0 = p.total_bytes;
    p.off_dense = p.off_part0 + align((size_t)p.ranges * p.Rpad * sizeof(float));
    p.off_bins = p.off_dense + align(S * 2 * p.Rpad * sizeof(float));
    p.off_lse = p.off_bins + S * kHists * kHistBins * sizeof(uint32_t);
    p.off_bounds = p.off_lse + S * 512 * sizeof(float);
    p.off_lists = p.off_bounds + align(S * kBoundWords * sizeof(uint32_t));
    p.one_scan_bytes = p.off_lists + S * kSelCandidates * sizeof(uint32_t) - p.total_bytes;
  }
}

static void layer_geometry(const slkv_layer_desc* d, Geometry& g) {
  g.ragged = false; g.h_begin = d->h_cu_seqlens; g.h_caps = d->h_budgets;
  g.dtype = d->dtype; g.Hq = d->Hq; g.Hkv = d->Hkv; g.d = d->d; g.w = d->w;
  g.pool_kernel = d->pool_kernel; g.pool = d->pool;
  g.k_stride_tok = d->k_stride_tok; g.k_stride_head = d->k_stride_head;
  g.v_stride_tok = d->v_stride_tok; g.v_stride_head = d->v_stride_head;
  g.score_elems = (int64_t)d->Hkv * d->h_cu_seqlens[d->B];
  const int G = d->Hq / d->Hkv;
  g.segs.resize((size_t)d->B * d->Hkv);
  for (int b = 0; b < d->B; ++b) {
    const int64_t n = d->h_cu_seqlens[b + 1] - d->h_cu_seqlens[b];
    for (int h = 0; h < d->Hkv; ++h) {
      Seg& s = g.segs[(size_t)b * d->Hkv + h];
      s.row_begin = d->h_cu_seqlens[b];
      s.n = n;
      s.cap = d->h_budgets[h];
      s.head = h;
      s.qrow_off = ((int64_t)b * d->Hq + (int64_t)h * G) * d->w;
      s.score_off = (int64_t)d->Hkv * d->h_cu_seqlens[b] + (int64_t)h * n;
    }
  }
  g.longest = longest_ranked(g);
}

static void ragged_geometry(const slkv_ragged_desc* d, Geometry& g) {
  g.ragged = true; g.h_begin = d->h_in_offsets; g.h_caps = d->h_budgets;
  g.dtype = d->dtype; g.Hq = d->Hq; g.Hkv = d->Hkv; g.d = d->d; g.w = d->w;
  g.pool_kernel = d->pool_kernel; g.pool = d->pool;
  g.k_stride_tok = g.v_stride_tok = d->d;     // packed rows
  g.k_stride_head = g.v_stride_head = 0;      // a segment's rows are addressed by row_begin alone
  const int S = d->B * d->Hkv;
  g.score_elems = d->h_in_offsets[S] - d->h_in_offsets[0];
  const int G = d->Hq / d->Hkv;
  g.segs.resize((size_t)S);
  for (int i = 0; i < S; ++i) {
    const int b = i / d->Hkv, h = i % d->Hkv;
    Seg& s = g.segs[(size_t)i];
    s.row_begin = d->h_in_offsets[i];
    s.n = d->h_in_offsets[i + 1] - d->h_in_offsets[i];
    s.cap = d->h_budgets[h];
    s.head = 0;
    s.qrow_off = ((int64_t)b * d->Hq + (int64_t)h * G) * d->w;
    s.score_off = d->h_in_offsets[i] - d->h_in_offsets[0];
  }
  g.longest = longest_ranked(g);
}

// Grid of a scoring launch: `chunks` workgroups in a row, or (rows > 0) one row of `per_row`
// workgroups per segment.
struct ScoreGrid {
  int chunks, per_row, rows;
};

// The passes of a call: 1 and 2, both in one launch, these with the selection and the copy, or three for one pass over the keys.
constexpr int kPassSample = 0, kPassTogether = 3, kPassFinish = 4, kPassBoth = 5, kPassChosen = 6;

// What the scoring passes write, for each other and for the selection.
struct ScoreBuffers {
  float *part, *imp;
  uint32_t* gm;            // largest scores of the groups, or NULL
  OneScan one;             // the rest is for one pass over the keys
  float* pooled;
  uint32_t* blockhist;     // or NULL: one workgroup per segment selects
  meet_t* meet;            // both passes in one launch: where their workgroups meet (see meet_chunks), or NULL
  int limit;               // and how long they wait, in ticks of 10 ns
  FinishArgs fin;          // kPassFinish: the rest of the call
};

template <int DK, int MT, int RB, int KIND, class TAB>
static void launch_q_resident(int pass, ScoreGrid grid, hipStream_t st, const TAB& tab, const void* q, const void* k,
                              const Geometry& g, const Plan& p, float c_log2, const ScoreBuffers& buf) {
  // segments with like chunk counts: one grid row per segment (see the kernel's first lines)
  const bool two = grid.rows > 0;
  const dim3 gr = two ? dim3((unsigned)grid.per_row, (unsigned)grid.rows) : dim3((unsigned)grid.chunks);
  auto scan = [&](auto pass_c) {
    SLKV_LAUNCH((score_q_resident_kernel<DK, MT, RB, decltype(pass_c)::value, KIND, TAB>), gr, dim3(256), 0, st, tab, (const uint16_t*)q, k,
                g.k_stride_tok, g.k_stride_head, p.R, p.Rpad, g.w, p.CH, c_log2, buf.part, buf.imp, two ? 1 : 0, buf.gm, buf.meet, buf.limit, buf.fin);
  };
  if (pass == 1) scan(std::integral_constant<int, 1>{});
  if (pass == 2) scan(std::integral_constant<int, 2>{});
  if (pass == kPassTogether) scan(std::integral_constant<int, 3>{});
  if constexpr (std::is_same_v<TAB, SegTableBig>) {
    if (pass == kPassFinish) scan(std::integral_constant<int, 4>{});
  }
  if constexpr (MT <= 2 && std::is_same_v<TAB, SegTable>) {
    const unsigned S = (unsigned)g.segs.size();
    if (pass == kPassSample)
      SLKV_LAUNCH((score_sample_kernel<DK, MT * RB, KIND>), dim3((unsigned)p.ranges), dim3(512), 0, st, tab, (const uint16_t*)q, k, g.k_stride_tok,
                  g.k_stride_head, p.R, p.Rpad, g.w, p.sampled, c_log2, buf.one);
    if (pass == kPassBoth)
      SLKV_LAUNCH((score_both_kernel<DK, MT, RB, KIND>), gr, dim3(256), 0, st, tab, (const uint16_t*)q, k, g.k_stride_tok,
                  g.k_stride_head, p.R, p.Rpad, g.w, p.CH, c_log2, buf.part, buf.imp, two ? 1 : 0, buf.one);
    if (pass == kPassChosen) {
      const int radius = g.pool == SLKV_POOL_NONE ? 0 : g.pool_kernel / 2;
      SLKV_LAUNCH(approx_hist_kernel, dim3((unsigned)((g.longest + kApproxBlock - 1) / kApproxBlock + 1), S), dim3(256), 0, st, tab, g.w, radius, p.R, p.Rpad,
                  buf.part, buf.imp, buf.one);
      auto exact = [&](int probe) {
        SLKV_LAUNCH((select_chosen_kernel<DK, MT * RB, KIND>), dim3((unsigned)p.ranges), dim3(512), 0, st, tab, (const uint16_t*)q, k,
                    g.k_stride_tok, g.k_stride_head, p.R, g.w, p.sampled, radius, c_log2, buf.one, buf.imp, buf.pooled, buf.blockhist, probe);
      };
      exact(1);
      exact(0);
    }
  }
}

template <int DK, int KIND, class TAB>
static void launch_score_k(int pass, ScoreGrid grid, hipStream_t st, const TAB& tab, const void* q, const void* k,
                           const Geometry& g, const Plan& p, float c_log2, const ScoreBuffers& buf) {
  if constexpr (KIND <= 1) {
    if (p.R <= 64) launch_q_resident<DK, 1, 2, KIND>(pass, grid, st, tab, q, k, g, p, c_log2, buf);
    else if (p.R <= 128) launch_q_resident<DK, 2, 2, KIND>(pass, grid, st, tab, q, k, g, p, c_log2, buf);
    else if (p.R <= 256) launch_q_resident<DK, 2, 4, KIND>(pass, grid, st, tab, q, k, g, p, c_log2, buf);
    else launch_q_resident<DK, 4, 4, KIND>(pass, grid, st, tab, q, k, g, p, c_log2, buf);
  } else {
    const bool two = grid.rows > 0;
    const dim3 gr = two ? dim3((unsigned)grid.per_row, (unsigned)grid.rows) : dim3((unsigned)grid.chunks);
    const size_t lds = score_lds_bytes<DK, KIND>(std::min((p.R + 31) / 32, ScoreCfg<DK, KIND>::RBT), p.waves);
    auto scan = [&](auto pass_c) {
      SLKV_LAUNCH((score_k_resident_kernel<DK, KIND, decltype(pass_c)::value, TAB>), gr, dim3(64 * p.waves), lds, st, tab, q, k, g.k_stride_tok,
                  g.k_stride_head, p.R, p.Rpad, g.w, p.CH, c_log2, buf.part, buf.imp, two ? 1 : 0, p.rsplit, buf.gm, buf.meet, buf.limit);
    };
    if (pass == 1) scan(std::integral_constant<int, 1>{});
    if (pass == 2) scan(std::integral_constant<int, 2>{});
    if (pass == kPassTogether) scan(std::integral_constant<int, 3>{});
  }
}

template <class TAB>
static void launch_score(int pass, ScoreGrid grid, hipStream_t st, const TAB& tab, const void* q, const void* k,
                         const Geometry& g, const Plan& p, float c_log2, const ScoreBuffers& buf) {
  with_score_kind(g.d, g.dtype, [&](auto dk, auto kind) {
    launch_score_k<decltype(dk)::value, decltype(kind)::value>(pass, grid, st, tab, q, k, g, p, c_log2, buf);
  });
}

template <class TAB>
static void launch_select(int nseg, int blocks, hipStream_t st, const TAB& tab, const Geometry& g, const float* imp,
                          float* pooled, uint32_t* blockhist, uint32_t* lists, int32_t* kept_idx, int64_t* d_out_offsets,
                          const GatherArgs& ga, const OneScan& one) {
  const bool chosen = one.hist != nullptr;
  const int radius = g.pool == SLKV_POOL_NONE ? 0 : g.pool_kernel / 2;
  const int pool_kernel = g.pool == SLKV_POOL_NONE ? 1 : g.pool_kernel;
#define SLKV_POOL_LAUNCH(RAD)                                                                                          \
  SLKV_LAUNCH((select_pool_kernel<RAD, TAB>), dim3(blocks), dim3(kSelThreads), 0, st, tab, g.w, pool_kernel, g.pool, imp, \
              pooled, blockhist)
  if (blocks > 0 && !chosen) {                           // (chosen: select_chosen_kernel has pooled and listed the scores)
    switch (radius) {
      case 0: SLKV_POOL_LAUNCH(0); break;
      case 1: SLKV_POOL_LAUNCH(1); break;
      case 2: SLKV_POOL_LAUNCH(2); break;
      case 3: SLKV_POOL_LAUNCH(3); break;
      default: SLKV_POOL_LAUNCH(-1); break;
    }
  }
#undef SLKV_POOL_LAUNCH
  // with blocks, the ordered compaction runs per block (two short launches over the whole chip)
  // instead of per segment inside the ranking workgroup
  const int split = blocks > 0 ? 1 : 0;
  const int64_t longest = (g.longest + kSelBlock - 1) / kSelBlock;
  // block-wise launches: a grid row per segment unless that would launch mostly empty workgroups
  // (one long history among many short ones) or more rows than a grid has
  const bool rows = nseg <= 65535 && longest * nseg <= 4 * (int64_t)blocks;
  const dim3 grid = rows ? dim3((unsigned)std::max<int64_t>(longest, 1), (unsigned)nseg) : dim3((unsigned)std::max(blocks, 1));
  if (split && !chosen) {
    // first-level digit per segment, then the blocks list the scores of that digit
    SLKV_LAUNCH(select_rank_kernel<TAB>, dim3(nseg), dim3(kSelThreads), 0, st, tab, g.w, (const float*)pooled,
                blockhist, kept_idx, d_out_offsets, ga, split, (const uint32_t*)lists, 0, one);
    SLKV_LAUNCH(select_collect_kernel<TAB>, grid, dim3(kSelEmitThreads), 0, st, tab, g.w, (const float*)pooled, blockhist,
                lists, rows ? 0 : -1);
  }
  SLKV_LAUNCH(select_rank_kernel<TAB>, dim3(nseg), dim3(kSelThreads), 0, st, tab, g.w, (const float*)pooled,
              blockhist, kept_idx, d_out_offsets, ga, split, (const uint32_t*)lists, 1, one);
  if (split) {
    SLKV_LAUNCH(select_count_kernel<TAB>, grid, dim3(kSelEmitThreads), 0, st, tab, g.w, (const float*)pooled, blockhist,
                rows ? 0 : -1);
    SLKV_LAUNCH(select_emit_kernel<TAB>, grid, dim3(kSelEmitThreads), 0, st, tab, g.w, (const float*)pooled,
                (const uint32_t*)blockhist, kept_idx, rows ? 0 : -1);
  }
}

// select_resident_kernel needs more LDS than a kernel gets by default: the limit is raised for all
// of its instances once per device, by slkv_init() or by the first call that selects on that
// device (setting it is not a stream operation, but the first call on a device should still not
// be the one a graph capture records).
template <int RADIUS, int EPT>
static hipError_t raise_lds_limit() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&select_resident_kernel<RADIUS, EPT, SegTable>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLdsBytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&select_resident_kernel<RADIUS, EPT, SegTableBig>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLdsBytes);
}

template <int EPT>
static hipError_t raise_lds_limits() {
  hipError_t e;
  if ((e = raise_lds_limit<0, EPT>()) != hipSuccess) return e;
  if ((e = raise_lds_limit<1, EPT>()) != hipSuccess) return e;
  if ((e = raise_lds_limit<2, EPT>()) != hipSuccess) return e;
  if ((e = raise_lds_limit<3, EPT>()) != hipSuccess) return e;
  return raise_lds_limit<-1, EPT>();
}

template <int DK, int KIND, class TAB>
static hipError_t raise_score_limit() {
  if constexpr (KIND <= 1) return hipSuccess;          // (score_q_resident_kernel has static LDS)
  else {
    for (const void* kernel : {reinterpret_cast<const void*>(&score_k_resident_kernel<DK, KIND, 1, TAB>), reinterpret_cast<const void*>(&score_k_resident_kernel<DK, KIND, 2, TAB>),
                               reinterpret_cast<const void*>(&score_k_resident_kernel<DK, KIND, 3, TAB>)}) {
      const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
}

static hipError_t raise_score_limits() {
  for (const int d : {64, 128})
    for (const int dtype : {SLKV_F32, SLKV_BF16_KV_FP8}) {
      const hipError_t e = with_score_kind(d, dtype, [](auto dk, auto kind) {
        const hipError_t a = raise_score_limit<decltype(dk)::value, decltype(kind)::value, SegTable>();
        return a != hipSuccess ? a : raise_score_limit<decltype(dk)::value, decltype(kind)::value, SegTableBig>();
      });
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

// The set-up of the current device, whose number of CUs goes to `cus`.
static hipError_t ensure_device_init(int* cus = nullptr) {
  static std::mutex mu;
  static uint64_t done = 0;                      // bit per device
  static int cus_of[64];
  int dev = 0, have = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t(1) << dev) : 0;
  if (done & bit) {
    if (cus) *cus = cus_of[dev];
    return hipSuccess;
  }
  if ((e = hipDeviceGetAttribute(&have, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  if (cus) *cus = have;
  if (bit) cus_of[dev] = have;
  if ((e = raise_score_limits()) != hipSuccess) return e;
  if ((e = raise_lds_limits<kSelEPT>()) != hipSuccess) return e;
  if ((e = raise_lds_limits<kSelEPTLong>()) != hipSuccess) return e;
  if ((e = raise_lds_limits<kSelEPTMore>()) != hipSuccess) return e;
  if ((e = raise_lds_limits<kSelEPTLess>()) != hipSuccess) return e;
  if ((e = raise_lds_limits<kSelEPTMid>()) != hipSuccess) return e;
  if ((e = raise_lds_limits<kSelEPTSmall>()) != hipSuccess) return e;
  done |= bit;
  return hipSuccess;
}

// Workgroups of select_resident_kernel: one per segment, or per slice of 2^slice_log2 kept rows of one.
struct SelectGrid {
  int workgroups, slice_log2;
};

template <int RADIUS, int EPT, class TAB>
static hipError_t launch_select_resident_e(SelectGrid sel, hipStream_t st, const TAB& tab, const Geometry& g, bool write_pooled, const uint32_t* gm,
                                           const float* imp, float* pooled, int32_t* kept_idx, int64_t* d_out_offsets,
                                           const GatherArgs& ga, meet_t* meet) {
  const hipError_t e = ensure_device_init();
  if (e != hipSuccess) return e;
  const int pool_kernel = g.pool == SLKV_POOL_NONE ? 1 : g.pool_kernel;
  SLKV_LAUNCH((select_resident_kernel<RADIUS, EPT, TAB>), dim3(sel.workgroups), dim3(kSelThreads), kResLdsBytes, st, tab, g.w,
                     pool_kernel, g.pool, (int)write_pooled, imp, gm, pooled, kept_idx, d_out_offsets, ga, meet, sel.slice_log2);
  return hipSuccess;
}

// Positions per thread: the fewest of 2, 4, 8, 16, 24, 32 whose round holds the longest ranked history (every
// wave runs through all of a thread's positions, whether or not the history reaches them).  Without 4, 16 and 24 / with them, us a call:
// averages, 8 x 9 K 34.2 / 29.6, 8 x 16 K 37.1 / 33.1, 8 x 20 K 39.8 / 37.6, of 13 and 700 kept, 8 x 12 K 62.6 / 45.6; 21 K fp16, budgets of 1024 59.5 / 56.8; maxima,
// budgets of 1024, 8 x 12 K 38.6 / 33.2; fp32 4 x 10 K 40.5 / 37.2; 8 x 4 K 22.2 / 21.5, averages 21.9 / 20.9; 8 prompts of 2 to 4 K 42.4 / 41.3.  (Window maxima
// above 8192 positions mostly go by groups, whatever the form.)
template <int RADIUS, class TAB>
static hipError_t launch_select_resident_r(SelectGrid sel, hipStream_t st, const TAB& tab, const Geometry& g, bool write_pooled, const uint32_t* gm,
                                           const float* imp, float* pooled, int32_t* kept_idx, int64_t* d_out_offsets,
                                           const GatherArgs& ga, meet_t* meet) {
  if (g.longest <= kSelThreads * kSelEPTSmall)
    return launch_select_resident_e<RADIUS, kSelEPTSmall>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
  if (g.longest <= kSelThreads * kSelEPTLess)
    return launch_select_resident_e<RADIUS, kSelEPTLess>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
  if (g.longest <= kSelThreads * kSelEPTMid)
    return launch_select_resident_e<RADIUS, kSelEPTMid>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
  if (g.longest <= kSelThreads * kSelEPTMore)
    return launch_select_resident_e<RADIUS, kSelEPTMore>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
  if (g.longest <= kSelThreads * kSelEPTLong)
    return launch_select_resident_e<RADIUS, kSelEPTLong>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
  return launch_select_resident_e<RADIUS, kSelEPT>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
}

template <class TAB>
static hipError_t launch_select_resident(SelectGrid sel, hipStream_t st, const TAB& tab, const Geometry& g, bool write_pooled, const uint32_t* gm,
                                         const float* imp, float* pooled, int32_t* kept_idx, int64_t* d_out_offsets,
                                         const GatherArgs& ga, meet_t* meet) {
  const int radius = g.pool == SLKV_POOL_NONE ? 0 : g.pool_kernel / 2;
  switch (radius) {
    case 0: return launch_select_resident_r<0>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
    case 1: return launch_select_resident_r<1>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
    case 2: return launch_select_resident_r<2>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
    case 3: return launch_select_resident_r<3>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
    default: return launch_select_resident_r<-1>(sel, st, tab, g, write_pooled, gm, imp, pooled, kept_idx, d_out_offsets, ga, meet);
  }
}

// SLKV_SELECT=resident|blocks in the environment forces one selection kernel (tests run both on
// every shape the resident one covers); default: chosen per call, or none where the scoring launch selects.  0 auto, 1 resident, 2 blocks.
static int select_mode() {
  const char* e = std::getenv("SLKV_SELECT");
  if (!e) return 0;
  if (!std::strcmp(e, "resident")) return 1;
  if (!std::strcmp(e, "blocks")) return 2;
  return 0;
}

// How long the workgroups of a launch that does both passes wait for each other, in ticks of 10 ns.  Alone they start and end up to 10 us apart, but other
// streams' workgroups hold CUs for the time of a pass of their own, and a short last chunk waits for a whole one of the others.  Who leaves too early costs much: the few
// that come last complete the chunks of all others, one by one.  So it is twice the time of both passes by the plan, and some for what else keeps them.  us a call on 1, 2,
// 3 and 4 streams, limits of 50 us / of this / two launches: E4M3 32 x 32 K 152 146 425 405 / 152 146 148 150 / 159 149 151 151; 64 x 32 K 280 276 498 470 / 278 276 282 283 /
// 283 285 284 284; six prompts of 2 to 32 K 151 143 314 356 / 151 141 144 144 / 163 144 145 143.  (Least that avoids it: 100, 200 and 75 us; 8 x 32 K 35 us, 16-bit keys 50.)
// SLKV_MEET_US in the environment sets another limit (tests: 0, so that nearly all leave and the last ones complete their chunks).
static int meet_limit(const Plan& p) {
  const char* e = std::getenv("SLKV_MEET_US");
  const double us = e ? (double)std::atoi(e) : 20 + 2 * p.passes_us;
  return (int)(std::min(std::max(us, 0.0), 10000.0) * 100);
}

// Checks and launches shared by the two entry points.
static slkv_status run_geometry(const Geometry& g, const void* d_qwin, const void* d_k, const void* d_v,
                                const int32_t* d_pos_in, void* d_k_out, void* d_v_out, int32_t* d_kept_idx,
                                int32_t* d_pos_out, int64_t* d_out_offsets, float* d_importance, float* d_pooled,
                                int64_t out_capacity_rows, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  // an input without rows, or an output without kept rows, may come with NULL buffers
  int64_t rows_in = 0, rows_kept = 0;
  for (const Seg& sg : g.segs) {
    rows_in += sg.n;
    rows_kept += kept_rows(sg.n, g.w, sg.cap);
  }
  if (!d_qwin || !d_workspace || (rows_in > 0 && (!d_k || !d_v)) ||
      (rows_kept > 0 && (!d_k_out || !d_v_out || !d_kept_idx)))
    return fail(SLKV_ERR_NULL, "a required device pointer is NULL");
  if (rows_kept > 0 && (d_pos_in == nullptr) != (d_pos_out == nullptr))
    return fail(SLKV_ERR_NULL, "d_pos_in and d_pos_out must be given together");
  if (!d_pos_in || !d_pos_out) d_pos_in = nullptr, d_pos_out = nullptr;   // nothing kept: nothing to carry

  const void* ptrs[] = {d_qwin, d_k, d_v, d_pos_in, d_k_out, d_v_out, d_kept_idx, d_pos_out, d_out_offsets,
                        d_importance, d_pooled, d_workspace};
  for (const void* ptr : ptrs)
    if (reinterpret_cast<uintptr_t>(ptr) % 16) return fail(SLKV_ERR_BAD_ARG, "device pointer %p not 16-byte aligned", ptr);
  const int elt = g.dtype == SLKV_F32 ? 4 : (g.dtype == SLKV_BF16_KV_FP8 ? 1 : 2);   // bytes per element of K and V
  const int64_t S = (int64_t)g.segs.size();
  if (S / g.Hkv * g.Hq * g.w >= (int64_t(1) << 31)) return fail(SLKV_ERR_BAD_ARG, "B*Hq*w >= 2^31");
  int64_t total_kept = 0;
  for (int64_t i = 0; i < S; ++i) {   // the kernels address a segment's keys with 32-bit byte offsets
    const Seg& s = g.segs[(size_t)i];
    if (s.n * g.k_stride_tok * elt >= (int64_t(1) << 31))
      return fail(SLKV_ERR_UNSUPPORTED, "segment %lld spans 2 GiB or more of K", (long long)i);
    total_kept += kept_rows(s.n, g.w, s.cap);
  }
  if (total_kept >= (int64_t(1) << 31)) return fail(SLKV_ERR_BAD_ARG, "kept rows >= 2^31");
  Plan p;
  make_plan(g, p);
  if (workspace_bytes < p.total_bytes)
    return fail(SLKV_ERR_WORKSPACE, "workspace %zu < %zu bytes", workspace_bytes, p.total_bytes);
  if (out_capacity_rows < total_kept)
    return fail(SLKV_ERR_CAPACITY, "out_capacity_rows %lld < %lld", (long long)out_capacity_rows, (long long)total_kept);

  hipStream_t st = (hipStream_t)hip_stream;
  unsigned char* ws = (unsigned char*)d_workspace;
  float* part = (float*)(ws + p.off_part);
  float* imp = d_importance ? d_importance : (float*)(ws + p.off_imp);
  float* pooled = d_pooled ? d_pooled : (float*)(ws + p.off_pooled);
  const float c_log2 = (float)(1.4426950408889634 / std::sqrt((double)g.d));
  const int lanes_per_row = g.d * elt / 16;

  GatherArgs ga;
  ga.k = (const unsigned char*)d_k;
  ga.v = (const unsigned char*)d_v;
  ga.k_out = (unsigned char*)d_k_out;
  ga.v_out = (unsigned char*)d_v_out;
  ga.k_stride_tok = g.k_stride_tok;
  ga.k_stride_head = g.k_stride_head;
  ga.v_stride_tok = g.v_stride_tok;
  ga.v_stride_head = g.v_stride_head;
  ga.lanes_per_row = lanes_per_row;
  ga.elt_bytes = elt;
  ga.pos_in = d_pos_in;
  ga.pos_out = d_pos_out;

  uint32_t* blockhist = (uint32_t*)(ws + p.off_hist);
  // candidate lists of the block-wise selection: the workspace's importance area, which is either
  // unused (the caller asked for the importance scores in an array of its own) or dead by then
  // (pooling has consumed the scores)
  uint32_t* lists = (uint32_t*)(ws + p.off_imp);

  int cus = 0;
  const hipError_t ie = ensure_device_init(&cus);
  if (ie != hipSuccess) return fail(SLKV_ERR_HIP, "device set-up failed: %s", hipGetErrorString(ie));
  const bool k_resident = g.dtype == SLKV_F32 || g.dtype == SLKV_BF16_KV_FP8;

  // The kernels of the pass over the segments one table describes.
  // Selection kernel: if every history fits one round, the one-workgroup-per-segment kernel;
  // otherwise the histories are cut into blocks.
  const bool resident_select = select_mode() != 2 && g.longest <= kSelRound;
  const int nseg = (int)S;
  // The selection starts from the groups' largest scores where a thread would have 16, 24 or 32 positions to go through otherwise (with 8 or fewer the shorter
  // chain of phases wins: 8 x 8 K keys 25.7 us either way, 8 x 900 keys 22.4 us without, 24.8 with), and not for
  // fp32, whose scoring kernel got slower by it on short calls (4 x 1 K 19.7 -> 20.1).  They lie in the pooled array, which nobody writes then.
  // (a group's place counts the segments before it, see group_off: with thousands of empty ones the array may be too short)
  const bool groups = resident_select && !d_pooled && g.pool != SLKV_POOL_AVG && g.dtype != SLKV_F32 && g.longest > kSelThreads * kSelEPTMid &&
                      g.score_elems / kGroup + S + 1 <= g.score_elems;
  // one pass over the keys where no importance or pooled score is asked for: only the selection is exact there
  const bool one_scan = p.one_scan && !d_importance && !d_pooled && workspace_bytes >= p.total_bytes + p.one_scan_bytes;
  OneScan one{};
  if (one_scan)
    one = OneScan{(float*)(ws + p.off_part0), (float*)(ws + p.off_dense), (uint32_t*)(ws + p.off_bins), (float*)(ws + p.off_lse), (uint32_t*)(ws + p.off_bounds),
                  (uint32_t*)(ws + p.off_lists)};
  uint32_t* const gm = groups && !one_scan ? (uint32_t*)pooled : nullptr;
  ScoreBuffers buf{part, imp, gm, one, pooled, resident_select ? nullptr : blockhist, nullptr, 0, FinishArgs{}};
  int64_t unranked = 0;                              // workgroups that copy segments that are not ranked, where one launch does everything
  auto launch_group = [&](const auto& tab, int chunks, int max_chunks, int blocks, bool any_large, const int64_t* slices, int64_t rows) -> slkv_status {
    using TAB = std::decay_t<decltype(tab)>;
    // one grid row per segment where that leaves at most a seventh of the grid empty (a segment with
    // fewer chunks than the longest leaves the surplus of its row empty; with more empty workgroups
    // the full ones no longer spread evenly over the CUs: a ragged batch ran 22 % slower), else one
    // row over all chunks
    ScoreGrid sgrid{chunks, 0, 0};
    if (tab.nseg <= 65535 && (int64_t)max_chunks * tab.nseg * 6 <= (int64_t)chunks * 7) {
      sgrid.per_row = max_chunks;
      sgrid.rows = tab.nseg;
    }
    // Both passes in one launch where all its workgroups fit the chip at once and the selection clears their meeting places.
    if (!one_scan && resident_select && S <= kMeetSegments && max_chunks > (k_resident ? 1 : 0) && max_chunks <= p.meet_most &&
        chunks <= p.per_cu * cus) {
      buf.meet = (meet_t*)ws;
      buf.limit = meet_limit(p);
    }
    SelectGrid sel{nseg, 0};
    const bool slice = resident_select && (any_large || g.longest > kSelThreads * kSelEPTSmall);
    for (int l = kSliceLog2Least; slice && !sel.slice_log2 && l <= kSliceLog2Most; ++l)
      if (slices[l - kSliceLog2Least] <= cus) sel = SelectGrid{(int)slices[l - kSliceLog2Least], l};
    // The selection and the copy in the same launch too, where a gather would follow (both sides: finish_segment).
    if (std::is_same_v<TAB, SegTableBig> && !k_resident && buf.meet && any_large && !sel.slice_log2 && g.longest <= kFinishMost && select_mode() == 0) {
      buf.fin = FinishArgs{ga, pooled, d_kept_idx, d_out_offsets, g.pool == SLKV_POOL_NONE ? 1 : g.pool_kernel, g.pool, d_pooled != nullptr, chunks};
      sgrid.chunks = chunks + (int)unranked;
      if (unranked > 0) sgrid.rows = 0;
      ScopedKernelTimer tm(SLKV_K_SCORE_ACCUM, st);
      launch_score(kPassFinish, sgrid, st, tab, d_qwin, d_k, g, p, c_log2, buf);
      const hipError_t e = hipGetLastError();
      return e == hipSuccess ? SLKV_OK : fail(SLKV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    }
    if (chunks > 0 && buf.meet) {
      ScopedKernelTimer tm(SLKV_K_SCORE_ACCUM, st);
      launch_score(kPassTogether, sgrid, st, tab, d_qwin, d_k, g, p, c_log2, buf);
    } else if (chunks > 0) {
      {
        ScopedKernelTimer tm(SLKV_K_SCORE_STATS, st);
        launch_score(one_scan ? kPassSample : 1, sgrid, st, tab, d_qwin, d_k, g, p, c_log2, buf);
      }
      if (one_scan) {
        ScopedKernelTimer tm(SLKV_K_SCORE_ACCUM, st);
        launch_score(kPassBoth, sgrid, st, tab, d_qwin, d_k, g, p, c_log2, buf);
        launch_score(kPassChosen, sgrid, st, tab, d_qwin, d_k, g, p, c_log2, buf);
      } else if (max_chunks > 1 || !k_resident) {             // (score_k_resident_kernel completes segments of one chunk in its first pass)
        ScopedKernelTimer tm(SLKV_K_SCORE_ACCUM, st);
        launch_score(2, sgrid, st, tab, d_qwin, d_k, g, p, c_log2, buf);
      }
    }
    {
      ScopedKernelTimer tm(SLKV_K_SELECT, st);
      if (resident_select) {
        hipError_t se = launch_select_resident(sel, st, tab, g, d_pooled != nullptr, gm, imp, pooled, d_kept_idx, d_out_offsets, ga, buf.meet);
        if (se != hipSuccess) return fail(SLKV_ERR_HIP, "select launch setup failed: %s", hipGetErrorString(se));
      } else {
        launch_select(nseg, blocks, st, tab, g, imp, pooled, blockhist, one_scan ? one.lists : lists, d_kept_idx, d_out_offsets, ga, one);
      }
    }
    const bool gather_all = !resident_select && blocks > 0;   // the block-wise selection copies no rows itself
    if ((any_large || gather_all) && !sel.slice_log2 && rows > 0) {
      ScopedKernelTimer tm(SLKV_K_GATHER, st);
      const int64_t threads = rows * lanes_per_row;
      if (threads > kGatherThreads)
        SLKV_LAUNCH((gather_kernel<4, TAB>), dim3((unsigned)((threads + 1023) / 1024)), dim3(256), 0, st, tab, ga, d_kept_idx, gather_all ? 1 : 0);
      else
        SLKV_LAUNCH((gather_kernel<1, TAB>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, tab, ga, d_kept_idx, gather_all ? 1 : 0);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SLKV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    return SLKV_OK;
  };

  // The segment table, with the prefixes of output rows, key chunks and selection blocks over the segments.
  int64_t out_run = 0, chunks = 0, max_chunks = 0, blocks = 0, slices[kSliceLog2Most - kSliceLog2Least + 1] = {};
  bool any_large = false;
  auto walk = [&](int32_t* out, int32_t* chunk, int32_t* blk) {   // (blk may be NULL)
    for (int64_t i = 0; i < S; ++i) {
      const Seg& sg = g.segs[(size_t)i];
      out[i] = (int32_t)out_run;
      chunk[i] = (int32_t)chunks;
      if (blk) blk[i] = (int32_t)blocks;
      const int64_t kept = kept_rows(sg.n, g.w, sg.cap), nc = seg_chunks(sg, g.w, p.CH);
      any_large |= kept > kInlineGatherRows;
      for (int l = kSliceLog2Least; l <= kSliceLog2Most; ++l) slices[l - kSliceLog2Least] += 1 + (std::max<int64_t>(kept - 1, 0) >> l);
      if (nc == 0) unranked += 1 + (std::max<int64_t>(kept - 1, 0) >> kFinishRowsLog2);
      out_run += kept;
      chunks += nc;
      max_chunks = std::max(max_chunks, nc);
      blocks += seg_blocks(sg, g.w);
    }
    out[S] = (int32_t)out_run;
    chunk[S] = (int32_t)chunks;
    if (blk) blk[S] = (int32_t)blocks;
    return chunks < (int64_t(1) << 31) && blocks < (int64_t(1) << 31);
  };
  if (S <= kMaxSegPerLaunch) {
    SegTable tab;
    tab.nseg = (int32_t)S;
    for (int64_t i = 0; i < S; ++i) {
      const Seg& sg = g.segs[(size_t)i];
      tab.tok_[i] = (int32_t)sg.row_begin;
      tab.n_[i] = (int32_t)sg.n;
      tab.head_[i] = sg.head;
      const bool all = sg.n <= g.w || sg.n <= sg.cap;
      tab.kk_[i] = all ? -1 : (int32_t)std::min<int64_t>(std::max<int64_t>(sg.cap - g.w, 0), sg.n - g.w);
      tab.score_[i] = (int32_t)sg.score_off;
    }
    if (!walk(tab.out_, tab.chunk_, tab.blk_)) return fail(SLKV_ERR_BAD_ARG, "too many key chunks");
    if (one_scan) {
      tab.range_[0] = 0;
      for (int64_t i = 0; i < S; ++i) tab.range_[i + 1] = tab.range_[i] + (int32_t)seg_ranges(g.segs[(size_t)i], g.w, p.sampled);
    }
    return launch_group(tab, (int)chunks, (int)max_chunks, (int)blocks, any_large, slices, out_run);
  }
  SegTableBig tab;
  const int nbeg = (int)(g.ragged ? S : S / g.Hkv) + 1;
  tab.nseg = (int32_t)S;
  tab.hkv = g.Hkv;
  tab.w = g.w;
  tab.ragged = g.ragged ? 1 : 0;
  tab.off_cap = nbeg;
  tab.off_out = tab.off_cap + g.Hkv;
  tab.off_chunk = tab.off_out + (int32_t)S + 1;
  tab.off_blk = tab.off_chunk + (int32_t)S + 1;            // (only the block-wise selection reads these)
  const size_t count = (size_t)tab.off_blk + (resident_select ? 0 : (size_t)S + 1);
  const bool in_arg = count <= (size_t)kArgWords;
  std::vector<int32_t> spill;
  if (!in_arg) spill.resize(count);
  int32_t* const words = in_arg ? tab.words : spill.data();
  for (int i = 0; i < nbeg; ++i) words[i] = (int32_t)g.h_begin[i];
  for (int h = 0; h < g.Hkv; ++h) words[tab.off_cap + h] = g.h_caps[h];
  if (!walk(words + tab.off_out, words + tab.off_chunk, resident_select ? nullptr : words + tab.off_blk))
    return fail(SLKV_ERR_BAD_ARG, "too many key chunks");
  tab.mem = nullptr;
  if (!in_arg) {
    int32_t* const t = (int32_t*)(ws + p.off_table);
    for (size_t i = 0; i < count; i += kArgWords) {
      UploadWords part;
      const int c = (int)std::min<size_t>(kArgWords, count - i);
      std::memcpy(part.w, words + i, (size_t)c * sizeof(int32_t));
      SLKV_LAUNCH(upload_kernel, dim3(1), dim3(1024), 0, st, part, c, t + i);
    }
    tab.mem = t;
  }
  return launch_group(tab, (int)chunks, (int)max_chunks, (int)blocks, any_large, slices, out_run);
}

}  // namespace slkv

using namespace slkv;

// Scratch of slkv_compress_layer_static: one copy per GPU, held until the process ends.
static __device__ __align__(256) unsigned char scratch[SLKV_STATIC_SCRATCH_BYTES];

// Device address of `scratch` on the current device, looked up, and its header cleared, once per device and again after a call that failed
// between its launches (failed: nothing is returned).
static slkv_status static_scratch(void** out, bool failed = false) {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static void* ptrs[kMaxDev] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(SLKV_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDev) return fail(SLKV_ERR_UNSUPPORTED, "device index %d outside 0..%d", dev, kMaxDev - 1);
  std::lock_guard<std::mutex> lk(mu);
  if (failed) {
    ptrs[dev] = nullptr;
    return SLKV_OK;
  }
  if (!ptrs[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) return fail(SLKV_ERR_HIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    e = hipMemset(ptr, 0, SLKV_WORKSPACE_HEADER_BYTES);      // the header of a workspace is zero (not under capture)
    if (e != hipSuccess) return fail(SLKV_ERR_HIP, "clearing the static scratch failed: %s", hipGetErrorString(e));
    ptrs[dev] = ptr;
  }
  *out = ptrs[dev];
  return SLKV_OK;
}

extern "C" slkv_status slkv_init(void) {
  clear_error();
  const hipError_t e = ensure_device_init();
  if (e != hipSuccess) return fail(SLKV_ERR_HIP, "device set-up failed: %s", hipGetErrorString(e));
  void* ptr = nullptr;
  return static_scratch(&ptr);
}

extern "C" slkv_status slkv_workspace_bytes(const slkv_layer_desc* desc, size_t* bytes) {
  clear_error();
  if (!bytes) return fail(SLKV_ERR_NULL, "bytes is NULL");
  slkv_status st = validate_desc(desc);
  if (st != SLKV_OK) return st;
  Geometry g;
  layer_geometry(desc, g);
  Plan p;
  make_plan(g, p);
  *bytes = p.total_bytes + p.one_scan_bytes;
  return SLKV_OK;
}

extern "C" slkv_status slkv_compress_layer(const slkv_layer_desc* desc, const void* d_qwin, const void* d_k,
                                           const void* d_v, void* d_k_out, void* d_v_out, int32_t* d_kept_idx,
                                           int64_t* d_out_offsets, float* d_importance, float* d_pooled,
                                           int64_t out_capacity_rows, void* d_workspace, size_t workspace_bytes,
                                           void* hip_stream) {
  clear_error();
  slkv_status vs = validate_desc(desc);
  if (vs != SLKV_OK) return vs;
  Geometry g;
  layer_geometry(desc, g);
  return run_geometry(g, d_qwin, d_k, d_v, nullptr, d_k_out, d_v_out, d_kept_idx, nullptr, d_out_offsets, d_importance,
                      d_pooled, out_capacity_rows, d_workspace, workspace_bytes, hip_stream);
}

extern "C" slkv_status slkv_compress_layer_static(const slkv_layer_desc* desc, const void* d_qwin, const void* d_k,
                                                  const void* d_v, void* d_k_out, void* d_v_out, int32_t* d_kept_idx,
                                                  int64_t* d_out_offsets, float* d_importance, float* d_pooled,
                                                  int64_t out_capacity_rows, void* hip_stream) {
  clear_error();
  slkv_status vs = validate_desc(desc);
  if (vs != SLKV_OK) return vs;
  Geometry g;
  layer_geometry(desc, g);
  Plan p;
  make_plan(g, p);
  if (p.total_bytes > (size_t)SLKV_STATIC_SCRATCH_BYTES)
    return fail(SLKV_ERR_WORKSPACE, "this call needs %zu bytes of scratch, the static buffer holds %zu: use slkv_compress_layer",
                p.total_bytes, (size_t)SLKV_STATIC_SCRATCH_BYTES);
  void* ws = nullptr;
  vs = static_scratch(&ws);
  if (vs != SLKV_OK) return vs;
  vs = run_geometry(g, d_qwin, d_k, d_v, nullptr, d_k_out, d_v_out, d_kept_idx, nullptr, d_out_offsets, d_importance,
                    d_pooled, out_capacity_rows, ws, (size_t)SLKV_STATIC_SCRATCH_BYTES, hip_stream);
  if (vs == SLKV_ERR_HIP) (void)static_scratch(&ws, true);
  return vs;
}

extern "C" slkv_status slkv_recompress_workspace_bytes(const slkv_ragged_desc* desc, size_t* bytes) {
  clear_error();
  if (!bytes) return fail(SLKV_ERR_NULL, "bytes is NULL");
  slkv_status st = validate_ragged_desc(desc);
  if (st != SLKV_OK) return st;
  Geometry g;
  ragged_geometry(desc, g);
  Plan p;
  make_plan(g, p);
  *bytes = p.total_bytes + p.one_scan_bytes;
  return SLKV_OK;
}

extern "C" slkv_status slkv_recompress_layer(const slkv_ragged_desc* desc, const void* d_qwin, const void* d_k_in,
                                             const void* d_v_in, const int32_t* d_pos_in, void* d_k_out, void* d_v_out,
                                             int32_t* d_kept_idx, int32_t* d_pos_out, int64_t* d_out_offsets,
                                             float* d_importance, float* d_pooled, int64_t out_capacity_rows,
                                             void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  clear_error();
  slkv_status vs = validate_ragged_desc(desc);
  if (vs != SLKV_OK) return vs;
  Geometry g;
  ragged_geometry(desc, g);
  return run_geometry(g, d_qwin, d_k_in, d_v_in, d_pos_in, d_k_out, d_v_out, d_kept_idx, d_pos_out,
                      d_out_offsets, d_importance, d_pooled, out_capacity_rows, d_workspace, workspace_bytes, hip_stream);
}
