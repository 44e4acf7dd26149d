// Multi-source BFS (Section "Multi-Source BFS", Alg. 5) and closeness
// centrality (Section "Closeness Centrality", Eq. 4 and Eq. 5) for gfx950.
//
// kappa = 64 * W concurrent traversals share one pass over the BVSS. Every
// vertex u owns W 64-bit words in each of F (frontier), V (visited) and N
// (marked during Stage 1), stored at getVI(u) = (u mod sigma) * rho +
// floor(u / sigma), rho = number of slice sets, so that consecutive slice
// sets touch consecutive words (the paper's coalescing remap).
//
// Stage 1, top-down over BVSS (E0): a wave takes one queued virtual slice set
// of set s, stages the sigma * W frontier words of s's vertices in LDS, and
// for each slice (row, mask) forms M = OR of the staged words selected by the
// mask bits -- bit c of M is set iff the row has a neighbour in the frontier
// of traversal c, which is what the paper's per-source ballot + binary MMA
// loop computes. Words whose sources are inactive in s (activeSets) are
// skipped; bits already visited are dropped; the rest is OR-ed into N with
// one no-return 64-bit atomic per word, and the row's set is marked dirty.
// Stage 2 then visits dirty slice sets only: new = N & ~V, V |= new, F = new,
// activeSets[s] = OR of the set's new words, the set's VSSs are enqueued when
// nonzero, levels are written, and per-source counts of newly reached
// vertices feed the closeness sums.
// Bottom-up (E2) and dense top-down levels take the gather step instead (its
// own section below): the rows of A one by one, Stage 2 included. Only live
// traversals count there (those whose frontier is non-empty, from the OR of
// all new words): a traversal with an empty frontier can reach nothing more,
// and waiting for its bit (a source in a small component, or one that has
// finished) would turn every early exit into a full adjacency scan.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "device_common.h"
#include "mlp_infer.h"
#include "msbfs.h"
#include "row_pos.h"

namespace blest {

namespace {

constexpr int kWMax = 8;  // up to 512 sources per batch

// LDS words per wave for the top-down engine: the frontier words of one slice
// set (sigma * W), and for sigma = 8 also two 16-entry nibble tables per word
// (32 * W).
template <int SIGMA>
constexpr int ms_lds_words() {
  return (SIGMA == 8 ? SIGMA + 32 : SIGMA) * kWMax;
}

// Statistics of one level: words of a 128-byte line that each XCD's
// workgroups accumulate into by themselves (kMsLive and above by OR, the
// others by addition); readers combine the eight lines.
enum MsStat : int {
  MS_FRESH = 0,    // new (vertex, traversal) pairs
  MS_QUEUE = 1,    // VSSs of the sets that gained a vertex
  MS_QSLICES = 2,  // their slices
  MS_CUMIN = 3,    // pairs visited before this level
  kMsLive = 8,     // + w: OR of the level's new words w (live traversals)
};
static_assert(kMsLive + kWMax <= kMsStatWords, "statistics line");

struct MsBatch {
  int32_t offset;  // first source index of the batch in the call's source list
  int32_t count;   // sources in the batch (<= 64 * W)
  int32_t W;       // 64-bit words per vertex
  int32_t pad;
};

// A call's source list and batch plan travel with the kernel arguments where
// they are this small (512 is the widest batch); otherwise they are copied to
// device memory first, two copies from pageable memory and a synchronisation,
// about 30 us.
constexpr int kMsInlineSrcs = 512, kMsInlineBatches = 8;

struct MsArgs {
  gptr<const int32_t> rp_in;   // in-arcs (the gather step); rp/col for an undirected graph
  gptr<const int32_t> col_in;
  gptr<const int32_t> rows;    // vertices of in-degree > kMsLightDeg, by descending in-degree
  int32_t nrows, nwide, nlong;  // their number; the first nwide have in-degree > kMsWideDeg, the first nlong > kMsLongDeg
  gptr<const uint32_t> slice_ptr;
  gptr<const void> slices;
  gptr<const int32_t> orig_id;
  int64_t n, m, nsets;
  int32_t tau;
  gptr<unsigned long long> F[2];  // frontier words of even and odd levels (valid where the level's front bit is set)
  gptr<unsigned long long> V;
  gptr<unsigned long long> N;
  gptr<unsigned long long> act;
  gptr<uint32_t> fb[3];    // front bits of level l in fb[l % 3]: bit u set iff a traversal reached vertex u at level l
  gptr<uint8_t> dirty;
  gptr<uint4> queue[2];
  gptr<const int32_t> srcs;
  gptr<const MsBatch> batches;
  int32_t nbatches;
  gptr<int16_t> levels16;  // k * n or NULL
  gptr<unsigned long long> planes;  // bit planes of the batch's levels, or NULL: levels16 is written directly
  gptr<const int32_t> perm;  // input id -> internal id, or NULL when not relabelled
  gptr<int64_t> sums;      // k or NULL
  gptr<int64_t> reach;     // k or NULL
  gptr<double> cc;         // k or NULL
  gptr<int64_t> far;       // n (input ids) or NULL: per-target sums of Eq. 4, accumulated
  gptr<long long> part;    // per block: kappa sums then kappa reach counts
  gptr<Ctl> ctl;
  int32_t policy;
  float eta;
  uint64_t seed;
  int64_t nvss, nslices;  // BVSS totals (switch features)
  gptr<const MlpDev> mlp;      // multi-source switch network (policy LEARNED), or NULL
  int32_t probe;          // 1: every level runs both engines from the same state and times each
  gptr<MsLevelRec> log;        // one record per level of the call, or NULL
  int32_t log_cap;
  unsigned long long timeout_ticks;
  int32_t queue_form;     // 1: BVSS levels never take the gather form
  int32_t ablation;       // BLEST_MS_NO_GETVI | BLEST_MS_NO_DIRTY (the paper's ablation steps), else 0
  gptr<unsigned long long> hstat;  // pinned host word: how the launch went
  int32_t fb_words;       // front-bit words the gather keeps in LDS (all of them), or 0: read from memory
  int32_t mlp_shared;     // 1: the switch network's weights lie in the gather's LDS and are reloaded for each level
  int32_t inlined;        // 1: the sources and the plan are these, not srcs and batches
  MsBatch plan_in[kMsInlineBatches];
  int32_t srcs_in[kMsInlineSrcs];
};

__device__ __forceinline__ gptr<const int32_t> ms_srcs(args_ref<MsArgs> a) {
  return a.inlined ? (gptr<const int32_t>)(uintptr_t)&a.srcs_in[0] : a.srcs;
}

__device__ __forceinline__ long long get_vi(long long u, long long rho, int sigma) {
  return (u % sigma) * rho + u / sigma;
}

// Ablation flags: ABL >= 0 is a compile-time value (the full method's kernel
// uses 0, so the flags cost it nothing); ABL = -1 reads them from the arguments.
template <int ABL>
__device__ __forceinline__ int ms_abl(args_ref<MsArgs> a) {
  if constexpr (ABL >= 0)
    return ABL;
  else
    return a.ablation;
}

// Word index of vertex u: getVI order, or u itself in the ablation without it.
template <int ABL>
__device__ __forceinline__ long long ms_vi(args_ref<MsArgs> a, long long u, long long rho, int sigma) {
  return (ms_abl<ABL>(a) & BLEST_MS_NO_GETVI) ? u : get_vi(u, rho, sigma);
}

__device__ __forceinline__ unsigned long long batch_mask(int count, int w) {
  const int lo = w * 64;
  if (count >= lo + 64) return ~0ULL;
  if (count <= lo) return 0ULL;
  return (1ULL << (count - lo)) - 1ULL;
}

__device__ __forceinline__ unsigned long long mix64_ms(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

__device__ __forceinline__ unsigned long long readlane64(unsigned long long x, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(x), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(x >> 32), l);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// Switch inputs of a multi-source level, counted in (vertex, traversal) pairs
// (base-2 logarithms): new pairs and queued slices (absolute), then shares:
// new pairs / all pairs, VSSs / N_v, queued slices / all slices, unvisited
// pairs / all pairs, the batch width, the ratio of the pairs rule
// (log |Q| - log unvisited pairs), live traversals / batch width; three
// reserved zeros.
__device__ __forceinline__ void ms_features(float (&f)[kMaxSwitchFeatures], args_ref<MsArgs> a, long long fresh,
                                            long long qlen, long long qslices, long long unv, int count,
                                            int live) {
  const float pairs = log2f(static_cast<float>(count) * static_cast<float>(a.n));
  const float lu = log2f(1.0f + static_cast<float>(unv));
  f[0] = log2f(1.0f + static_cast<float>(fresh));
  f[1] = log2f(1.0f + static_cast<float>(qslices));
  f[2] = f[0] - pairs;
  f[3] = log2f(1.0f + static_cast<float>(qlen)) - log2f(1.0f + static_cast<float>(a.nvss));
  f[4] = f[1] - log2f(1.0f + static_cast<float>(a.nslices));
  f[5] = lu - pairs;
  f[6] = log2f(static_cast<float>(count));
  f[7] = log2f(1.0f + static_cast<float>(qlen)) - lu;
  f[8] = log2f(static_cast<float>(max(live, 1))) - f[6];
#pragma unroll
  for (int k = 9; k < kMaxSwitchFeatures; ++k) f[k] = 0.0f;
}

// A level's statistics, spread over the lanes of the calling wave: lane t
// holds word t % 16 (get() makes one wave-uniform).
struct MsView {
  unsigned long long raw;
  __device__ __forceinline__ long long get(int t) const { return static_cast<long long>(readlane64(raw, t)); }
  // live traversals: words beyond the batch width stay zero
  __device__ __forceinline__ int live() const {
    int c = 0;
#pragma unroll
    for (int w = 0; w < kWMax; ++w) c += __popcll(readlane64(raw, kMsLive + w));
    return c;
  }
};

__device__ __forceinline__ MsView ms_stats(gptr<Ctl> ctl, int slot) {
  const gptr<const unsigned long long> p = &ctl->ms_acc[slot][0][0];
  const int lane = lane_id();
  const bool add = (lane % kMsStatWords) < kMsLive;
  unsigned long long v = p[lane];
  static_assert(8 * kMsStatWords == 128, "two words per lane");
  const unsigned long long b = p[lane + 64];
  v = add ? v + b : v | b;
#pragma unroll
  for (int d = kMsStatWords; d < 64; d <<= 1) {
    const unsigned long long o = __shfl_xor(v, d, 64);
    v = add ? v + o : v | o;
  }
  return MsView{v};
}

// Workgroup 0 clears one statistics slot and its queue cursor.
__device__ __forceinline__ void ms_clear_slot(gptr<Ctl> ctl, int slot) {
  for (int t = threadIdx.x; t < 8 * kMsStatWords; t += blockDim.x) ctl->ms_acc[slot][0][t] = 0ULL;
  if (threadIdx.x == 0) ctl->acc[slot][F_QUEUE][0] = 0ULL;
}

// Adds a workgroup's statistics (LDS, complete after the barrier inside) to
// its XCD's line of the slot and zeroes them.
__device__ __forceinline__ void ms_publish(gptr<Ctl> ctl, int slot, unsigned xcc, lptr<unsigned long long> s_stat) {
  __syncthreads();
  if (threadIdx.x < kMsStatWords) {
    const unsigned long long v = s_stat[threadIdx.x];
    const gptr<unsigned long long> p = &ctl->ms_acc[slot][xcc][threadIdx.x];
    if (v) {
      if (threadIdx.x < kMsLive)
        add_u64(p, v);
      else
        __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_stat[threadIdx.x] = 0ULL;
    }
  }
}

__device__ __forceinline__ void lds_add(lptr<unsigned long long> p, unsigned long long v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_or(lptr<unsigned long long> p, unsigned long long v) {
  __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Engine of a multi-source level, computed by each wave on its own (every
// input is uniform over the grid). Eq. 3 counted in (vertex, traversal) pairs.
// LEARNED: the switch network (output 0 = BVSS, 2 = bottom-up; anything else,
// or low confidence, falls back to the pairs rule).
__device__ __forceinline__ int ms_choose(args_ref<MsArgs> a, const float (&feat)[kMaxSwitchFeatures], long long qlen, long long unv,
                         int level, int bi, lptr<const float> s_mlp, bool learned, int* fallback) {
  *fallback = 0;
  const int rule = (static_cast<double>(unv) < static_cast<double>(a.eta) * static_cast<double>(qlen))
                       ? BLEST_ENGINE_BOTTOM_UP
                       : BLEST_ENGINE_BVSS;
  switch (a.policy) {
    case BLEST_POLICY_BVSS:
    case BLEST_POLICY_PUSH:
      return BLEST_ENGINE_BVSS;
    case BLEST_POLICY_BOTTOM_UP:
      return BLEST_ENGINE_BOTTOM_UP;
    case BLEST_POLICY_RANDOM:
      return (mix64_ms(a.seed + 0x9E3779B97F4A7C15ULL * static_cast<unsigned long long>(level + 1 + 977 * bi)) & 1ULL)
                 ? BLEST_ENGINE_BOTTOM_UP
                 : BLEST_ENGINE_BVSS;
    case BLEST_POLICY_LEARNED:
      if (learned) {
        const int c = mlp_choose_wave(s_mlp, feat);
        if (c == BLEST_ENGINE_BVSS || c == BLEST_ENGINE_BOTTOM_UP) return c;
      }
      *fallback = 1;
      return rule;
    default:
      return rule;
  }
}

// Sets count int16 values to -1: elementwise up to 16-byte alignment, then
// 16-byte stores, then the tail.
__device__ __forceinline__ void fill_minus_one(gptr<int16_t> p, long long count, long long gtid, long long nthreads) {
  const long long mis = (16 - ((uintptr_t)p & 15)) & 15;
  const long long head = min(count, mis / 2);
  for (long long i = gtid; i < head; i += nthreads) p[i] = -1;
  const long long nvec = (count - head) / 8;
  const gptr<u64x2> v = (gptr<u64x2>)(p + head);
  for (long long i = gtid; i < nvec; i += nthreads) v[i] = u64x2{~0ULL, ~0ULL};
  for (long long i = head + nvec * 8 + gtid; i < count; i += nthreads) p[i] = -1;
}

// Zeroes count 64-bit words (16-byte aligned) with 16-byte stores.
__device__ __forceinline__ void zero_words(gptr<unsigned long long> p, long long count, long long gtid, long long nthreads) {
  const gptr<u64x2> v = (gptr<u64x2>)p;
  for (long long i = gtid; i < count / 2; i += nthreads) v[i] = u64x2{0ULL, 0ULL};
  if (gtid == 0 && (count & 1)) p[count - 1] = 0ULL;
}

// Front bits of a slice set (bit b: vertex s * SIGMA + b).
template <int SIGMA>
__device__ __forceinline__ uint32_t set_bits(gptr<const uint32_t> fb, long long s) {
  return ((gptr<const typename MaskOf<SIGMA>::T>)fb)[s];
}

// What a level reads and writes, the same for both forms of the step.
struct MsStep {
  gptr<const unsigned long long> F;  // frontier words of the level
  gptr<unsigned long long> Fn;       // of the next level
  gptr<const uint32_t> fb;           // front bits of the level
  gptr<uint32_t> fbn;                // of the next level (all zero when the step starts)
  int offset, count, W;              // the batch
  int new_level, slot_out;
};

// Batch bi of the call's plan (bi wave-uniform: scalar loads; the plan is
// written before the launch).
__device__ __forceinline__ MsBatch ms_batch(args_ref<MsArgs> a, int bi) {
  const cptr<const MsBatch> p =
      a.inlined ? (cptr<const MsBatch>)(uintptr_t)&a.plan_in[bi] : (cptr<const MsBatch>)a.batches + bi;
  return MsBatch{p->offset, p->count, p->W, 0};
}

__device__ __forceinline__ MsStep ms_step(args_ref<MsArgs> a, int bi, int level) {
  const MsBatch bt = ms_batch(a, bi);
  return MsStep{a.F[level & 1],      a.F[(level & 1) ^ 1], a.fb[level % 3], a.fb[(level + 1) % 3], bt.offset,
                bt.count,            bt.W,                 level + 1,       (level + 1) % kStatSlots};
}

// ---------------------------------------------------------------- Stage 1

// The calling wave's place among the queue's takers: neighbouring VSSs go to
// different workgroups, so that a queue shorter than the grid's waves keeps
// every compute unit busy instead of 16 waves of a few.
__device__ __forceinline__ long long ms_queue_wave() {
  return static_cast<long long>(wave_in_block()) * gridDim.x + blockIdx.x;
}

template <int SIGMA, class SliceT, int K, int ABL>
__device__ __attribute__((noinline)) void ms_engine_bvss_k(args_ref<MsArgs> a_, int bi, int level, long long qlen,
                                 lptr<unsigned long long> lds_f) {
  args_ref<MsArgs> a = uniform_args(a_);
  bi = uniform(bi);
  level = uniform(level);
  const MsStep sp = ms_step(a, bi, level);
  qlen = uniform(qlen);
  const gptr<const uint4> q = a.queue[level & 1];
  const long long nw = blockDim.x / 64, nwaves = gridDim.x * nw;
  const long long gwave = ms_queue_wave();
  const int W = sp.W;
  const gptr<const SliceT> sl = (gptr<const SliceT>)a.slices;
  const long long rho = a.nsets;
  const int lane = lane_id();
  for (long long i = gwave; i < qlen; i += nwaves) {
    const uint4 d = q[i];
    const uint32_t start = d.x, cnt = d.y;
    const long long s = d.w;
    // Stage the frontier words of the set's sigma vertices (vertex s*SIGMA+b
    // sits at b*rho + s in getVI order); those without a front bit hold words
    // of other levels.
    const uint32_t bits = set_bits<SIGMA>(sp.fb, s);
    for (int j = lane; j < SIGMA * W; j += 64) {
      const int b = j / W, w = j % W;
      const unsigned long long x = sp.F[ms_vi<ABL>(a, s * SIGMA + b, rho, SIGMA) * W + w];
      lds_f[j] = ((bits >> b) & 1u) ? x : 0ULL;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    SliceT sv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t j = static_cast<uint32_t>(lane) + 64u * k;
      sv[k] = (j < cnt) ? sl[start + j] : SliceT(0);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t mask = static_cast<uint32_t>(sv[k] & ((SliceT(1) << SIGMA) - 1));
      if (!mask) continue;
      const long long row = static_cast<long long>(sv[k] >> SliceFmt<SliceT>::kRowShift);
      const long long vi = ms_vi<ABL>(a, row, rho, SIGMA);
      bool any = false;
      for (int w = 0; w < W; ++w) {
        if (!a.act[s * W + w]) continue;
        unsigned long long mw = 0;
        uint32_t t = mask;
        while (t) {
          const int b = __builtin_ctz(t);
          t &= t - 1;
          mw |= lds_f[b * W + w];
        }
        if (!mw) continue;
        mw &= ~a.V[vi * W + w];
        if (mw) {
          __hip_atomic_fetch_or(&a.N[vi * W + w], mw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          any = true;
        }
      }
      if (any) a.dirty[row / SIGMA] = 1;
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// The sigma = 8 form of the engine above, shaped for memory latency. Per VSS
// the slices, the set's frontier words and its activity words are loaded
// together. The frontier words are staged in LDS and expanded into two
// 16-entry tables per word w: lo[i] = OR of the words of the vertices in bit
// subset i of bits 0..3, hi[i] the same for bits 4..7, so a slice's
// neighbour word for w is lo[mask & 15] | hi[mask >> 4] (two LDS reads, where
// the bit loop took up to eight dependent ones). Then, two words at a time
// (one 16-byte load per vertex), the next words of all the lane's K slices
// are loaded at once before any is used, and an atomic OR is issued only for
// bits not yet in them. As in Alg. 5's V_next, a next word holds the visited
// bits plus this level's marks, so this one load filters both; it only grows
// during Stage 1, so a bit seen set needs no OR, and a stale read only costs
// an OR that changes nothing. On this GPU the device-scope ORs, performed at
// the memory side, are what bounds the step. LDS layout per wave: F at [b * W + w], tables at
// [8 W + (h * 16 + i) * W + w].
// (Not inlined: it gets its own register allocation instead of adding to the
// persistent kernel's; its pointers are converted to the global address space.)
template <class SliceT, int K, int ABL>
__device__ __attribute__((noinline)) void ms_engine_bvss8(args_ref<MsArgs> a_, int bi, int level,
                                                          long long qlen, lptr<unsigned long long> lds) {
  args_ref<MsArgs> a = uniform_args(a_);
  bi = uniform(bi);
  level = uniform(level);
  const MsStep sp = ms_step(a, bi, level);
  qlen = uniform(qlen);
  const gptr<const uint4> q = a.queue[level & 1];
  const long long nw = blockDim.x / 64, nwaves = gridDim.x * nw;
  const long long gwave = ms_queue_wave();
  constexpr int SIGMA = 8;
  const int W = sp.W;
  const gptr<const SliceT> sl = (gptr<const SliceT>)a.slices;
  const gptr<const unsigned long long> F = sp.F;
  const gptr<const unsigned long long> act = a.act;
  const gptr<unsigned long long> N = a.N;
  const gptr<uint8_t> dirty = a.dirty;
  const long long rho = a.nsets;
  const int lane = lane_id();
  const lptr<unsigned long long> tab = lds + SIGMA * W;
  for (long long i = gwave; i < qlen; i += nwaves) {
    const uint4 d = q[i];
    const uint32_t start = d.x, cnt = d.y;
    const long long s = d.w;
    SliceT sv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t j = static_cast<uint32_t>(lane) + 64u * k;
      sv[k] = (j < cnt) ? sl[start + j] : SliceT(0);
    }
    unsigned long long fw = 0ULL, aw = 0ULL;
    const uint32_t bits = set_bits<SIGMA>(sp.fb, s);  // vertices without a front bit hold words of other levels
    if (lane < SIGMA * W) fw = F[ms_vi<ABL>(a, s * SIGMA + lane / W, rho, SIGMA) * W + lane % W];
    if (lane < W) aw = act[s * W + lane];
    if (lane < SIGMA * W) lds[lane] = ((bits >> (lane / W)) & 1u) ? fw : 0ULL;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int e = lane; e < 32 * W; e += 64) {
      const int w = e % W, t = e / W;
      const int h = t >> 4, sub = t & 15;
      unsigned long long x = 0ULL;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if ((sub >> b) & 1) x |= lds[(4 * h + b) * W + w];
      tab[e] = x;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    long long vi[K];
    uint32_t m8[K];
    bool any[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      m8[k] = static_cast<uint32_t>(sv[k] & SliceT(0xff));
      vi[k] = ms_vi<ABL>(a, static_cast<long long>(sv[k] >> SliceFmt<SliceT>::kRowShift), rho, SIGMA);
      any[k] = false;
    }
    if (W == 1) {
      if (readlane64(aw, 0)) {
        unsigned long long mw[K], v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) mw[k] = m8[k] ? (tab[m8[k] & 15u] | tab[16u + (m8[k] >> 4)]) : 0ULL;
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = mw[k] ? N[vi[k]] : ~0ULL;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const unsigned long long m = mw[k] & ~v[k];
          if (m) {
            __hip_atomic_fetch_or(&N[vi[k]], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            any[k] = true;
          }
        }
      }
    } else {
      // W is even: words w and w + 1 of a vertex are one aligned 16-byte
      // load (N is 16-byte aligned and vi * W + w is even)
      for (int w = 0; w < W; w += 2) {
        if (!(readlane64(aw, w) | readlane64(aw, w + 1))) continue;
        unsigned long long m0[K], m1[K];
        u64x2 v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          m0[k] = m8[k] ? (tab[(m8[k] & 15u) * W + w] | tab[(16u + (m8[k] >> 4)) * W + w]) : 0ULL;
          m1[k] = m8[k] ? (tab[(m8[k] & 15u) * W + w + 1] | tab[(16u + (m8[k] >> 4)) * W + w + 1]) : 0ULL;
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
          v[k] = (m0[k] | m1[k]) ? *(gptr<const u64x2>)(N + vi[k] * W + w) : u64x2{~0ULL, ~0ULL};
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const unsigned long long x0 = m0[k] & ~v[k].x, x1 = m1[k] & ~v[k].y;
          if (x0) __hip_atomic_fetch_or(&N[vi[k] * W + w], x0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (x1) __hip_atomic_fetch_or(&N[vi[k] * W + w + 1], x1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          any[k] = any[k] || (x0 | x1) != 0ULL;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (any[k]) dirty[(sv[k] >> SliceFmt<SliceT>::kRowShift) / SIGMA] = 1;
    __builtin_amdgcn_wave_barrier();
  }
}

// The same neighbour check as an int8 matrix product on the matrix cores (an
// experiment kept behind opts.ms_mfma; sigma = 8 only). For 16 slices of a VSS
// and 16 traversals c, C = A B with A[i][b] = bit b of slice i's mask and
// B[b][c] = bit c of vertex b's frontier word: C[i][c] > 0 iff row i has a
// neighbour in traversal c's frontier, the count Eq. 2 tests (popc(a & x) > 0).
// One v_mfma_i32_16x16x32_i8 per (16 slices, 16 traversals): K = 32 holds the
// 8 mask bits and 24 zeros; lane l supplies A[l % 16][8 (l / 16) .. + 7] and
// B[8 (l / 16) .. + 7][l % 16], so only lanes 0..15 carry nonzero operands,
// and receives C[4 (l / 16) + r][l % 16] in its r-th result.
typedef int ms_v4i __attribute__((ext_vector_type(4)));

template <class SliceT, int ABL>
__device__ __attribute__((noinline)) void ms_engine_mfma(args_ref<MsArgs> a_, int bi, int level, long long qlen,
                                 lptr<unsigned long long> lds_f) {
  args_ref<MsArgs> a = uniform_args(a_);
  bi = uniform(bi);
  level = uniform(level);
  const MsStep sp = ms_step(a, bi, level);
  qlen = uniform(qlen);
  const gptr<const uint4> q = a.queue[level & 1];
  const long long nw = blockDim.x / 64, nwaves = gridDim.x * nw;
  const long long gwave = ms_queue_wave();
  constexpr int SIGMA = 8;
  const int W = sp.W;
  const gptr<const SliceT> sl = (gptr<const SliceT>)a.slices;
  const long long rho = a.nsets;
  const int lane = lane_id();
  const int c16 = lane & 15;
  const bool carrier = lane < 16;
  for (long long i = gwave; i < qlen; i += nwaves) {
    const uint4 d = q[i];
    const uint32_t start = d.x, cnt = d.y;
    const long long s = d.w;
    const uint32_t bits = set_bits<SIGMA>(sp.fb, s);
    for (int j = lane; j < SIGMA * W; j += 64) {
      const int b = j / W, w = j % W;
      const unsigned long long x = sp.F[ms_vi<ABL>(a, s * SIGMA + b, rho, SIGMA) * W + w];
      lds_f[j] = ((bits >> b) & 1u) ? x : 0ULL;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t t0 = 0; t0 < cnt; t0 += 16) {
      SliceT sw = 0;
      if (carrier && t0 + c16 < cnt) sw = sl[start + t0 + c16];
      const uint32_t mask = static_cast<uint32_t>(sw & SliceT(0xff));
      long afrag = 0;
#pragma unroll
      for (int b = 0; b < 8; ++b) afrag |= static_cast<long>((mask >> b) & 1u) << (8 * b);
      unsigned long long hw[kWMax];
#pragma unroll
      for (int w = 0; w < kWMax; ++w) hw[w] = 0ULL;
      for (int w = 0; w < W; ++w) {
        if (!a.act[s * W + w]) continue;
#pragma unroll
        for (int j4 = 0; j4 < 4; ++j4) {
          long bfrag = 0;
          if (carrier) {
#pragma unroll
            for (int b = 0; b < 8; ++b)
              bfrag |= static_cast<long>((lds_f[b * W + w] >> (16 * j4 + c16)) & 1ULL) << (8 * b);
          }
          ms_v4i c = {0, 0, 0, 0};
          c = __builtin_amdgcn_mfma_i32_16x16x32_i8(afrag, bfrag, c, 0, 0, 0);
          // row i = 4 q + r of the tile holds its 16 bits at [16 q, 16 q + 16) of ballot r
          unsigned long long bal[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) bal[r] = __ballot(c[r] > 0);
          const int rq = c16 >> 2, rr = c16 & 3;
          const unsigned long long br = rr == 0 ? bal[0] : rr == 1 ? bal[1] : rr == 2 ? bal[2] : bal[3];
          hw[w] |= ((br >> (16 * rq)) & 0xffffULL) << (16 * j4);
        }
      }
      if (carrier && mask) {
        const long long row = static_cast<long long>(sw >> SliceFmt<SliceT>::kRowShift);
        const long long vi = ms_vi<ABL>(a, row, rho, SIGMA);
        bool any = false;
        for (int w = 0; w < W; ++w) {
          unsigned long long mw = hw[w];
          if (!mw) continue;
          mw &= ~a.V[vi * W + w];
          if (mw) {
            __hip_atomic_fetch_or(&a.N[vi * W + w], mw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            any = true;
          }
        }
        if (any) a.dirty[row / SIGMA] = 1;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <int SIGMA, class SliceT, bool MF, int ABL>
__device__ __forceinline__ void ms_engine_bvss(args_ref<MsArgs> a, int bi, int level, long long qlen,
                               lptr<unsigned long long> lds_f) {
  if constexpr (MF && SIGMA == 8) {
    ms_engine_mfma<SliceT, ABL>(a, bi, level, qlen, lds_f);
    return;
  }
  if constexpr (SIGMA == 8) {
    switch (a.tau) {
      case 64:
        ms_engine_bvss8<SliceT, 1, ABL>(a, bi, level, qlen, lds_f);
        break;
      case 128:
        ms_engine_bvss8<SliceT, 2, ABL>(a, bi, level, qlen, lds_f);
        break;
      case 192:
        ms_engine_bvss8<SliceT, 3, ABL>(a, bi, level, qlen, lds_f);
        break;
      default:
        ms_engine_bvss8<SliceT, 4, ABL>(a, bi, level, qlen, lds_f);
        break;
    }
    return;
  }
  switch (a.tau) {
    case 64:
      ms_engine_bvss_k<SIGMA, SliceT, 1, ABL>(a, bi, level, qlen, lds_f);
      break;
    case 128:
      ms_engine_bvss_k<SIGMA, SliceT, 2, ABL>(a, bi, level, qlen, lds_f);
      break;
    case 192:
      ms_engine_bvss_k<SIGMA, SliceT, 3, ABL>(a, bi, level, qlen, lds_f);
      break;
    default:
      ms_engine_bvss_k<SIGMA, SliceT, 4, ABL>(a, bi, level, qlen, lds_f);
      break;
  }
}

// ------------------------------------------------------- gather step
//
// The dense form of a level: every vertex with an open (unvisited, live)
// traversal ORs the frontier words of its in-neighbours, row by row of A
// (Eq. 1 read literally; Alg. 4's bottom-up scan for kappa traversals), and
// stops once every open traversal is covered. The row is owned by the lanes
// that scan it, so nothing is marked with atomics, and Stage 2 is done in the
// same pass (FUSED): visited, next-frontier and level words are written once,
// with one device-wide barrier per level instead of two.
//
// What bounds it is the gathers of W-word frontier rows, one per arc to a
// frontier vertex (an arc to any other vertex costs one bit of fb, which a
// scale-18 graph holds in 32 KB), and before their rate the three dependent
// loads to one (column, front bit, frontier row). A row of W words is read by
// W / 2 lanes of 16 bytes each (kRowLanes), so a wave reads kRowsPerWave
// neighbours per load. Four kinds of task, so that every wave has many arcs
// in flight and none is much longer than the rest: kRowsPerWave consecutive
// vertices of in-degree <= kMsLightDeg, a lane group each; two (four) longer
// rows of about the same degree (a list kept with the graph, by descending
// degree), 64 columns of each at a time; one row above kMsLongDeg, 128 (256)
// of its columns at a time; a piece of a row above kMsWideDeg. The tasks of a
// kind are dealt to the workgroups in turn; inside a workgroup each wave
// takes the next one from a counter in LDS (dealt to the waves in turn, the
// slowest wave of a workgroup finished 1.4 times later than its first). The
// row-owner replaces a lane-per-vertex scan whose hub rows (60,000 arcs by
// one lane) took 20 to 66 ms at scale 20.
constexpr int kMsWidePieces = 16;  // tasks a wide row is cut into
template <int W>
constexpr int kRowLanes = W <= 2 ? 1 : W / 2;
template <int W>
constexpr int kRowsPerWave = 64 / kRowLanes<W>;

// N consecutive 32-bit entries from any entry on.
template <int N>
using i32_vec = int __attribute__((ext_vector_type(N), aligned(4)));

// Words 2 sub, 2 sub + 1 of a row (W = 1: its only word and 0).
template <int W>
__device__ __forceinline__ u64x2 load_pair(gptr<const unsigned long long> base, long long vi, int sub) {
  if constexpr (W == 1)
    return u64x2{base[vi], 0ULL};
  else
    return *(gptr<const u64x2>)(base + vi * W + 2 * sub);
}
template <int W>
__device__ __forceinline__ void store_pair(gptr<unsigned long long> base, long long vi, int sub, u64x2 x) {
  if constexpr (W == 1)
    base[vi] = x.x;
  else
    *(gptr<u64x2>)(base + vi * W + 2 * sub) = x;
}

// Lane J of the caller's group of G lanes (a quad permutation).
template <int G, int J>
__device__ __forceinline__ int group_bcast(int v) {
  if constexpr (G == 1)
    return v;
  else if constexpr (G == 2)
    return __builtin_amdgcn_mov_dpp(v, J | (J << 2) | ((2 + J) << 4) | ((2 + J) << 6), 0xf, 0xf, true);
  else
    return __builtin_amdgcn_mov_dpp(v, J * 0x55, 0xf, 0xf, true);
}

// OR of v over the lanes l, l + L, l + 2 L, ... of the wave (L = 1, 2 or 4),
// in every one of them: rotations within 16 lanes, then swaps of 16- and
// 32-lane halves, all of them register moves (no LDS).
template <int L>
__device__ __forceinline__ uint32_t or_slots32(uint32_t v) {
  if constexpr (L <= 1) v |= __builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x121, 0xf, 0xf, true);
  if constexpr (L <= 2) v |= __builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x122, 0xf, 0xf, true);
  v |= __builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x124, 0xf, 0xf, true);
  v |= __builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x128, 0xf, 0xf, true);
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = a[0] | a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return b[0] | b[1];
}
template <int W>
__device__ __forceinline__ u64x2 or_slots(u64x2 x) {
  constexpr int L = kRowLanes<W>;
  auto one = [](unsigned long long q) {
    return (static_cast<unsigned long long>(or_slots32<L>(static_cast<uint32_t>(q >> 32))) << 32) |
           or_slots32<L>(static_cast<uint32_t>(q));
  };
  x.x = one(x.x);
  if (W > 1) x.y = one(x.y);
  return x;
}

// Per-traversal counts of a wave's new bits, bit-sliced: lane l adds its word
// pairs into six carry-save planes (63 additions), flush() adds the planes of
// all lanes holding the same pair and the totals go to LDS counters. About
// one vector instruction per row, where a ballot per traversal took 70.
template <int W>
struct MsCounter {
  static constexpr int P = 6;
  u64x2 c[P];
  int added;
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < P; ++i) c[i] = u64x2{0ULL, 0ULL};
    added = 0;
  }
  __device__ __forceinline__ void flush(lptr<int> cnt) {
    constexpr int L = kRowLanes<W>, R = kRowsPerWave<W>;
    constexpr int T = P + (R == 64 ? 6 : R == 32 ? 5 : 4);
    u64x2 s[T];
#pragma unroll
    for (int i = 0; i < T; ++i) s[i] = i < P ? c[i < P ? i : 0] : u64x2{0ULL, 0ULL};
#pragma unroll
    for (int k = 0; k < T - P; ++k) {
      const int d = L << k;
      u64x2 carry = {0ULL, 0ULL};
#pragma unroll
      for (int i = 0; i < P + k; ++i) {
        const u64x2 x = s[i];
        const u64x2 o = {__shfl_xor(x.x, d, 64), __shfl_xor(x.y, d, 64)};
        const u64x2 t = x ^ o;
        s[i] = t ^ carry;
        carry = (x & o) | (t & carry);
      }
      s[P + k] = carry;
    }
    constexpr int PER = W == 1 ? 1 : 128 / R;  // counters each lane extracts
    const int lane = lane_id(), sub = lane % L, r = lane / L;
#pragma unroll 1
    for (int i = 0; i < PER; ++i) {
      const int t = r * PER + i;
      int v = 0;
#pragma unroll
      for (int j = 0; j < T; ++j)
        v |= static_cast<int>(((t < 64 ? s[j].x : s[j].y) >> (t & 63)) & 1ULL) << j;
      if (v)
        __hip_atomic_fetch_add(cnt + 128 * sub + t, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    clear();
  }
  __device__ __forceinline__ void add(u64x2 x) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const u64x2 t = c[i] & x;
      c[i] ^= x;
      x = t;
    }
    ++added;
  }
  __device__ __forceinline__ bool full() const { return added == (1 << P) - 1; }
};

// LDS of one gather step.
struct MsGatherLds {
  lptr<int> row;                  // 256 ints of the wave: compacted neighbours
  lptr<unsigned long long> wide;  // kWMax words per wide row of the workgroup: the OR of its pieces
  lptr<int> done;                 // finished pieces per wide row
  lptr<int> cnt;                  // 64 * kWMax per-traversal counts
  lptr<unsigned long long> stat;  // kMsStatWords statistics
  lptr<int> next;                 // the workgroup's next task
  lptr<uint32_t> fbits;           // the level's front bits (FL)
};

// FUSED: also Stage 2 of the level; otherwise the marks go to N and the dirty
// flags for ms_finalize. COUNT: per-traversal counts of the new pairs. FL: the
// front bits are read from LDS, where every workgroup copies them first.
template <int SIGMA, int W, int BLOCK, bool FUSED, bool COUNT, bool FL, int ABL>
__device__ __attribute__((noinline)) void ms_gather(args_ref<MsArgs> a_, int bi, int level,
                                                    unsigned long long raw_stats, MsGatherLds lds) {
  args_ref<MsArgs> a = uniform_args(a_);
  bi = uniform(bi);
  level = uniform(level);
  const MsStep sp = ms_step(a, bi, level);
  constexpr int L = kRowLanes<W>, R = kRowsPerWave<W>;
  const int lane = lane_id();
  const int sub = lane % L, r = lane / L;
  const long long rho = a.nsets, n = a.n;
  const long long plane = rho * SIGMA * W;  // words of one level plane
  const gptr<const int32_t> rp = a.rp_in, col = a.col_in, rows = a.rows;
  const gptr<const unsigned long long> F = sp.F;
  const gptr<const uint32_t> fb = sp.fb;
  const gptr<unsigned long long> Fn = sp.Fn, V = a.V, N = a.N;
  const gptr<uint32_t> fbn = sp.fbn;
  const gptr<const uint32_t> slp = a.slice_ptr;
  const gptr<unsigned long long> planes = a.planes;
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  const int new_level = sp.new_level;
  const bool direct = FUSED && a.levels16 != nullptr && a.planes == nullptr;
  const bool overflow = FUSED && a.levels16 != nullptr && new_level > 32767;
  // open traversals of this lane's word pair: in the batch and live
  const int w0 = W == 1 ? 0 : 2 * sub;
  u64x2 bm;
  bm.x = batch_mask(sp.count, w0) & __shfl(raw_stats, kMsLive + w0, 64);
  bm.y = W == 1 ? 0ULL : batch_mask(sp.count, w0 + 1) & __shfl(raw_stats, kMsLive + w0 + 1, 64);

  uint32_t fresh = 0, nq = 0, nqs = 0;
  u64x2 live = {0ULL, 0ULL};
  MsCounter<W> counter;
  if (COUNT) counter.clear();
  // The set whose front bits this lane last ORed into: whether it was the
  // first to do so is read off the returned word one row later, when the
  // atomic has long returned.
  bool pend = false;
  uint32_t pend_old = 0, pend_mask = 0;
  int pend_s = 0;
  auto resolve = [&]() {
    if (pend && !(pend_old & pend_mask)) {
      const uint32_t ns = slp[pend_s + 1] - slp[pend_s];
      nqs += ns;
      nq += (ns + tau - 1) / tau;
    }
    pend = false;
  };
  auto front = [&](int u, uint32_t bits) {  // bits of vertices u, u + 1, ... of one set
    const int s = u / SIGMA;
    pend_s = s;
    pend_mask = (SIGMA == 32 ? ~0u : ((1u << (SIGMA & 31)) - 1u)) << (static_cast<unsigned>(s * SIGMA) & 31u);
    pend_old = __hip_atomic_fetch_or(fbn + (u >> 5), bits << (u & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    pend = true;
  };
  // Writes a finished row: `on` lanes (whole groups) hold the row's visited
  // words v and new words x.
  auto commit = [&](bool on, int u, long long vi, u64x2 v, u64x2 x) {
    if (!on) return;
    const u64x2 vx = v | x;
    if constexpr (!FUSED) {
      store_pair<W>(N, vi, sub, vx);  // N = visited words plus this level's marks
      if (sub == 0) a.dirty[u / SIGMA] = 1;
      return;
    }
    store_pair<W>(V, vi, sub, vx);
    store_pair<W>(N, vi, sub, vx);
    store_pair<W>(Fn, vi, sub, x);
    const uint32_t pc = static_cast<uint32_t>(__popcll(x.x) + __popcll(x.y));
    fresh += pc;
    live |= x;
    if (overflow) {
      __hip_atomic_store(&a.ctl->error[0], static_cast<int>(BLEST_ERR_OVERFLOW), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    } else if (planes) {
      if (pc)
        for (int nl = new_level; nl; nl &= nl - 1) {
          const gptr<unsigned long long> pl = planes + static_cast<long long>(__builtin_ctz(nl)) * plane;
          store_pair<W>(pl, vi, sub, load_pair<W>(pl, vi, sub) | x);
        }
    } else if (direct) {
      const long long o = a.orig_id ? a.orig_id[u] : u;
#pragma unroll
      for (int k = 0; k < (W == 1 ? 1 : 2); ++k) {
        unsigned long long t = k ? x.y : x.x;
        const gptr<int16_t> out = a.levels16 + (static_cast<long long>(sp.offset) + 64 * (w0 + k)) * n + o;
        while (t) {
          const int c = __builtin_ctzll(t);
          t &= t - 1;
          out[c * n] = static_cast<int16_t>(new_level);
        }
      }
    }
    if (a.far) {
      uint32_t s = pc;
      if (L >= 2) s += __shfl_xor(s, 1, 64);
      if (L >= 4) s += __shfl_xor(s, 2, 64);
      if (sub == 0) a.far[a.orig_id ? a.orig_id[u] : u] += static_cast<int64_t>(new_level) * s;
    }
  };
  auto slots = [&](u64x2 x) { return or_slots<W>(x); };  // OR over the lanes that hold the same word pair
  auto is_open = [](u64x2 x) { return (x.x | x.y) != 0ULL; };

  // Scanning rows by the whole wave, 64 columns of each of M pieces per step
  // (piece m: columns P[m] .. E[m]). The front bits of a step's columns are
  // tested together, the frontier ones compacted through LDS so that every
  // lane group has a neighbour to read, and their frontier rows ORed into
  // acc[m] (this lane's part). load_cols() and load_words() take the columns
  // and front words of the first step; scan() also takes those of the next
  // one, `stride` columns on, while the frontier rows are in flight.
  constexpr int M = W == 8 ? 2 : 4;
  constexpr int MP = W == 4 ? 2 : M;  // pieces whose frontier rows are in flight together
  struct Cols {
    int c[M];
    uint32_t w[M];
  };
  auto load_cols = [&](const row_pos (&P)[M], const row_pos (&E)[M], uint32_t ahead, int (&c)[M]) {
#pragma unroll
    for (int m = 0; m < M; ++m)
      c[m] = row_has(P[m], ahead + lane, E[m]) ? col[P[m] + (ahead + lane)] : -1;
  };
  auto front_word = [&](int c) -> uint32_t {
    if constexpr (FL)
      return lds.fbits[c >> 5];
    else
      return fb[c >> 5];
  };
  auto load_words = [&](Cols& k) {
#pragma unroll
    for (int m = 0; m < M; ++m) k.w[m] = k.c[m] >= 0 ? front_word(k.c[m]) : 0u;
  };
  auto scan = [&](const row_pos (&P)[M], const row_pos (&E)[M], uint32_t stride, Cols& k, u64x2 (&acc)[M]) {
    Cols nx;
    load_cols(P, E, stride, nx.c);
    int na[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const bool hit = (k.w[m] >> (k.c[m] & 31)) & 1u;
      if constexpr (L == 1) {
        if (!hit) k.c[m] = -1;
      } else {
        const unsigned long long b = __ballot(hit);
        na[m] = __popcll(b);
        if (hit)
          lds.row[64 * m + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32),
                                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u))] = k.c[m];
      }
    }
    if constexpr (L > 1) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
#pragma unroll
    for (int pass = 0; pass < M / MP; ++pass) {
      u64x2 f[MP][L];
#pragma unroll
      for (int kk = 0; kk < MP; ++kk)
#pragma unroll
        for (int q = 0; q < L; ++q) {
          const int m = pass * MP + kk;
          int cv = -1;
          if constexpr (L == 1)
            cv = k.c[m];
          else if (q * R + r < na[m])
            cv = lds.row[64 * m + q * R + r];
          f[kk][q] = cv >= 0 ? load_pair<W>(F, ms_vi<ABL>(a, cv, rho, SIGMA), sub) : u64x2{0ULL, 0ULL};
        }
      if (pass == M / MP - 1) load_words(nx);
#pragma unroll
      for (int kk = 0; kk < MP; ++kk)
#pragma unroll
        for (int q = 0; q < L; ++q) acc[pass * MP + kk] |= f[kk][q];
    }
    if constexpr (L > 1) __builtin_amdgcn_wave_barrier();
    k = nx;
  };
  auto group = [&](bool b) {  // any lane of the caller's group
    const unsigned long long t = __ballot(b);
    return L == 1 ? b : ((t >> (r * L)) & ((1ULL << L) - 1ULL)) != 0ULL;
  };

  // The workgroup's tasks: its share of the wide rows (kMsWidePieces pieces
  // each), of the long rows, of the groups of M medium rows and of the chunks
  // of R vertices.
  const int grid = static_cast<int>(gridDim.x), me = static_cast<int>(blockIdx.x);
  auto share = [&](long long total) { return total > me ? static_cast<int>((total - 1 - me) / grid + 1) : 0; };
  const int twide = share(a.nwide) * kMsWidePieces;
  const int tlong = twide + share(a.nlong - a.nwide);
  const int tmed = tlong + share((a.nrows - a.nlong + M - 1) / M);
  const int tall = tmed + share((n + R - 1) / R);
  // Round k's chunks are dealt in another order of the workgroups each time,
  // so that positions which recur at a fixed stride in the vertex order (a
  // relabelling that puts each window's long rows first) go round them: dealt
  // always in the same order, the slowest workgroup took 3.5 times as long as
  // the fastest one on scale-20 R-MAT.
  const int rounds = static_cast<int>((n + R - 1) / R) / grid;  // full ones; the last, partial round keeps its order
  const int p2 = 1 << (31 - __builtin_clz(static_cast<unsigned>(grid)));  // largest power of two up to grid
  auto take = [&]() {
    int t = 0;
    if (lane == 0) t = __hip_atomic_fetch_add(lds.next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return uniform(t);
  };
  // What a task reads first: this lane group's vertex (-1: none), its columns
  // and its visited words. The next task's are loaded before the current one
  // is worked on.
  struct Head {
    int u;
    row_pos p0, p1;
  };
  auto head = [&](int t) {
    Head h{-1, 0, 0};
    if (t < tmed) {
      const long long i = t < twide   ? me + static_cast<long long>(t / kMsWidePieces) * grid
                          : t < tlong ? a.nwide + me + static_cast<long long>(t - twide) * grid
                                      : a.nlong + (me + static_cast<long long>(t - tlong) * grid) * M + r;
      if (r < M && i < a.nrows) h.u = rows[i];
    } else if (t < tall) {
      const int k = t - tmed;
      const int b = k < rounds && me < p2 ? me ^ ((37 * k) & (p2 - 1)) : me;
      const long long u = (static_cast<long long>(k) * grid + b) * R + r;
      if (u < n) h.u = static_cast<int>(u);
    }
    if (h.u >= 0) {
      h.p0 = rp[h.u];
      h.p1 = rp[h.u + 1];
    }
    return h;
  };
  auto visited = [&](int u) {
    return u >= 0 ? load_pair<W>(V, ms_vi<ABL>(a, u, rho, SIGMA), sub) : u64x2{~0ULL, ~0ULL};
  };
  for (int i = threadIdx.x; i < kMsWideSlots * kWMax; i += BLOCK) lds.wide[i] = 0ULL;
  if (threadIdx.x < kMsWideSlots) lds.done[threadIdx.x] = 0;
  if (threadIdx.x == 0) *lds.next = 0;
  if constexpr (FL) {
    // 16 bytes per thread and load, four loads in flight (the buffer and the
    // LDS copy are padded to 16 bytes)
    const gptr<const u32x4> src = (gptr<const u32x4>)fb;
    const lptr<u32x4> dst = (lptr<u32x4>)lds.fbits;
    const int nv = (a.fb_words + 3) / 4;
    for (int i0 = threadIdx.x; i0 < nv; i0 += 4 * BLOCK) {
      u32x4 q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i0 + j * BLOCK < nv) q[j] = src[i0 + j * BLOCK];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i0 + j * BLOCK < nv) dst[i0 + j * BLOCK] = q[j];
    }
  }
  __syncthreads();
  int t = take();
  Head cur = head(t);
  u64x2 v = visited(cur.u);
  while (t < tall) {
    const int tn = take();
    const Head nxt = head(tn);
    const u64x2 op = ~v & bm;
    u64x2 x = {0ULL, 0ULL};
    if (t < tlong) {
      // One row, or a piece of a wide one, 64 M columns per step; every slot
      // holds the row, slot 0 writes it. The pieces of a wide row meet in
      // LDS; the wave that adds the last one goes on with the whole row.
      const bool open = __ballot(is_open(op)) != 0ULL;
      row_pos p = __builtin_amdgcn_readlane(cur.p0, 0), pe = __builtin_amdgcn_readlane(cur.p1, 0);
      const int slot = t / kMsWidePieces;
      if (t < twide) {
        const uint32_t len = row_piece_len(p, pe, kMsWidePieces);
        p += (t % kMsWidePieces) * len;
        pe = row_part_end(p, len, pe);
      }
      if (open) {
        row_pos P[M], E[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
          P[m] = p + 64 * m;
          E[m] = pe;
        }
        Cols k;
        load_cols(P, E, 0, k.c);
        load_words(k);
        while (P[0] < pe) {
          u64x2 acc[M];
#pragma unroll
          for (int m = 0; m < M; ++m) acc[m] = u64x2{0ULL, 0ULL};
          scan(P, E, 64 * M, k, acc);
#pragma unroll
          for (int m = 0; m < M; ++m) {
            x |= acc[m];
            P[m] += 64 * M;
          }
          x = slots(x);
          if (!__ballot(is_open(op & ~x))) break;
        }
      }
      if (t < twide) {
        if (r == 0) {
          if (x.x) lds_or(lds.wide + slot * kWMax + w0, x.x);
          if (W > 1 && x.y) lds_or(lds.wide + slot * kWMax + w0 + 1, x.y);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        int d = 0;
        if (lane == 0) d = __hip_atomic_fetch_add(lds.done + slot, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        x = u64x2{0ULL, 0ULL};
        if (uniform(d) == kMsWidePieces - 1) {
          x.x = lds.wide[slot * kWMax + w0];
          if (W > 1) x.y = lds.wide[slot * kWMax + (W > 1 ? w0 + 1 : 0)];
        }
      }
      x = r == 0 ? x & op : u64x2{0ULL, 0ULL};
    } else if (t < tmed) {
      // M rows (neighbours in the list, so of about the same degree), 64
      // columns of each per step; slot m writes row m
      const bool open = group(is_open(op));
      row_pos P[M], E[M];
      u64x2 acc[M];
      bool more = false;
#pragma unroll
      for (int m = 0; m < M; ++m) {
        P[m] = __builtin_amdgcn_readlane(cur.p0, m * L);
        E[m] = __builtin_amdgcn_readlane(open ? cur.p1 : cur.p0, m * L);
        acc[m] = u64x2{0ULL, 0ULL};
        more |= P[m] < E[m];
      }
      if (more) {
        Cols k;
        load_cols(P, E, 0, k.c);
        load_words(k);
        while (more) {
          scan(P, E, 64, k, acc);
          more = false;
#pragma unroll
          for (int m = 0; m < M; ++m) {
            P[m] += 64;
            acc[m] = slots(acc[m]);
            if (P[m] < E[m] && !__ballot(r == m && is_open(op & ~acc[m]))) E[m] = P[m];  // covered
            more |= P[m] < E[m];
          }
        }
#pragma unroll
        for (int m = 0; m < M; ++m)
          if (r == m) x = acc[m] & op;
      }
    } else {
      // R consecutive vertices, a lane group each, 8 columns (4 where a lane
      // is a whole group) of each per step. Columns are loaded two steps
      // ahead and their front bits one, so a step waits for one round of
      // frontier rows.
      constexpr int G = L == 1 ? 4 : 8 / L, STEP = G * L;
      row_pos p = cur.p0;
      const row_pos p1 = cur.p1 - cur.p0 > kMsLightDeg ? cur.p0 : cur.p1;  // longer rows are in the lists above
      bool run = group(is_open(op)) && p < p1;
      if (__ballot(run)) {
        // a lane's G consecutive columns in one load (they may start at any
        // entry; col is padded by 4): G loads of one column each, spread over
        // R rows, kept the address unit busy for most of a sparse level
        auto columns = [&](row_pos q, int (&c)[G]) {
          const row_pos i = q + G * sub;
          i32_vec<G> x;
#pragma unroll
          for (int g = 0; g < G; ++g) x[g] = -1;
          if (run && i < p1) x = *(gptr<const i32_vec<G>>)(col + i);
#pragma unroll
          for (int g = 0; g < G; ++g) c[g] = row_has(i, g, p1) ? x[g] : -1;
        };
        auto words = [&](const int (&c)[G], uint32_t (&w)[G]) {
#pragma unroll
          for (int g = 0; g < G; ++g) w[g] = c[g] >= 0 ? front_word(c[g]) : 0u;
        };
        int c0[G], c1[G];
        uint32_t fw[G];
        columns(p, c0);
        columns(p + STEP, c1);
        words(c0, fw);
        for (;;) {
#pragma unroll
          for (int g = 0; g < G; ++g)
            if (!run || !((fw[g] >> (c0[g] & 31)) & 1u)) c0[g] = -1;
          u64x2 f[G][L];
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const int cv[4] = {group_bcast<L, 0>(c0[g]), group_bcast<L, (L > 1 ? 1 : 0)>(c0[g]),
                               group_bcast<L, (L > 2 ? 2 : 0)>(c0[g]), group_bcast<L, (L > 2 ? 3 : 0)>(c0[g])};
#pragma unroll
            for (int q = 0; q < L; ++q)
              f[g][q] = cv[q] >= 0 ? load_pair<W>(F, ms_vi<ABL>(a, cv[q], rho, SIGMA), sub) : u64x2{0ULL, 0ULL};
          }
          words(c1, fw);
#pragma unroll
          for (int g = 0; g < G; ++g) c0[g] = c1[g];
          columns(p + 2 * STEP, c1);
#pragma unroll
          for (int g = 0; g < G; ++g)
#pragma unroll
            for (int q = 0; q < L; ++q) x |= f[g][q];
          p += STEP;
          const bool left = group(is_open(op & ~x));
          run = run && left && p < p1;
          if (!__ballot(run)) break;
        }
        x &= op;
      }
    }
    const bool any = group(is_open(x));
    const int u = cur.u;
    const u64x2 vu = v;
    const bool chunk = t >= tmed;
    t = tn;
    cur = nxt;
    v = visited(nxt.u);
    if (__ballot(any)) {
      commit(any, u, any ? ms_vi<ABL>(a, u, rho, SIGMA) : 0, vu, x);
      if (FUSED) {
        resolve();
        if (chunk) {
          // front bits of the wave's vertices, a set (or the part of it) per lane
          const unsigned long long b64 = __ballot(any);
          const unsigned long long bits = __ballot(lane < R && ((b64 >> (lane * L)) & 1ULL));
          constexpr int S = SIGMA < R ? SIGMA : R;
          const int u0 = __builtin_amdgcn_readlane(u, 0);
          if (lane < R / S) {
            const uint32_t b = static_cast<uint32_t>((bits >> (lane * S)) & ((1ULL << S) - 1ULL));
            if (b) front(u0 + lane * S, b);
          }
        } else if (any && sub == 0) {
          front(u, 1u);
        }
        if (COUNT) counter.add(x);
      }
    }
    if (COUNT && (counter.full() || (t >= tall && counter.added))) counter.flush(lds.cnt);
  }
  if constexpr (FUSED) {
    resolve();
    const unsigned long long sf = wave_sum(static_cast<unsigned long long>(fresh));
    if (sf) {  // uniform in the wave
      const unsigned long long sq = wave_sum(static_cast<unsigned long long>(nq)), ss = wave_sum(static_cast<unsigned long long>(nqs));
      live = slots(live);
      if (lane == 0) {
        lds_add(lds.stat + MS_FRESH, sf);
        const bool track = !(ms_abl<ABL>(a) & BLEST_MS_NO_DIRTY);
        if (sq && track) lds_add(lds.stat + MS_QUEUE, sq);
        if (ss && track) lds_add(lds.stat + MS_QSLICES, ss);
      }
      if (r == 0) {
        if (live.x) lds_or(lds.stat + kMsLive + w0, live.x);
        if (W > 1 && live.y) lds_or(lds.stat + kMsLive + w0 + 1, live.y);
      }
    }
  }
}

template <int SIGMA, int BLOCK, bool FUSED, int ABL>
__device__ __forceinline__ void ms_gather_any(args_ref<MsArgs> a, int bi, int level, int W, const MsView& st,
                                              const MsGatherLds& lds, bool count) {
  constexpr bool FL = SIGMA == 8 && FUSED && ABL == 0;  // kernels that may hold the front bits in LDS
  auto go = [&](auto width) {
    constexpr int WW = decltype(width)::value;
    if (FL && a.fb_words && count)
      ms_gather<SIGMA, WW, BLOCK, FUSED, FUSED, FL, ABL>(a, bi, level, st.raw, lds);
    else if (FL && a.fb_words)
      ms_gather<SIGMA, WW, BLOCK, FUSED, false, FL, ABL>(a, bi, level, st.raw, lds);
    else if (FUSED && count)
      ms_gather<SIGMA, WW, BLOCK, FUSED, FUSED, false, ABL>(a, bi, level, st.raw, lds);
    else
      ms_gather<SIGMA, WW, BLOCK, FUSED, false, false, ABL>(a, bi, level, st.raw, lds);
  };
  switch (W) {
    case 1:
      return go(std::integral_constant<int, 1>{});
    case 2:
      return go(std::integral_constant<int, 2>{});
    case 4:
      return go(std::integral_constant<int, 4>{});
    default:
      return go(std::integral_constant<int, 8>{});
  }
}

// ---------------------------------------------------------------- Stage 2

// Copies a finished batch's levels to the caller's rows: levels16[(offset +
// c) * n + v] = level of input vertex v in traversal c, -1 if the traversal
// did not reach it. The levels were kept as bit planes: plane j holds bit j
// of every (vertex, traversal) level, in the layout of the visited words
// (a vertex's row of W words per plane), so a level's writes are whole rows
// and a vertex costs W * 8 bytes per plane instead of 128 W of int16.
// Thread t handles input ids v = t, t + nthreads, ...: a lane reads its
// vertex's rows of Q words per plane at once (a word at a time, the rows of
// the workgroup's lanes would leave the L1 between words), and a pair of
// lanes exchanges values so that each stores both vertices of one traversal:
// one 4-byte store per lane covers 128 bytes of two traversals' rows.
// P: planes read (those past np are zero).
typedef uint32_t u32_half_aligned __attribute__((aligned(2)));

template <int SIGMA, int ABL, int P, int Q>
__device__ __attribute__((noinline)) void ms_copy_planes(args_ref<MsArgs> a_, int bi, int np) {
  args_ref<MsArgs> a = uniform_args(a_);
  bi = uniform(bi);
  np = uniform(np);
  const MsBatch bt = ms_batch(a, bi);
  const long long nthreads = static_cast<long long>(gridDim.x) * blockDim.x;
  const int lane = lane_id();
  const int W = bt.W;
  const long long n = a.n, rho = a.nsets;
  const long long plane = rho * SIGMA * W;
  const int count = bt.count;
  const gptr<const unsigned long long> V = a.V, planes = a.planes;
  const gptr<int16_t> out = a.levels16 + static_cast<long long>(bt.offset) * n;
  const gptr<const int32_t> perm = a.perm;
  // whole waves: the lanes of a pair both take part in every exchange
  for (long long base = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x - lane; base < n;
       base += nthreads) {
    const long long v = base + lane;
    const bool in = v < n;
    const long long i = in ? (perm ? perm[v] : v) : 0;
    const long long vi = ms_vi<ABL>(a, i, rho, SIGMA) * W;
    const bool odd = lane & 1;
    const bool pair = (v | 1) < n;  // both vertices of the pair exist
    for (int q0 = 0; q0 < W && 64 * q0 < count; q0 += Q) {
      unsigned long long nv[Q], pl[P][Q];
#pragma unroll
      for (int k = 0; k < Q; ++k) nv[k] = q0 + k < W ? ~V[vi + q0 + k] : 0ULL;
#pragma unroll
      for (int j = 0; j < P; ++j)
#pragma unroll
        for (int k = 0; k < Q; ++k) pl[j][k] = j < np && q0 + k < W ? planes[j * plane + vi + q0 + k] : 0ULL;
#pragma unroll
      for (int k = 0; k < Q; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c0 = 64 * (q0 + k) + 32 * h;
          if (c0 >= count) continue;
          const uint32_t u = static_cast<uint32_t>(nv[k] >> (32 * h));
          uint32_t p[P];
#pragma unroll
          for (int j = 0; j < P; ++j) p[j] = static_cast<uint32_t>(pl[j][k] >> (32 * h));
          gptr<int16_t> o = out + static_cast<long long>(c0 + (odd && pair ? 1 : 0)) * n + (pair ? base + (lane & ~1) : v);
          const int cn = min(32, count - c0);
          auto emit2 = [&](int c) {
            // both traversals' levels of this vertex, 0xffff where not reached
            uint32_t lv = ((u >> c) & 1u ? 0xffffu : 0u) | ((u >> (c + 1)) & 1u ? 0xffff0000u : 0u);
#pragma unroll
            for (int j = 0; j < P; ++j) {
              const uint32_t t = p[j] >> c;
              lv |= ((t & 1u) | ((t & 2u) << 15)) << j;
            }
            const uint32_t ot = static_cast<uint32_t>(
                __builtin_amdgcn_mov_dpp(static_cast<int>(lv), 0xb1, 0xf, 0xf, true));  // the pair's other lane
            if (pair) {
              const uint32_t w = odd ? (lv & 0xffff0000u) | (ot >> 16) : (lv & 0xffffu) | (ot << 16);
              if (c + (odd ? 1 : 0) < cn) *(gptr<u32_half_aligned>)o = w;
            } else if (in) {
              o[0] = static_cast<int16_t>(lv & 0xffffu);
              if (c + 1 < cn) o[n] = static_cast<int16_t>(lv >> 16);
            }
            o += 2 * n;
          };
          if (cn == 32) {
#pragma unroll
            for (int c = 0; c < 32; c += 2) emit2(c);
          } else {
#pragma unroll 1
            for (int c = 0; c < cn; c += 2) emit2(c);
          }
        }
    }
  }
}

// last: the batch's deepest level.
template <int SIGMA, int ABL>
__device__ __forceinline__ void ms_copy_levels(args_ref<MsArgs> a, int bi, int last) {
  const int np = last > 0 ? 32 - __builtin_clz(static_cast<unsigned>(last)) : 0;
  if (np <= 4)
    ms_copy_planes<SIGMA, ABL, 4, 8>(a, bi, np);
  else if (np <= 8)
    ms_copy_planes<SIGMA, ABL, 8, 4>(a, bi, np);
  else
    ms_copy_planes<SIGMA, ABL, kMsPlanes, 2>(a, bi, np);
}

struct MsExpandRec {
  unsigned long long out;
  uint32_t n, s0, ns, s;
};
constexpr int kMsExpandMin = 8;
constexpr int kMsMaxExpand = 128;

// LDS of ms_append.
template <int BLOCK>
struct MsAppendLds {
  int scan[BLOCK / 64];
  unsigned long long base;
  MsExpandRec rec[kMsMaxExpand];
  int nrec;
};

// Appends the nq VSSs of each calling thread's slice set s (slices s0 .. s0 +
// ns) to the queue; cursor is its length. Called by the whole workgroup;
// L.nrec must be zero before (visible to all) and is zero after.
template <int BLOCK>
__device__ __forceinline__ void ms_append(gptr<uint4> queue, gptr<unsigned long long> cursor, uint32_t tau, int nq, uint32_t s0,
                                          uint32_t ns, long long s, MsAppendLds<BLOCK>& L) {
  int v1[1] = {nq}, ex1[1], tot1[1];
  block_exclusive_scan<BLOCK, 1>(v1, ex1, tot1, L.scan);
  if (threadIdx.x == 0) L.base = tot1[0] ? fetch_add_u64(cursor, tot1[0]) : 0ULL;
  __syncthreads();
  const long long oq = static_cast<long long>(L.base) + ex1[0];
  if (nq > kMsExpandMin) {
    const int r = atomicAdd(&L.nrec, 1);
    if (r < kMsMaxExpand) {
      L.rec[r] = MsExpandRec{static_cast<unsigned long long>(oq), static_cast<uint32_t>(nq), s0, ns,
                             static_cast<uint32_t>(s)};
      nq = 0;
    }
  }
  for (int k2 = 0; k2 < nq; ++k2) {
    const uint32_t off = static_cast<uint32_t>(k2) * tau;
    queue[oq + k2] = make_uint4(s0 + off, min(tau, ns - off), 0u, static_cast<uint32_t>(s));
  }
  __syncthreads();
  const int nr = min(L.nrec, kMsMaxExpand);
  for (int r = 0; r < nr; ++r) {
    const MsExpandRec e = L.rec[r];
    for (uint32_t i = threadIdx.x; i < e.n; i += BLOCK) {
      const uint32_t off = i * tau;
      queue[e.out + i] = make_uint4(e.s0 + off, min(tau, e.ns - off), 0u, e.s);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) L.nrec = 0;
  __syncthreads();
}

// Slice sets that a workgroup takes at a time in a sweep over all of them: one
// a thread, or fewer (whole waves) where that leaves workgroups without any.
template <int BLOCK>
__device__ __forceinline__ int ms_sweep_sets(long long nsets) {
  const long long share = (nsets + gridDim.x - 1) / gridDim.x;
  return static_cast<int>(min((share + 63) / 64 * 64, static_cast<long long>(BLOCK)));
}

// The queue and the activity words of a level whose frontier a gather step
// (or the seeding) wrote, for a level that the queue form takes.
template <int SIGMA, int BLOCK, int ABL>
__device__ __attribute__((noinline)) void ms_emit(args_ref<MsArgs> a_, int W, int level) {
  args_ref<MsArgs> a = uniform_args(a_);
  W = uniform(W);
  level = uniform(level);
  __shared__ MsAppendLds<BLOCK> L;
  if (threadIdx.x == 0) L.nrec = 0;
  const bool track = !(ms_abl<ABL>(a) & BLEST_MS_NO_DIRTY);
  const gptr<const unsigned long long> F = a.F[level & 1];
  const gptr<const uint32_t> fb = a.fb[level % 3];
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  const long long rho = a.nsets;
  const int per = ms_sweep_sets<BLOCK>(rho);
  for (long long base = static_cast<long long>(blockIdx.x) * per; base < rho;
       base += static_cast<long long>(gridDim.x) * per) {
    const long long s = base + threadIdx.x;
    const bool in = static_cast<int>(threadIdx.x) < per && s < rho;
    const uint32_t bits = in ? set_bits<SIGMA>(fb, s) : 0u;
    const bool mine = in && (bits || !track);
    if (!__syncthreads_or(mine)) continue;
    uint32_t s0 = 0, ns = 0;
    int nq = 0;
    if (mine) {
      for (int w = 0; w < W; ++w) {
        unsigned long long x = 0ULL;
        for (uint32_t t = bits; t; t &= t - 1)
          x |= F[ms_vi<ABL>(a, s * SIGMA + __builtin_ctz(t), rho, SIGMA) * W + w];
        a.act[s * W + w] = track ? x : ~0ULL;
      }
      s0 = a.slice_ptr[s];
      ns = a.slice_ptr[s + 1] - s0;
      nq = static_cast<int>((ns + tau - 1) / tau);
    }
    ms_append<BLOCK>(a.queue[level & 1], &a.ctl->acc[level % kStatSlots][F_QUEUE][0], tau, nq, s0, ns, s, L);
  }
}

// Stage 2 of a queue level: every dirty slice set.
template <int SIGMA, int BLOCK, int ABL>
__device__ __attribute__((noinline)) void ms_finalize(args_ref<MsArgs> a_, int bi, int level, lptr<int> lds_cnt,
                                                      lptr<unsigned long long> s_stat, bool count_sources) {
  args_ref<MsArgs> a = uniform_args(a_);
  bi = uniform(bi);
  level = uniform(level);
  const MsStep sp = ms_step(a, bi, level);
  __shared__ MsAppendLds<BLOCK> L;
  if (threadIdx.x == 0) L.nrec = 0;
  const int W = sp.W, new_level = sp.new_level;
  const long long rho = a.nsets;
  const long long plane = rho * SIGMA * W;
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  const int lane = lane_id();
  constexpr int VG = 8;  // vertices of a set handled together (their words stay in registers)
  unsigned long long fresh = 0, qs = 0, nqs = 0;
  const bool overflow = a.levels16 != nullptr && new_level > 32767;
  // Without dynamic slice-set tracking (an ablation step) every set is
  // finalised at every level, all its words count as active and all its
  // VSSs are queued.
  const bool track = !(ms_abl<ABL>(a) & BLEST_MS_NO_DIRTY);
  const int per = ms_sweep_sets<BLOCK>(a.nsets);
  for (long long base = static_cast<long long>(blockIdx.x) * per; base < a.nsets;
       base += static_cast<long long>(gridDim.x) * per) {
    const long long s = base + threadIdx.x;
    const bool mine = static_cast<int>(threadIdx.x) < per && s < a.nsets && (!track || a.dirty[s]);
    if (!__syncthreads_or(mine)) continue;
    int nq = 0;
    uint32_t s0 = 0, ns = 0, fbits = 0;
    if (mine) a.dirty[s] = 0;
    if (__ballot(mine)) {
      for (int w = 0; w < W; ++w) {
        unsigned long long Aw = 0ULL;
        int cnt_c = 0;  // lane c: new vertices of traversal w*64+c in this wave
#pragma unroll 1
        for (int b0 = 0; b0 < SIGMA; b0 += VG) {
          // N holds the visited words plus this level's marks (Alg. 5's
          // V_next); the new bits are its difference from V. All words of
          // the group are loaded before any store (the stores would
          // otherwise order each vertex's loads after the previous vertex's).
          unsigned long long dw[VG], nx[VG];
          long long idx[VG];
#pragma unroll
          for (int b = 0; b < VG; ++b) {
            idx[b] = ms_vi<ABL>(a, s * SIGMA + b0 + b, rho, SIGMA) * W + w;
            nx[b] = mine ? a.N[idx[b]] : 0ULL;
            dw[b] = mine ? a.V[idx[b]] : 0ULL;
          }
#pragma unroll
          for (int b = 0; b < VG; ++b) {
            const unsigned long long dd = nx[b] & ~dw[b];
            if (mine) {
              if (dd) a.V[idx[b]] = nx[b];
              sp.Fn[idx[b]] = dd;
            }
            dw[b] = dd;
            Aw |= dd;
            fbits |= dd ? 1u << (b0 + b) : 0u;
            fresh += __popcll(dd);
          }
          if (Aw && overflow) {
            __hip_atomic_store(&a.ctl->error[0], static_cast<int>(BLEST_ERR_OVERFLOW), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          } else if (a.planes && new_level > 0) {
            for (int nl = new_level; nl; nl &= nl - 1) {
              const gptr<unsigned long long> pl = a.planes + static_cast<long long>(__builtin_ctz(nl)) * plane;
              unsigned long long pv[VG];
#pragma unroll
              for (int b = 0; b < VG; ++b) pv[b] = dw[b] ? pl[idx[b]] : 0ULL;
#pragma unroll
              for (int b = 0; b < VG; ++b)
                if (dw[b]) pl[idx[b]] = pv[b] | dw[b];
            }
          } else if (a.levels16) {
            // direct: for each traversal c with new vertices in this set, the
            // set's vertices in c's output row (scattered when relabelled)
            unsigned long long any = 0ULL;
#pragma unroll
            for (int b = 0; b < VG; ++b) any |= dw[b];
            while (any) {
              const int c = __builtin_ctzll(any);
              any &= any - 1;
              const gptr<int16_t> out = a.levels16 + (static_cast<long long>(sp.offset) + w * 64 + c) * a.n;
#pragma unroll
              for (int b = 0; b < VG; ++b)
                if ((dw[b] >> c) & 1ULL) {
                  const long long u = s * SIGMA + b0 + b;
                  out[a.orig_id ? a.orig_id[u] : u] = static_cast<int16_t>(new_level);
                }
            }
          }
          if (a.far && mine && new_level > 0) {
            // Eq. 4: far[u] += level * (traversals reaching u at this level);
            // the thread owns set s, so no other thread updates these vertices
#pragma unroll
            for (int b = 0; b < VG; ++b)
              if (dw[b]) {
                const long long u = s * SIGMA + b0 + b;
                a.far[a.orig_id ? a.orig_id[u] : u] += static_cast<int64_t>(new_level) * __popcll(dw[b]);
              }
          }
          // Per-source counts of new vertices: lane c accumulates traversal
          // w*64+c by a ballot over the wave's lanes (vertical popcount).
          if (count_sources) {
#pragma unroll
            for (int b = 0; b < VG; ++b)
              if (__ballot(dw[b] != 0ULL))
                for (int c = 0; c < 64; ++c) {
                  const int pc = __popcll(__ballot((dw[b] >> c) & 1ULL));
                  if (lane == c) cnt_c += pc;
                }
          }
        }
        if (mine) a.act[s * W + w] = track ? Aw : ~0ULL;
        if (Aw & ~s_stat[kMsLive + w]) lds_or(s_stat + kMsLive + w, Aw);
        if (cnt_c) __hip_atomic_fetch_add(lds_cnt + w * 64 + lane, cnt_c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    if (mine && fbits) ((gptr<typename MaskOf<SIGMA>::T>)sp.fbn)[s] = static_cast<typename MaskOf<SIGMA>::T>(fbits);
    if (mine && (fbits || !track)) {
      s0 = a.slice_ptr[s];
      ns = a.slice_ptr[s + 1] - s0;
      nq = static_cast<int>((ns + tau - 1) / tau);
      qs += ns;
      nqs += static_cast<unsigned long long>(nq);
    }
    // enqueue the VSSs of every set that gained a vertex in some traversal
    ms_append<BLOCK>(a.queue[new_level & 1], &a.ctl->acc[sp.slot_out][F_QUEUE][0], tau, nq, s0, ns, s, L);
  }
  const unsigned long long sf = wave_sum(fresh), sq = wave_sum(nqs), ss = wave_sum(qs);
  if (lane == 0) {
    if (sf) lds_add(s_stat + MS_FRESH, sf);
    if (sq) lds_add(s_stat + MS_QUEUE, sq);
    if (ss) lds_add(s_stat + MS_QSLICES, ss);
  }
}

// ------------------------------------------------------------- batches

// LDS every multi-source kernel needs: the queue engine's tables (f), in whose
// place the gather step has 256 ints per wave of compacted neighbours and then
// the front bits. DYN: that region is dynamic LDS, sized by the host
// (ms_dynamic_lds).
constexpr int kMsRowWords = 128;  // 64-bit words of a wave's compacted neighbours
template <int SIGMA, int BLOCK, bool DYN>
struct MsLds {
  unsigned long long f[DYN ? 1 : (BLOCK / 64) * ms_lds_words<SIGMA>()];
  unsigned long long wide[kMsWideSlots * kWMax];
  int done[kMsWideSlots];
  unsigned long long stat[kMsStatWords];
  int cnt[64 * kWMax];
  int next;
};

template <int SIGMA, int BLOCK, bool DYN>
__device__ __forceinline__ void ms_lds_init(MsLds<SIGMA, BLOCK, DYN>& s) {
  for (int c = threadIdx.x; c < 64 * kWMax; c += BLOCK) s.cnt[c] = 0;
  if (threadIdx.x < kMsStatWords) s.stat[threadIdx.x] = 0ULL;
  __syncthreads();
}

// region: the LDS of the queue engine's tables.
template <int SIGMA, int BLOCK, bool DYN>
__device__ __forceinline__ MsGatherLds ms_gather_lds(MsLds<SIGMA, BLOCK, DYN>& s, lptr<unsigned long long> region) {
  static_assert(ms_lds_words<SIGMA>() >= kMsRowWords, "the gather compacts up to 256 columns per wave");
  return MsGatherLds{(lptr<int>)(region + wave_in_block() * kMsRowWords), to_lds(s.wide), to_lds(s.done),
                     to_lds(s.cnt), to_lds(s.stat), to_lds(&s.next),
                     (lptr<uint32_t>)(region + (BLOCK / 64) * kMsRowWords)};
}

// Clears what a batch starts from: visited and next words, the front bits,
// the first level plane, its sources' rows of the level-0 frontier words (the
// other rows are read only where a front bit is set), its level rows when
// they are written directly, the partial sums and the statistics.
template <int SIGMA, int ABL>
__device__ __attribute__((noinline)) void ms_batch_clear(args_ref<MsArgs> a_, int bi, bool count_sources) {
  args_ref<MsArgs> a = uniform_args(a_);
  const MsBatch bt = ms_batch(a, uniform(bi));
  const long long nthreads = static_cast<long long>(gridDim.x) * blockDim.x;
  const long long gtid = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int W = bt.W;
  const long long nhat = a.nsets * SIGMA;
  zero_words(a.V, nhat * W, gtid, nthreads);
  zero_words(a.N, nhat * W, gtid, nthreads);
  if (a.planes) zero_words(a.planes, nhat * W, gtid, nthreads);
  for (int b = 0; b < 3; ++b)
    for (long long i = gtid; i < (nhat + 31) / 32; i += nthreads) a.fb[b][i] = 0u;
  for (long long i = gtid; i < static_cast<long long>(bt.count) * W; i += nthreads)
    a.F[0][ms_vi<ABL>(a, ms_srcs(a)[bt.offset + i / W], a.nsets, SIGMA) * W + i % W] = 0ULL;
  if (a.levels16 && !a.planes)
    fill_minus_one(a.levels16 + static_cast<long long>(bt.offset) * a.n, static_cast<long long>(bt.count) * a.n, gtid,
                   nthreads);
  if (count_sources) {
    const gptr<long long> part = a.part + static_cast<long long>(blockIdx.x) * (2 * 64 * kWMax);
    for (int c = threadIdx.x; c < 2 * 64 * kWMax; c += blockDim.x) part[c] = 0;
  }
  if (blockIdx.x == 0)
    for (int t = 0; t < kStatSlots; ++t) ms_clear_slot(a.ctl, t);
}

// Level 0: every source in its own traversal's bit, and its statistics.
template <int SIGMA, int ABL>
__device__ __attribute__((noinline)) void ms_batch_seed(args_ref<MsArgs> a_, int bi, unsigned xcc) {
  args_ref<MsArgs> a = uniform_args(a_);
  const MsBatch bt = ms_batch(a, uniform(bi));
  const long long nthreads = static_cast<long long>(gridDim.x) * blockDim.x;
  const long long gtid = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  using M = typename MaskOf<SIGMA>::T;
  const bool track = !(ms_abl<ABL>(a) & BLEST_MS_NO_DIRTY);
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  const gptr<unsigned long long> st = &a.ctl->ms_acc[0][xcc][0];
  for (long long c = gtid; c < bt.count; c += nthreads) {
    const long long u = ms_srcs(a)[bt.offset + c];
    const long long i = ms_vi<ABL>(a, u, a.nsets, SIGMA) * bt.W + c / 64;
    const unsigned long long bit = 1ULL << (c % 64);
    __hip_atomic_fetch_or(a.V + i, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_or(a.N + i, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_or(a.F[0] + i, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a.planes == nullptr && a.levels16) a.levels16[(bt.offset + c) * a.n + (a.orig_id ? a.orig_id[u] : u)] = 0;
    const uint32_t old = __hip_atomic_fetch_or(a.fb[0] + (u >> 5), 1u << (u & 31), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
    const long long s = u / SIGMA;
    if (track && !static_cast<M>(old >> ((s * SIGMA) & 31))) {  // the set's first source
      const uint32_t ns = a.slice_ptr[s + 1] - a.slice_ptr[s];
      add_u64(st + MS_QUEUE, (ns + tau - 1) / tau);
      add_u64(st + MS_QSLICES, ns);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    add_u64(st + MS_FRESH, static_cast<unsigned long long>(bt.count));
    if (!track) {
      add_u64(st + MS_QUEUE, static_cast<unsigned long long>(a.nvss));
      add_u64(st + MS_QSLICES, static_cast<unsigned long long>(a.nslices));
    }
    for (int w = 0; w < bt.W; ++w)
      __hip_atomic_fetch_or(st + kMsLive + w, batch_mask(bt.count, w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Housekeeping of the step that builds level new_level: the statistics slot
// and the front bits that the step after it accumulates into, and the level
// plane whose first writer is that step.
template <int SIGMA>
__device__ __attribute__((noinline)) void ms_prepare_next(args_ref<MsArgs> a_, int W, int new_level) {
  args_ref<MsArgs> a = uniform_args(a_);
  W = uniform(W);
  new_level = uniform(new_level);
  const long long nthreads = static_cast<long long>(gridDim.x) * blockDim.x;
  const long long gtid = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  const long long nhat = a.nsets * SIGMA;
  if (blockIdx.x == 0) ms_clear_slot(a.ctl, (new_level + 1) % kStatSlots);
  const gptr<uint32_t> fbz = a.fb[(new_level + 1) % 3];
  for (long long i = gtid; i < (nhat + 31) / 32; i += nthreads) fbz[i] = 0u;
  const unsigned nx = static_cast<unsigned>(new_level) + 1u;
  if (a.planes && !(nx & (nx - 1u)) && nx < (1u << kMsPlanes)) {
    const long long words = nhat * W;
    zero_words(a.planes + static_cast<long long>(__builtin_ctz(nx)) * words, words, gtid, nthreads);
  }
}

// Adds a level's per-traversal counts to the workgroup's partial sums: sum +=
// level * count, reach += count.
__device__ __forceinline__ void ms_flush_counts(args_ref<MsArgs> a, lptr<int> cnt, int W, int new_level) {
  __syncthreads();
  const gptr<long long> part = a.part + static_cast<long long>(blockIdx.x) * (2 * 64 * kWMax);
  for (int c = threadIdx.x; c < 64 * W; c += blockDim.x) {
    const int x = cnt[c];
    if (x) {
      part[c] += static_cast<long long>(new_level) * x;
      part[64 * kWMax + c] += x;
      cnt[c] = 0;
    }
  }
}

// Sums the workgroups' partials of a batch, one wave per source (a lane per
// workgroup, so a source costs one round of loads instead of a chain of one
// per workgroup). Each source reaches itself at level 0.
__device__ __attribute__((noinline)) void ms_reduce_batch(args_ref<MsArgs> a_, int bi) {
  args_ref<MsArgs> a = uniform_args(a_);
  const MsBatch bt = ms_batch(a, uniform(bi));
  const long long nw = blockDim.x / 64, nwaves = gridDim.x * nw;
  const long long gwave = blockIdx.x * nw + wave_in_block();
  const gptr<const long long> part = a.part;
  const int lane = lane_id();
  for (long long c = gwave; c < bt.count; c += nwaves) {
    long long su = 0, re = 0;
    for (unsigned b = lane; b < gridDim.x; b += 64) {
      su += part[b * (2LL * 64 * kWMax) + c];
      re += part[b * (2LL * 64 * kWMax) + 64 * kWMax + c];
    }
    su = wave_sum(su);
    re = wave_sum(re) + 1;
    if (lane == 0) {
      const long long row = bt.offset + c;
      if (a.sums) a.sums[row] = su;
      if (a.reach) a.reach[row] = re;
      if (a.cc) a.cc[row] = su ? static_cast<double>(re - 1) / static_cast<double>(su) : 0.0;
    }
  }
}

// A level whose queue holds at least 1 / kMsDenseDenom of the graph's arcs as
// slices takes the gather step, which reads at most the arcs of the vertices
// still open; one with fewer the queue form of a BVSS step, unless even so the
// gather step is the quicker. A gather step takes 14 us (16 K vertices) and up
// to 18 more with the vertices (256 K and beyond), and 1 us per 250,000 arcs of
// open vertices; a level by the queue about 65 with what it adds to its
// neighbours (a list of its own, a second pass, two more barriers). The batch
// width moves both sides alike: closeness of 64, 128, 256 and 512 sources, plain
// method, on uniform graphs of mean degree 4 and 16 (30 K to 4 M vertices), grids
// (29 K to 1 M) and R-MAT of scale 15 to 22 takes by this rule at most 4% longer
// than with every level gathered or every level queued, and up to 18% less. (64
// sources, us by the rule, all gathered, all queued: 250 K vertices of degree 4
// 503, 504, 1,184; 490 K grid 35,640, 35,910, 75,800; scale 22 3,080, 3,740, 4,240.
// With 28 in the place of 65, and 53 from 2,048 slices on, 569, 38,550 and 3,080.)
constexpr long long kMsDenseDenom = 128;
constexpr float kMsQueueLevelUs = 65.0f;
__device__ __forceinline__ bool ms_gather_quicker(long long n, long long m, float open_part) {
  return 14.0f + fminf(static_cast<float>(n) * (1.0f / 13000.0f), 18.0f) +
             static_cast<float>(m) * (1.0f / 250000.0f) * open_part <=
         kMsQueueLevelUs;
}

// What a level does, from its statistics alone (the same in every wave).
struct MsChoice {
  bool dense;    // a BVSS step takes the gather form
  int engine, fallback;
  __device__ __forceinline__ bool gather() const { return dense || engine == BLEST_ENGINE_BOTTOM_UP; }
};

// Writes the level's record: workgroup 0, one lane of its first wave.
__device__ __forceinline__ void ms_log(args_ref<MsArgs> a, int nrec, int bi, int level, int width, const MsChoice& ch,
                                       long long fresh, long long qlen, long long qslices, long long unv, int live,
                                       const float (&feat)[kMaxSwitchFeatures]) {
  if (!a.log || nrec >= a.log_cap || lane_id() != 0) return;
  const gptr<MsLevelRec> rec = a.log + nrec;
  rec->batch = bi;
  rec->level = level;
  rec->engine = a.probe ? -1 : ch.engine;
  rec->gather = a.probe ? ch.dense : ch.gather();
  rec->fallback = ch.fallback;
  rec->width = width;
  rec->live = live;
  rec->fresh = fresh;
  rec->queue = qlen;
  rec->qslices = qslices;
  rec->unvisited = unv;
  rec->t_engine[0] = rec->t_engine[1] = 0ULL;
  for (int k = 0; k < kMaxSwitchFeatures; ++k) rec->feat[k] = feat[k];
}

// Whether a level takes the gather step whatever its engine.
__device__ __forceinline__ bool ms_dense(args_ref<MsArgs> a, const MsView& st, int count) {
  if (a.queue_form) return false;
  const long long slices = st.get(MS_QSLICES), all = static_cast<long long>(count) * a.n;
  const long long unv = all - st.get(MS_CUMIN) - st.get(MS_FRESH);
  return slices * kMsDenseDenom >= a.m ||
         ms_gather_quicker(a.n, a.m, static_cast<float>(unv) / static_cast<float>(all));
}

// Decides level `level` and logs it. The engine of a dense level changes
// nothing but its record (both engines take the gather form), so there only
// the last workgroup's first wave, which writes the record, evaluates it (the
// last has the fewest tasks, and workgroup 0 clears the next counters).
template <int ABL, bool MF>
__device__ __attribute__((noinline)) int ms_decide_level(args_ref<MsArgs> a_, unsigned long long raw_stats, int bi,
                                                         int level, int nrec, lptr<const float> s_mlp,
                                                         bool learned) {
  args_ref<MsArgs> a = uniform_args(a_);
  bi = uniform(bi);
  level = uniform(level);
  nrec = uniform(nrec);
  const MsView st{raw_stats};
  const MsBatch bt = ms_batch(a, bi);
  const long long fresh = st.get(MS_FRESH), qlen = st.get(MS_QUEUE), qslices = st.get(MS_QSLICES);
  const long long unv = static_cast<long long>(bt.count) * a.n - st.get(MS_CUMIN) - fresh;
  MsChoice ch{!MF && ms_abl<ABL>(a) == 0 && ms_dense(a, st, bt.count), BLEST_ENGINE_BVSS, 0};
  const bool writer = blockIdx.x == gridDim.x - 1 && wave_in_block() == 0;
  if (!ch.dense || writer) {
    float feat[kMaxSwitchFeatures];
    const int live = st.live();
    ms_features(feat, a, fresh, qlen, qslices, unv, bt.count, live);
    ch.engine = ms_choose(a, feat, qlen, unv, level, bi, s_mlp, learned, &ch.fallback);
    if (writer) ms_log(a, nrec, bi, level, bt.count, ch, fresh, qlen, qslices, unv, live, feat);
  }
  return (ch.dense ? 1 : 0) | (ch.engine << 1);
}

template <int ABL, bool MF>
__device__ __forceinline__ MsChoice ms_decide(args_ref<MsArgs> a, const MsView& st, int bi, int level, int nrec,
                                              lptr<const float> s_mlp, bool learned) {
  const int c = uniform(ms_decide_level<ABL, MF>(a, st.raw, bi, level, nrec, s_mlp, learned));
  return MsChoice{(c & 1) != 0, c >> 1, 0};
}

// Thread 0 of workgroup 0 adds what no workgroup counts: the pairs visited
// before the new level and, without slice-set tracking, the totals of the
// queue (every set counts) when the step was not a queue level.
template <int ABL>
__device__ __forceinline__ void ms_level_end(args_ref<MsArgs> a, const MsView& st, bool finalized, lptr<unsigned long long> s_stat) {
  if (blockIdx.x != 0 || wave_in_block() != 0) return;
  const long long cum = st.get(MS_CUMIN) + st.get(MS_FRESH);
  if (threadIdx.x == 0) {
    lds_add(s_stat + MS_CUMIN, static_cast<unsigned long long>(cum));
    if ((ms_abl<ABL>(a) & BLEST_MS_NO_DIRTY) && !finalized) {
      lds_add(s_stat + MS_QUEUE, static_cast<unsigned long long>(a.nvss));
      lds_add(s_stat + MS_QSLICES, static_cast<unsigned long long>(a.nslices));
    }
  }
}

// ------------------------------------------------------------- kernel

// MODE 0: the full method with the bitwise check; 1: the check on the matrix
// cores; 10 + f: the bitwise check with ablation flags f (each a kernel of its
// own, so no variant's branches or registers weigh on another).
template <int SIGMA, class SliceT, int BLOCK, int MODE = 0>
__global__ void __launch_bounds__(BLOCK) k_ms_persistent(MsArgs args) {
  args_ref<MsArgs> a = kernel_args(args);
  constexpr bool MF = MODE == 1;
  constexpr int ABL = MODE >= 10 ? MODE - 10 : 0;
  constexpr int GABL = MODE >= 10 ? -1 : 0;  // the gather's: one body for all ablation kernels
  extern __shared__ __attribute__((aligned(16))) float s_mlp[];
  // dynamic LDS: the switch network (learned policy), then the tables or front bits
  constexpr bool DYN = SIGMA == 8 && MODE == 0;
  __shared__ MsLds<SIGMA, BLOCK, DYN> lds;
  const lptr<unsigned long long> region =
      DYN ? (lptr<unsigned long long>)to_lds(s_mlp + (a.policy == BLEST_POLICY_LEARNED && !a.mlp_shared ? kLdsMlpFloats : 0))
          : to_lds(lds.f);
  static_assert(kLdsMlpFloats % 4 == 0, "the region is 16-byte aligned");
  const bool learned = a.policy == BLEST_POLICY_LEARNED && a.mlp != nullptr && a.mlp->valid;
  if (learned) mlp_to_lds((const MlpDev*)a.mlp, s_mlp);
  const int wave = wave_in_block();
  const lptr<unsigned long long> my_f = region + wave * ms_lds_words<SIGMA>();
  const MsGatherLds glds = ms_gather_lds(lds, region);
  const bool count_sources = a.sums != nullptr || a.reach != nullptr || a.cc != nullptr;
  ms_lds_init(lds);
  if (blockIdx.x == 0 && threadIdx.x == 0) host_status_begin(a.hstat);
  BarrierCtx bc;
  if (!barrier_register((Ctl*)a.ctl, &bc, a.timeout_ticks)) return;
  int total_levels = 0;
  int nrec = 0;  // level records written so far (the same count in every workgroup)
  for (int bi = 0; bi < a.nbatches; ++bi) {
    const MsBatch bt = ms_batch(a, bi);
    ms_batch_clear<SIGMA, ABL>(a, bi, count_sources);
    if (!grid_barrier((Ctl*)a.ctl, bc)) return;
    ms_batch_seed<SIGMA, ABL>(a, bi, bc.xcc);
    if (!grid_barrier((Ctl*)a.ctl, bc)) return;
    bool listed = false;  // the level's queue and activity words exist
    int level = 0;
    for (;; ++level) {
      const MsView st = ms_stats(a.ctl, level % kStatSlots);
      if (st.get(MS_FRESH) == 0) break;
      // (only the last workgroup evaluates the network at a dense level)
      const bool reload = DYN && learned && a.mlp_shared && (blockIdx.x == gridDim.x - 1 || !ms_dense(a, st, bt.count));
      if (reload) {
        mlp_to_lds((const MlpDev*)a.mlp, s_mlp);
        __syncthreads();
      }
      const MsChoice ch =
          ms_decide<ABL, MF>(a, st, bi, level, nrec, to_lds((const float*)s_mlp), learned);
      if (reload) __syncthreads();  // every wave has read the weights
      const gptr<MsLevelRec> rec = (a.log && nrec < a.log_cap) ? a.log + nrec : nullptr;
      ++nrec;
      ms_prepare_next<SIGMA>(a, bt.W, level + 1);
      const bool gather = ch.gather();
      const bool queued = !ch.dense && (a.probe || !gather);  // the queue form runs
      if (queued && !listed) {
        ms_emit<SIGMA, BLOCK, ABL>(a, bt.W, level);
        if (!grid_barrier((Ctl*)a.ctl, bc)) return;
      }
      const long long qlen = st.get(MS_QUEUE);
      if (a.probe) {
        // both engines from the same state, each in the form it takes at this
        // level: their marks are the same set. At a dense level both take the
        // gather step, so one run times both.
        const unsigned long long t0 = dev_ticks();
        if (queued) {
          ms_engine_bvss<SIGMA, SliceT, MF, ABL>(a, bi, level, qlen, my_f);
          if (!grid_barrier((Ctl*)a.ctl, bc)) return;
        }
        const unsigned long long t1 = queued ? dev_ticks() : t0;
        ms_gather_any<SIGMA, BLOCK, false, GABL>(a, bi, level, bt.W, st, glds, false);
        if (!grid_barrier((Ctl*)a.ctl, bc)) return;
        if (blockIdx.x == 0 && threadIdx.x == 0 && rec) {
          const unsigned long long t2 = dev_ticks();
          rec->t_engine[0] = (queued ? t1 : t2) - t0;  // (the same run where not queued)
          rec->t_engine[1] = t2 - t1;
        }
      } else if (gather) {
        ms_gather_any<SIGMA, BLOCK, true, GABL>(a, bi, level, bt.W, st, glds, count_sources);
      } else {
        ms_engine_bvss<SIGMA, SliceT, MF, ABL>(a, bi, level, qlen, my_f);
        if (!grid_barrier((Ctl*)a.ctl, bc)) return;
      }
      listed = a.probe || !gather;
      if (listed) ms_finalize<SIGMA, BLOCK, ABL>(a, bi, level, glds.cnt, glds.stat, count_sources);
      if (count_sources) ms_flush_counts(a, glds.cnt, bt.W, level + 1);
      ms_level_end<ABL>(a, st, listed, glds.stat);
      ms_publish(a.ctl, (level + 1) % kStatSlots, bc.xcc, glds.stat);
      if (!grid_barrier((Ctl*)a.ctl, bc)) return;
    }
    total_levels = max(total_levels, level);
    if (a.planes && a.ctl->error[0] == 0) ms_copy_levels<SIGMA, ABL>(a, bi, level - 1);
    if (count_sources) ms_reduce_batch(a, bi);
    if (!grid_barrier((Ctl*)a.ctl, bc)) return;
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x < 8) a.ctl->xcd_blocks[threadIdx.x][0] = 0u;
    if (threadIdx.x == 8) a.ctl->xcd_active[0] = 0u;
    if (threadIdx.x == 0) {
      a.ctl->nlevels[0] = total_levels;
      a.ctl->ms_nrec[0] = nrec;
      host_status_end(a.hstat, a.ctl, total_levels);
    }
  }
}

// ------------------------------------------------ hipGraph-captured levels
//
// The same traversal as k_ms_persistent, cut into one kernel per grid-wide
// phase so that a fixed sequence of launches can be captured in a hipGraph
// and replayed: the kernel's work is chosen by a state {phase, batch, level,
// records, listed} in the control block. Kernel i of a graph reads state slot
// i % 2 and workgroup 0 writes the next state to the other slot (the next
// kernel starts only after every workgroup of this one has finished, so no
// workgroup reads a slot while it is being written). After the last batch the
// phase is MS_DONE and the remaining kernels of a replay do nothing.
enum MsPhase : int { MS_INIT = 0, MS_SEED = 1, MS_LEVEL = 2, MS_FIN = 3, MS_END = 4, MS_DONE = 5 };
constexpr int kMsGraphKernels = 32;  // kernels per graph (even)
static_assert(sizeof(MsDev::gnode) / sizeof(hipGraphNode_t) == kMsGraphKernels, "one node handle per kernel");

template <int SIGMA, class SliceT, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_ms_phase(MsArgs args, int parity) {
  args_ref<MsArgs> a = kernel_args(args);
  constexpr int ABL = -1;
  extern __shared__ float s_mlp[];
  __shared__ MsLds<SIGMA, BLOCK, false> lds;
  const int phase = a.ctl->ms_state[parity][0];
  const int bi = uniform(a.ctl->ms_state[parity][1]);
  const int level = uniform(a.ctl->ms_state[parity][2]);
  const int nrec = a.ctl->ms_state[parity][3];
  const int listed = a.ctl->ms_state[parity][4];
  int next[5] = {MS_DONE, bi, level, nrec, 0};
  if (phase != MS_DONE) {
    const int wave = wave_in_block();
    const lptr<unsigned long long> my_f = to_lds(lds.f) + wave * ms_lds_words<SIGMA>();
    const MsGatherLds glds = ms_gather_lds(lds, to_lds(lds.f));
    const unsigned xcc = xcc_id();
    const bool count_sources = a.sums != nullptr || a.reach != nullptr || a.cc != nullptr;
    ms_lds_init(lds);
    const MsBatch bt = ms_batch(a, bi);
    switch (phase) {
      case MS_INIT:
        ms_batch_clear<SIGMA, ABL>(a, bi, count_sources);
        next[0] = MS_SEED;
        break;
      case MS_SEED:
        ms_batch_seed<SIGMA, ABL>(a, bi, xcc);
        next[0] = MS_LEVEL;
        next[2] = 0;
        break;
      case MS_LEVEL: {
        const MsView st = ms_stats(a.ctl, level % kStatSlots);
        if (st.get(MS_FRESH) == 0) {
          next[0] = MS_END;
          break;
        }
        const bool learned = a.policy == BLEST_POLICY_LEARNED && a.mlp != nullptr && a.mlp->valid;
        if (learned) {
          mlp_to_lds((const MlpDev*)a.mlp, s_mlp);
          __syncthreads();
        }
        const MsChoice ch = ms_decide<ABL, false>(a, st, bi, level, nrec, to_lds((const float*)s_mlp), learned);
        const bool gather = ch.gather();
        if (!gather && !listed) {
          ms_emit<SIGMA, BLOCK, ABL>(a, bt.W, level);
          next[0] = MS_LEVEL;
          next[4] = 1;
          break;
        }
        next[3] = nrec + 1;
        ms_prepare_next<SIGMA>(a, bt.W, level + 1);
        if (gather) {
          ms_gather_any<SIGMA, BLOCK, true, ABL>(a, bi, level, bt.W, st, glds, count_sources);
          if (count_sources) ms_flush_counts(a, glds.cnt, bt.W, level + 1);
          ms_level_end<ABL>(a, st, false, glds.stat);
          ms_publish(a.ctl, (level + 1) % kStatSlots, xcc, glds.stat);
          next[0] = MS_LEVEL;
          next[2] = level + 1;
        } else {
          ms_engine_bvss<SIGMA, SliceT, false, ABL>(a, bi, level, st.get(MS_QUEUE), my_f);
          next[0] = MS_FIN;
        }
        break;
      }
      case MS_FIN: {
        const MsView st = ms_stats(a.ctl, level % kStatSlots);
        ms_finalize<SIGMA, BLOCK, ABL>(a, bi, level, glds.cnt, glds.stat, count_sources);
        if (count_sources) ms_flush_counts(a, glds.cnt, bt.W, level + 1);
        ms_level_end<ABL>(a, st, true, glds.stat);
        ms_publish(a.ctl, (level + 1) % kStatSlots, xcc, glds.stat);
        next[0] = MS_LEVEL;
        next[2] = level + 1;
        next[4] = 1;
        break;
      }
      default:  // MS_END
        if (a.planes && a.ctl->error[0] == 0) ms_copy_levels<SIGMA, ABL>(a, bi, level - 1);
        if (count_sources) ms_reduce_batch(a, bi);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
          if (level > a.ctl->nlevels[0]) a.ctl->nlevels[0] = level;
          a.ctl->ms_nrec[0] = nrec;
        }
        next[0] = bi + 1 < a.nbatches ? MS_INIT : MS_DONE;
        next[1] = bi + 1;
        next[2] = 0;
        break;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0)
    for (int i = 0; i < 5; ++i) a.ctl->ms_state[parity ^ 1][i] = next[i];
}

__global__ void k_ms_start(Ctl* ctl, unsigned long long* hstat) {
  if (threadIdx.x == 0) {
    host_status_begin(to_global(hstat));  // (stays 0: the host reads the control block after graph replays)
    for (int i = 0; i < 5; ++i) ctl->ms_state[0][i] = 0;  // MS_INIT, batch 0
    ctl->nlevels[0] = 0;
    ctl->ms_nrec[0] = 0;
  }
}

// One workgroup of 16 waves per compute unit: the gather step is bound by the
// latency of its loads, so it wants as many waves as 128 registers allow, and
// the device-wide barrier wants few workgroups.
constexpr int kMsBlock = 1024;

template <int SIGMA, class SliceT>
const void* ms_phase_fn() {
  return reinterpret_cast<const void*>(&k_ms_phase<SIGMA, SliceT, kMsBlock>);
}

template <int SIGMA, class SliceT>
const void* ms_fn() {
  return reinterpret_cast<const void*>(&k_ms_persistent<SIGMA, SliceT, kMsBlock>);
}

constexpr int kMsLogCap = 1 << 16;  // level records per call

const void* ms_kernel(const DevGraph& g) {
  // the matrix-core check and the ablation steps are kernels of their own, so
  // their registers and branches never weigh on the full method's kernel
  if (g.ms_mfma && g.sigma == 8)
    return g.wide ? reinterpret_cast<const void*>(&k_ms_persistent<8, uint64_t, kMsBlock, 1>)
                  : reinterpret_cast<const void*>(&k_ms_persistent<8, uint32_t, kMsBlock, 1>);
  if (g.ms_ablation && g.sigma == 8) {
    if (g.wide)
      return g.ms_ablation == 1   ? reinterpret_cast<const void*>(&k_ms_persistent<8, uint64_t, kMsBlock, 11>)
             : g.ms_ablation == 2 ? reinterpret_cast<const void*>(&k_ms_persistent<8, uint64_t, kMsBlock, 12>)
                                  : reinterpret_cast<const void*>(&k_ms_persistent<8, uint64_t, kMsBlock, 13>);
    return g.ms_ablation == 1   ? reinterpret_cast<const void*>(&k_ms_persistent<8, uint32_t, kMsBlock, 11>)
           : g.ms_ablation == 2 ? reinterpret_cast<const void*>(&k_ms_persistent<8, uint32_t, kMsBlock, 12>)
                                : reinterpret_cast<const void*>(&k_ms_persistent<8, uint32_t, kMsBlock, 13>);
  }
  if (g.sigma == 8 && !g.wide) return ms_fn<8, uint32_t>();
  if (g.sigma == 8) return ms_fn<8, uint64_t>();
  if (g.sigma == 16) return ms_fn<16, uint64_t>();
  return ms_fn<32, uint64_t>();
}

void ms_graph_destroy(MsDev* ms) {
  if (ms->gexec) (void)hipGraphExecDestroy(ms->gexec);
  if (ms->graph) (void)hipGraphDestroy(ms->graph);
  ms->gexec = nullptr;
  ms->graph = nullptr;
  ms->gfn = nullptr;
  for (auto& nd : ms->gnode) nd = nullptr;
}

// Dynamic LDS of the persistent kernel, and whether its gather steps read the
// front bits from there (a.fb_words): when they fit beside the compaction rows,
// up to 1.07 M vertices. (From 0.91 M on the switch network's weights lie in the
// same place and are loaded again before each decision, 2 us.) The test of an
// arc is then one LDS read instead of one of the up to 64 cache lines of a
// wave's load. First gather level of 64 to 512 traversals on a 1 M vertex R-MAT
// (30 M arcs): 236, 238, 285 and 381 us with the bits in memory, 153, 152, 199
// and 286 in LDS; on 256 K vertices (32 KB of bits, as much as the vector L1)
// 90 and 80. A level pays the copy, 2 to 3 us for 128 KB.
unsigned ms_dynamic_lds(const DevGraph& g, const MsDev& ms, int policy, MsArgs* a) {
  const unsigned mlp = policy == BLEST_POLICY_LEARNED ? kLdsMlpFloats * sizeof(float) : 0u;
  a->fb_words = 0;
  a->mlp_shared = 0;
  if (g.sigma != 8 || g.ms_mfma || g.ms_ablation) return mlp;  // these kernels' tables are static
  constexpr unsigned waves = kMsBlock / 64;
  const unsigned tables = mlp + waves * ms_lds_words<8>() * 8u;
  const int64_t words = (g.nsets * g.sigma + 31) / 32;
  const int64_t front = waves * kMsRowWords * 8u + 16 * ((words + 3) / 4);
  const int64_t room = g.max_lds - static_cast<int64_t>(ms.static_lds);
  if (a->probe || front > room) return tables;
  a->fb_words = static_cast<int32_t>(words);
  a->mlp_shared = mlp + front > room;
  return std::max(a->mlp_shared ? tables - mlp : tables, static_cast<unsigned>(a->mlp_shared ? front : mlp + front));
}

hipError_t ensure(const DevGraph& g, MsDev* ms, int wmax, int32_t k, int nbatches) {
  const int64_t nhat = g.nsets * g.sigma;
  if (ms->wmax < wmax || ms->nhat != nhat) {
    ms_release(ms);
    const size_t words = static_cast<size_t>(nhat) * wmax;
    hipError_t e;
    for (auto& f : ms->F)
      if ((e = hipMalloc(&f, words * 8)) != hipSuccess) return e;
    for (auto& b : ms->fb)
      if ((e = hipMalloc(&b, static_cast<size_t>(nhat / 8) + 16)) != hipSuccess) return e;
    if ((e = hipMalloc(&ms->V, words * 8)) != hipSuccess) return e;
    if ((e = hipMalloc(&ms->N, words * 8)) != hipSuccess) return e;
    if ((e = hipMalloc(&ms->act, static_cast<size_t>(g.nsets) * wmax * 8)) != hipSuccess) return e;
    if ((e = hipMalloc(&ms->dirty, static_cast<size_t>(g.nsets))) != hipSuccess) return e;
    for (int i = 0; i < 2; ++i)
      if ((e = hipMalloc(&ms->queue[i], sizeof(uint4) * static_cast<size_t>(std::max<int64_t>(g.nvss, 1)))) !=
          hipSuccess)
        return e;
    if ((e = hipMemset(ms->N, 0, words * 8)) != hipSuccess) return e;
    if ((e = hipMemset(ms->dirty, 0, static_cast<size_t>(g.nsets))) != hipSuccess) return e;
    ms->wmax = wmax;
    ms->nhat = nhat;
    ms->nsets = g.nsets;
  }
  if (ms->srcs_cap < k) {
    if (ms->srcs) (void)hipFree(ms->srcs);
    ms->srcs = nullptr;
    hipError_t e = hipMalloc(&ms->srcs, sizeof(int32_t) * static_cast<size_t>(k));
    if (e != hipSuccess) return e;
    ms->srcs_cap = k;
  }
  if (ms->batches_cap < nbatches) {
    if (ms->batches) (void)hipFree(ms->batches);
    ms->batches = nullptr;
    hipError_t e = hipMalloc(&ms->batches, sizeof(MsBatch) * static_cast<size_t>(nbatches));
    if (e != hipSuccess) return e;
    ms->batches_cap = nbatches;
  }
  if (ms->grid == 0) {
    int nb = 0;
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, ms_kernel(g));
    if (e != hipSuccess) return e;
    ms->static_lds = attr.sharedSizeBytes;
    MsArgs any{};
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, ms_kernel(g), kMsBlock,
                                                     ms_dynamic_lds(g, *ms, BLEST_POLICY_LEARNED, &any));
    if (e != hipSuccess) return e;
    if (nb < 1) return hipErrorInvalidConfiguration;
    ms->grid = g.num_cu;
    ms->block = kMsBlock;
  }
  if (!ms->log) {
    hipError_t e = hipMalloc(&ms->log, sizeof(MsLevelRec) * static_cast<size_t>(kMsLogCap));
    if (e != hipSuccess) return e;
    ms->log_cap = kMsLogCap;
  }
  if (ms->part_blocks < ms->grid) {
    if (ms->part) (void)hipFree(ms->part);
    ms->part = nullptr;
    hipError_t e = hipMalloc(&ms->part, sizeof(long long) * 2 * 64 * kWMax * static_cast<size_t>(ms->grid));
    if (e != hipSuccess) return e;
    ms->part_blocks = ms->grid;
  }
  return hipSuccess;
}

// Kernel arguments of one multi-source call whose source list and batch plan
// are already on the device (srcs_dev, batches_dev).
MsArgs ms_args(const DevGraph& g, const MsDev* ms, const int32_t* srcs_dev, const MsBatch* batches_dev, int nplan,
               int policy, float eta, uint64_t seed, int16_t* levels16, int64_t* sums, int64_t* reach, double* cc,
               int64_t* far, int probe) {
  MsArgs a{};
  a.rp_in = to_global(g.rp_in);
  a.col_in = to_global(g.col_in);
  a.slice_ptr = to_global(g.slice_ptr);
  a.slices = to_global(g.slices);
  a.orig_id = to_global(g.orig_id);
  a.n = g.n;
  a.m = g.m;
  a.nsets = g.nsets;
  a.tau = g.tau;
  a.rows = to_global(g.ms_rows);
  a.nrows = g.ms_nrows;
  a.nwide = g.ms_nwide;
  a.nlong = g.ms_nlong;
  for (int i = 0; i < 2; ++i) a.F[i] = to_global(ms->F[i]);
  for (int i = 0; i < 3; ++i) a.fb[i] = to_global(ms->fb[i]);
  a.V = to_global(ms->V);
  a.N = to_global(ms->N);
  a.act = to_global(ms->act);
  a.dirty = to_global(ms->dirty);
  a.queue[0] = to_global(ms->queue[0]);
  a.queue[1] = to_global(ms->queue[1]);
  a.srcs = to_global(srcs_dev);
  a.batches = to_global(batches_dev);
  a.nbatches = nplan;
  a.levels16 = to_global(levels16);
  a.planes = to_global(levels16 ? ms->planes : nullptr);
  a.perm = to_global(ms->perm);
  a.sums = to_global(sums);
  a.reach = to_global(reach);
  a.cc = to_global(cc);
  a.far = to_global(far);
  a.nvss = g.nvss;
  a.nslices = g.nslices;
  a.mlp = to_global(g.ms_mlp);
  a.probe = probe;
  a.log = to_global(ms->log);
  a.log_cap = ms->log_cap;
  a.part = to_global(ms->part);
  a.ctl = to_global(g.ctl);
  a.policy = policy;
  a.eta = eta;
  a.seed = seed;
  a.timeout_ticks = 3000000000ULL;  // 30 s
  a.queue_form = g.ms_queue_form;
  a.ablation = g.ms_ablation;
  a.hstat = to_global(g.hstat);
  return a;
}

}  // namespace

__global__ void k_ms_perm(const int32_t* __restrict__ orig_id, int64_t n, int32_t* __restrict__ perm) {
  for (long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<long long>(gridDim.x) * blockDim.x)
    perm[orig_id[i]] = static_cast<int32_t>(i);
}

// Level planes for the int16 output of batches up to 64 * wmax wide (a level
// has kMsPlanes bits), and (for a relabelled graph) the input -> internal id
// map they are read back through.
hipError_t ensure_levels(const DevGraph& g, MsDev* ms, int wmax, hipStream_t st) {
  const int64_t need = static_cast<int64_t>(kMsPlanes) * g.nsets * g.sigma * wmax;
  hipError_t e;
  if (ms->plane_words < need) {
    if (ms->planes) (void)hipFree(ms->planes);
    ms->planes = nullptr;
    ms->plane_words = 0;
    if ((e = hipMalloc(&ms->planes, 8 * static_cast<size_t>(need))) != hipSuccess) return e;
    ms->plane_words = need;
  }
  if (g.orig_id && !ms->perm) {
    if ((e = hipMalloc(&ms->perm, sizeof(int32_t) * static_cast<size_t>(std::max<int64_t>(g.n, 1)))) != hipSuccess)
      return e;
    hipLaunchKernelGGL(k_ms_perm, dim3(static_cast<unsigned>(std::min<int64_t>((g.n + 255) / 256, 4096))),
                       dim3(256), 0, st, g.orig_id, g.n, ms->perm);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

// Words per vertex of a batch of `count` sources of a width. A level costs bytes
// per word, also those no source uses: one source in a 512-wide batch on scale-20
// R-MAT took 942 us with 8 words, 486 with one; 100 sources 1,602 with 8, 930
// with two. (Four words instead of eight gain on large graphs, 1,754 -> 1,349 us
// for 200 sources, but their gather steps take longer where rows are short: 12.0
// -> 13.1 ms on a 256 x 256 grid. So more than 128 sources keep the width's.)
int ms_batch_words(int count, int width) { return count <= 64 ? 1 : count <= 128 ? 2 : width / 64; }

hipError_t ms_run(const DevGraph& g, MsDev* ms, const int32_t* srcs, int32_t k, const int32_t* widths, int nwidths,
                  int policy, float eta, uint64_t seed, int16_t* levels16, int64_t* sums, int64_t* reach, double* cc,
                  hipStream_t st, int graph, int64_t* far, int probe) {
  if (k <= 0) return hipSuccess;
  // A capturing stream is refused before anything is allocated or launched: a
  // recorded launch of k_ms_perm would leave an id map that no kernel has written.
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &capture) == hipSuccess && capture != hipStreamCaptureStatusNone)
    return hipErrorStreamCaptureUnsupported;
  std::vector<MsBatch> plan;
  int32_t off = 0;
  int wmax = 1;  // the buffers hold the widths asked for
  for (int i = 0; off < k; ++i) {
    const int width = widths[nwidths > 0 ? std::min(i, nwidths - 1) : 0];
    const int count = std::min(width, k - off);
    plan.push_back(MsBatch{off, count, ms_batch_words(count, width), 0});
    wmax = std::max(wmax, width / 64);
    off += count;
  }
  const int nplan = static_cast<int>(plan.size());
  hipError_t e = ensure(g, ms, wmax, k, nplan);
  if (e != hipSuccess) return e;
  if (levels16 && (e = ensure_levels(g, ms, wmax, st)) != hipSuccess) return e;
  MsArgs a = ms_args(g, ms, ms->srcs, static_cast<const MsBatch*>(ms->batches), nplan, policy, eta, seed, levels16,
                     sums, reach, cc, far, probe);
  if (k <= kMsInlineSrcs && nplan <= kMsInlineBatches) {
    a.inlined = 1;
    std::copy(srcs, srcs + k, a.srcs_in);
    std::copy(plan.begin(), plan.end(), a.plan_in);
  } else {
    if ((e = hipMemcpyAsync(ms->srcs, srcs, sizeof(int32_t) * k, hipMemcpyHostToDevice, st)) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(ms->batches, plan.data(), sizeof(MsBatch) * nplan, hipMemcpyHostToDevice, st)) !=
        hipSuccess)
      return e;
    // the copies read pageable host memory; wait so `plan` may go out of scope
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  }
  const unsigned shmem = policy == BLEST_POLICY_LEARNED ? kLdsMlpFloats * sizeof(float) : 0u;
  if (!graph || probe) {
    void* args[] = {static_cast<void*>(&a)};
    const unsigned dyn = ms_dynamic_lds(g, *ms, policy, &a);
    return hipLaunchCooperativeKernel(ms_kernel(g), dim3(ms->grid), dim3(ms->block), args, dyn, st);
  }
  // Graph mode: kMsGraphKernels phase kernels, then copies of the state and
  // error words to pinned host memory, built once as a hipGraph for a stream
  // of our own (the caller's may be the null stream) and replayed until the
  // state says MS_DONE. One instantiated graph serves every call with the
  // same kernel, grid and LDS size: a call only rewrites the kernel nodes'
  // arguments. The replays are ordered after the caller's stream by an event.
  if (!ms->gstream) {
    if ((e = hipStreamCreateWithFlags(&ms->gstream, hipStreamNonBlocking)) != hipSuccess) return e;
    for (int i = 0; i < 2; ++i)
      if ((e = hipEventCreateWithFlags(&ms->gev[i], hipEventDisableTiming)) != hipSuccess) return e;
  }
  const void* fn = (g.sigma == 8 && !g.wide) ? ms_phase_fn<8, uint32_t>()
                   : g.sigma == 8            ? ms_phase_fn<8, uint64_t>()
                   : g.sigma == 16           ? ms_phase_fn<16, uint64_t>()
                                             : ms_phase_fn<32, uint64_t>();
  hipStream_t gs = ms->gstream;
  int* flags = g.host_flags;
  int par[kMsGraphKernels];
  void* kargs[kMsGraphKernels][2];
  hipKernelNodeParams kp[kMsGraphKernels];
  for (int i = 0; i < kMsGraphKernels; ++i) {
    par[i] = i & 1;
    kargs[i][0] = static_cast<void*>(&a);
    kargs[i][1] = static_cast<void*>(&par[i]);
    kp[i] = hipKernelNodeParams{};
    kp[i].func = const_cast<void*>(fn);
    kp[i].gridDim = dim3(ms->grid);
    kp[i].blockDim = dim3(kMsBlock);
    kp[i].sharedMemBytes = shmem;
    kp[i].kernelParams = kargs[i];
    kp[i].extra = nullptr;
  }
  if (ms->gexec && (ms->gfn != fn || ms->ggrid != ms->grid || ms->gshmem != shmem)) {
    ms_graph_destroy(ms);
  }
  if (!ms->gexec) {
    if ((e = hipGraphCreate(&ms->graph, 0)) != hipSuccess) return e;
    hipGraphNode_t prev = nullptr;
    for (int i = 0; i < kMsGraphKernels && e == hipSuccess; ++i) {
      e = hipGraphAddKernelNode(&ms->gnode[i], ms->graph, prev ? &prev : nullptr, prev ? 1 : 0, &kp[i]);
      prev = ms->gnode[i];
    }
    hipGraphNode_t cp[2] = {nullptr, nullptr};
    if (e == hipSuccess)
      e = hipGraphAddMemcpyNode1D(&cp[0], ms->graph, &prev, 1, flags + 2, &g.ctl->ms_state[0][0], sizeof(int),
                                  hipMemcpyDeviceToHost);
    if (e == hipSuccess)
      e = hipGraphAddMemcpyNode1D(&cp[1], ms->graph, &cp[0], 1, flags + 3, &g.ctl->error[0], sizeof(int),
                                  hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipGraphInstantiate(&ms->gexec, ms->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
      ms_graph_destroy(ms);
      return e;
    }
    ms->gfn = fn;
    ms->ggrid = ms->grid;
    ms->gshmem = shmem;
    ++ms->gcaptures;
  } else {
    for (int i = 0; i < kMsGraphKernels; ++i)
      if ((e = hipGraphExecKernelNodeSetParams(ms->gexec, ms->gnode[i], &kp[i])) != hipSuccess) return e;
  }
  if ((e = hipEventRecord(ms->gev[0], st)) != hipSuccess) return e;
  if ((e = hipStreamWaitEvent(gs, ms->gev[0], 0)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_ms_start, dim3(1), dim3(64), 0, gs, g.ctl, g.hstat);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // every batch has at most 3 + 3 * 32768 phases (levels are int16)
  const long long max_replays = static_cast<long long>(nplan) * (3LL * 32768 + 4) / kMsGraphKernels + 2;
  for (long long r = 0; e == hipSuccess; ++r) {
    if (r >= max_replays) {
      e = hipErrorLaunchTimeOut;
      break;
    }
    if ((e = hipGraphLaunch(ms->gexec, gs)) != hipSuccess) break;
    if ((e = hipStreamSynchronize(gs)) != hipSuccess) break;
    if (flags[2] == MS_DONE || flags[3] != 0) break;
  }
  if (e != hipSuccess) return e;
  if ((e = hipEventRecord(ms->gev[1], gs)) != hipSuccess) return e;
  return hipStreamWaitEvent(st, ms->gev[1], 0);
}

void ms_release(MsDev* ms) {
  for (void* p : {static_cast<void*>(ms->F[0]), static_cast<void*>(ms->F[1]), static_cast<void*>(ms->fb[0]),
                  static_cast<void*>(ms->fb[1]), static_cast<void*>(ms->fb[2]), static_cast<void*>(ms->V),
                  static_cast<void*>(ms->N), static_cast<void*>(ms->act), static_cast<void*>(ms->dirty),
                  static_cast<void*>(ms->queue[0]), static_cast<void*>(ms->queue[1])})
    if (p) (void)hipFree(p);
  for (auto& f : ms->F) f = nullptr;
  for (auto& b : ms->fb) b = nullptr;
  ms->V = ms->N = ms->act = nullptr;
  ms->dirty = nullptr;
  ms->queue[0] = ms->queue[1] = nullptr;
  ms->wmax = 0;
  ms->nhat = 0;
  if (ms->planes) (void)hipFree(ms->planes);
  if (ms->perm) (void)hipFree(ms->perm);
  ms->planes = nullptr;
  ms->plane_words = 0;
  ms->perm = nullptr;
}

void ms_free_all(MsDev* ms) {
  ms_release(ms);
  ms_graph_destroy(ms);
  if (ms->gstream) (void)hipStreamDestroy(ms->gstream);
  for (int i = 0; i < 2; ++i)
    if (ms->gev[i]) (void)hipEventDestroy(ms->gev[i]);
  ms->gstream = nullptr;
  ms->gev[0] = ms->gev[1] = nullptr;
  if (ms->srcs) (void)hipFree(ms->srcs);
  if (ms->part) (void)hipFree(ms->part);
  if (ms->batches) (void)hipFree(ms->batches);
  if (ms->log) (void)hipFree(ms->log);
  ms->log = nullptr;
  ms->log_cap = 0;
  ms->srcs = nullptr;
  ms->part = nullptr;
  ms->batches = nullptr;
  ms->srcs_cap = 0;
  ms->part_blocks = 0;
  ms->batches_cap = 0;
  ms->grid = 0;
}

void ms_reset(MsDev* ms) {
  // After a device-side error N and dirty may hold stale marks.
  if (ms->N && ms->nhat) (void)hipMemset(ms->N, 0, static_cast<size_t>(ms->nhat) * ms->wmax * 8);
  if (ms->dirty && ms->nsets) (void)hipMemset(ms->dirty, 0, static_cast<size_t>(ms->nsets));
}

// ----------------------------------------------------------- no-alloc entry
// blest_msbfs_noalloc keeps the source list and the batch plan of a call in
// this array instead of in buffers the library allocates: the first
// BLEST_MSBFS_NOALLOC_MAX_SOURCES entries hold internal source ids, then one
// 4-int batch descriptor per batch (at most one per 64 sources). Each device
// holds its own copy until the process ends; host code reaches it only
// through the address hipGetSymbolAddress gives for the current device.
constexpr int kNoAllocMaxSources = BLEST_MSBFS_NOALLOC_MAX_SOURCES;
constexpr int kNoAllocMaxBatches = kNoAllocMaxSources / 64;
static_assert(sizeof(MsBatch) == 4 * sizeof(int32_t), "batch descriptor layout");
static __device__ __align__(256) int32_t scratch[kNoAllocMaxSources + 4 * kNoAllocMaxBatches];

namespace {

constexpr int kNoAllocDevices = 64;
std::mutex g_noalloc_mu;
int32_t* g_noalloc_ptr[kNoAllocDevices] = {};

// This device's copy of `scratch`, looked up once per device (the caller
// has made `device` current).
hipError_t noalloc_scratch(int device, int32_t** out) {
  if (device < 0 || device >= kNoAllocDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_noalloc_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_noalloc_ptr[device] = static_cast<int32_t*>(p);
  }
  *out = g_noalloc_ptr[device];
  return hipSuccess;
}

}  // namespace

bool ms_ready(const DevGraph& g, const MsDev* ms, int W) {
  return ms->wmax >= W && ms->nhat == g.nsets * g.sigma && ms->F[0] && ms->F[1] && ms->fb[0] && ms->fb[1] && ms->fb[2] && ms->V && ms->N && ms->act && ms->dirty &&
         ms->queue[0] && ms->queue[1] && ms->grid > 0 && ms->log && ms->part && ms->part_blocks >= ms->grid;
}

hipError_t ms_run_noalloc(const DevGraph& g, MsDev* ms, const int32_t* srcs, const int32_t* perm, int32_t k,
                          int width, int policy, float eta, uint64_t seed, int16_t* levels16, hipStream_t st) {
  if (k <= 0) return hipSuccess;
  if (k > kNoAllocMaxSources || width % 64 != 0 || width < 64 || width > 64 * kWMax) return hipErrorInvalidValue;
  const int W = width / 64;
  if (!ms_ready(g, ms, W)) return hipErrorNotReady;
  int32_t* base = nullptr;
  hipError_t e = noalloc_scratch(g.device, &base);
  if (e != hipSuccess) return e;
  int32_t* dsrcs = base;
  MsBatch* dplan = reinterpret_cast<MsBatch*>(base + kNoAllocMaxSources);
  // Internal source ids through a fixed host staging buffer; the copies read
  // pageable memory, so each is waited for before the buffer is refilled.
  constexpr int kStage = 4096;
  int32_t stage[kStage];
  for (int32_t off = 0; off < k; off += kStage) {
    const int32_t c = std::min<int32_t>(kStage, k - off);
    for (int32_t i = 0; i < c; ++i) stage[i] = perm ? perm[srcs[off + i]] : srcs[off + i];
    if ((e = hipMemcpyAsync(dsrcs + off, stage, sizeof(int32_t) * c, hipMemcpyHostToDevice, st)) != hipSuccess)
      return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  }
  const int per = 64 * W;
  const int nplan = (k + per - 1) / per;
  MsBatch plan[kNoAllocMaxBatches];
  for (int i = 0; i < nplan; ++i) {
    const int count = std::min(per, k - i * per);
    plan[i] = MsBatch{i * per, count, ms_batch_words(count, width), 0};
  }
  if ((e = hipMemcpyAsync(dplan, plan, sizeof(MsBatch) * nplan, hipMemcpyHostToDevice, st)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  MsArgs a = ms_args(g, ms, dsrcs, dplan, nplan, policy, eta, seed, levels16, nullptr, nullptr, nullptr, nullptr, 0);
  // no level planes here (the entry point allocates nothing): the caller's
  // rows are written directly
  a.planes = nullptr;
  void* args[] = {static_cast<void*>(&a)};
  const unsigned dyn = ms_dynamic_lds(g, *ms, policy, &a);
  return hipLaunchCooperativeKernel(ms_kernel(g), dim3(ms->grid), dim3(ms->block), args, dyn, st);
}

}  // namespace blest
