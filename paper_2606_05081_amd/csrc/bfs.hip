// Single-source BVSS breadth-first search for gfx950.
//
// One traversal step turns frontier level l into level l+1 in two stages
// (Section "Lazy Vertex Updates", Alg. 3):
//   Stage 1 marks every vertex that has a neighbour in the frontier, with a
//           plain byte store of 1 into mark[] (idempotent, so no atomics).
//           Three interchangeable engines do this:
//             E0 BVSS top-down: one wave per queued virtual slice set; each
//                lane tests (mask & alpha) != 0 for its slices, alpha being
//                the frontier bits of the set (Eq. 1 / Eq. 2, popc(a&x) > 0
//                written as a bitwise AND).
//             E1 push: frontier vertices walk their CSR rows.
//             E2 bottom-up (Alg. 4): each unvisited vertex scans its row and
//                stops at the first frontier neighbour.
//   Stage 2 sweeps the marks of every slice set, keeps the bits not yet
//           visited (the XOR of V_next and V_curr), writes their level,
//           updates visited/frontier words, enqueues every VSS of each set
//           that gained a vertex and accumulates the per-level statistics.
// The engine of each step is chosen on the device (Eq. 3 heuristic, learned
// network, fixed or random) identically by every workgroup. All levels run in
// one cooperative persistent launch separated by a device-wide barrier
// (Section "Switching Mechanism", last paragraph); a per-stage launch mode is
// kept for comparison.
#include "device_common.h"
#include "mlp_infer.h"
#include "row_pos.h"

namespace blest {

// Frontier buffer of a level parity (level l reads buffer l & 1; its Stage 2
// writes the other one, so an engine never reads words being rewritten).
__device__ __forceinline__ gptr<void> front_buf(args_ref<BfsArgs> a, int sel) {
  return (gptr<char>)a.front + (sel ? a.fstride : 0LL);
}

// Per-workgroup Stage 2 partial counters: frontier, queued slices, frontier
// edges, deg >= 32, deg >= 1024, light, heavy and queue entries.
constexpr int kParts = 8;

// Row pointers rp[s*SIGMA .. s*SIGMA + SIGMA] of a slice set's vertices with
// 16-byte loads. rp is padded on the device to N_s*SIGMA + 1 entries (the
// tail repeats m), and s*SIGMA*4 is a multiple of 16, so the loads are aligned
// and in bounds.
template <int SIGMA>
__device__ __forceinline__ void load_set_rp(gptr<const int32_t> rp, long long s, int (&r)[SIGMA + 1]) {
  const gptr<const int4> p = (gptr<const int4>)(rp + s * SIGMA);
#pragma unroll
  for (int i = 0; i < SIGMA / 4; ++i) {
    const int4 q = p[i];
    r[4 * i + 0] = q.x;
    r[4 * i + 1] = q.y;
    r[4 * i + 2] = q.z;
    r[4 * i + 3] = q.w;
  }
  r[SIGMA] = rp[s * SIGMA + SIGMA];
}

// ------------------------------------------------------------- decisions

// (every count is at most n, m or the number of slices, all below 2^31; ten
// 32-bit words are passed to a function in registers)
struct LevelView {
  uint32_t frontier, queue, qslices, fedges, deg32, deg1024, light, heavy, cumv, cume;
};

__device__ __forceinline__ uint32_t u32_uniform(unsigned long long v) {
  return __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
}

__device__ __forceinline__ LevelView read_level(gptr<const Ctl> ctl, int slot) {
  const gptr<const unsigned long long> acc = &ctl->acc[slot][0][0];
  LevelView v;
  v.frontier = u32_uniform(acc[F_FRONTIER * kPad]);
  v.queue = u32_uniform(acc[F_QUEUE * kPad]);
  v.qslices = u32_uniform(acc[F_QSLICES * kPad]);
  v.fedges = u32_uniform(acc[F_FEDGES * kPad]);
  v.deg32 = u32_uniform(acc[F_DEG32 * kPad]);
  v.deg1024 = u32_uniform(acc[F_DEG1024 * kPad]);
  v.light = u32_uniform(acc[F_LIGHT * kPad]);
  v.heavy = u32_uniform(acc[F_HEAVY * kPad]);
  v.cumv = u32_uniform(acc[F_CUMV * kPad]);
  v.cume = u32_uniform(acc[F_CUME * kPad]);
  return v;
}

// The 12 switch features of a level (network inputs before standardising).
__device__ __forceinline__ void level_features(float (&f)[kMaxSwitchFeatures], const LevelView& v, args_ref<BfsArgs> a) {
  const long long unv = a.n - v.cumv, unv_e = a.m - v.cume;
  const float lf = log2f(1.0f + static_cast<float>(v.frontier));
  const float lqs = log2f(1.0f + static_cast<float>(v.qslices));
  const float ln = log2f(static_cast<float>(a.n));
  const float lm = log2f(1.0f + static_cast<float>(a.m));
  f[0] = lf;
  f[1] = lqs;
  f[2] = lf - ln;
  f[3] = log2f(1.0f + static_cast<float>(v.queue)) - log2f(1.0f + static_cast<float>(a.nvss));
  f[4] = lqs - log2f(1.0f + static_cast<float>(a.nslices));
  f[5] = log2f(1.0f + static_cast<float>(v.fedges)) - lm;
  f[6] = log2f(1.0f + static_cast<float>(unv)) - ln;
  f[7] = log2f(1.0f + static_cast<float>(unv_e)) - lm;
  // Eq. 3's own quantities, as a log ratio
  f[8] = log2f(1.0f + static_cast<float>(v.queue)) - log2f(1.0f + static_cast<float>(unv));
  // Reserved (zero). The frontier degree histogram and the growth ratio were
  // inputs once; on R-MAT + grid training data they let the network learn
  // family shortcuts that failed on Erdos-Renyi graphs.
  f[9] = 0.0f;
  f[10] = 0.0f;
  f[11] = 0.0f;
}

// Eq. 3: bottom-up iff #unvisited < eta * |Q_curr| (|Q| counts VSSs).
__device__ __forceinline__ int heuristic_engine(long long unvisited, long long queue, float eta) {
  return (static_cast<double>(unvisited) < static_cast<double>(eta) * static_cast<double>(queue))
             ? BLEST_ENGINE_BOTTOM_UP
             : BLEST_ENGINE_BVSS;
}

__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

// Engine choice for the step out of `level`, evaluated by each wave on its
// own (every input is uniform over the grid).
__device__ __forceinline__ int choose_engine(args_ref<BfsArgs> a, const LevelView& v,
                                             const float (&feat)[kMaxSwitchFeatures], int level, lptr<const float> s_mlp,
                                             bool learned, int* fallback) {
  const long long unvisited = a.n - v.cumv;
  *fallback = 0;
  switch (a.policy) {
    case BLEST_POLICY_BVSS:
      return BLEST_ENGINE_BVSS;
    case BLEST_POLICY_PUSH:
      return BLEST_ENGINE_PUSH;
    case BLEST_POLICY_BOTTOM_UP:
      return BLEST_ENGINE_BOTTOM_UP;
    case BLEST_POLICY_RANDOM:
      return static_cast<int>(mix64(a.seed + 0x9E3779B97F4A7C15ULL * static_cast<unsigned long long>(level + 1)) % 3ULL);
    case BLEST_POLICY_LEARNED:
      if (learned) {
        const int c = mlp_choose_wave(s_mlp, feat);
        if (c >= 0) return c;
      }
      *fallback = 1;
      return heuristic_engine(unvisited, v.queue, a.eta);
    default:
      return heuristic_engine(unvisited, v.queue, a.eta);
  }
}

__device__ __forceinline__ bool use_panel(args_ref<BfsArgs> a, const LevelView& v);

// Chooses the engine of the step out of `level` and (workgroup 0, one lane)
// writes the level's record, all but its times. EAGER: a push choice runs the
// BVSS engine, and never over the panel copy. A function of its own, so that
// its features and network stay out of the kernel's registers.
template <bool EAGER>
__device__ __attribute__((noinline)) int decide_level(args_ref<BfsArgs> a_, LevelView v, int level,
                                                      lptr<const float> s_mlp, bool learned) {
  args_ref<BfsArgs> a = uniform_args(a_);
  level = uniform(level);
  float feat[kMaxSwitchFeatures];
  level_features(feat, v, a);
  int fallback = 0;
  int engine = choose_engine(a, v, feat, level, s_mlp, learned, &fallback);
  if (EAGER && engine == BLEST_ENGINE_PUSH) engine = BLEST_ENGINE_BVSS;
  if (blockIdx.x == 0 && threadIdx.x == 0 && level < a.log_cap) {
    const gptr<LevelRec> r = a.log + level;
    r->frontier = v.frontier;
    r->queue = v.queue;
    r->qslices = v.qslices;
    r->fedges = v.fedges;
    r->unvisited = a.n - v.cumv;
    r->unvisited_edges = a.m - v.cume;
    r->deg32 = v.deg32;
    r->deg1024 = v.deg1024;
    r->engine = a.probe ? -1 : engine;
    r->fallback = fallback;
    r->panel = !EAGER && engine == BLEST_ENGINE_BVSS && use_panel(a, v);
    r->t_mid = 0;
    r->t_end = 0;
    r->t_count = 0;
    r->t_engine[0] = r->t_engine[1] = r->t_engine[2] = 0;
    r->work = 0;
#pragma unroll
    for (int k = 0; k < kMaxSwitchFeatures; ++k) r->feat[k] = feat[k];
  }
  return uniform(engine);
}

// ------------------------------------------------------------ Stage 1

constexpr int kSingleHash = 8192;              // LDS hash-set slots (power of two)
constexpr long long kSingleMaxMarks = 4096;    // keeps the hash set at most half full
// LDS layout of a single-workgroup level: hs[kSingleHash] hash slots, then
// the list of recorded sets hs[kSingleHash + 1 + i] with its length at
// hs[kSingleHash].
constexpr int kSingleLds = kSingleHash + 1 + kSingleMaxMarks;

__device__ __forceinline__ void record_set(lptr<int> hs, long long s, gptr<Ctl> ctl) {
  uint32_t h = (static_cast<uint32_t>(s) * 2654435761u) >> (32 - 13);
  for (int probe = 0; probe < kSingleHash; ++probe) {
    int old = -1;
    __hip_atomic_compare_exchange_strong(hs + h, &old, static_cast<int>(s), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
    if (old == -1) {
      const int idx = __hip_atomic_fetch_add(hs + kSingleHash, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      hs[kSingleHash + 1 + idx] = static_cast<int>(s);
      return;
    }
    if (old == static_cast<int>(s)) return;
    h = (h + 1) & (kSingleHash - 1);
  }
  __hip_atomic_store(&ctl->error[0], static_cast<int>(BLEST_ERR_INVALID_ARG), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}


// E0: BVSS top-down with pull mechanics and lazy marking. A wave takes G
// consecutive queue entries at a time and issues all their slice loads before
// testing any, so each lane keeps G * K independent loads in flight
// (K = tau / 64 slices per lane per VSS).
template <int SIGMA, class SliceT, int K, bool REC>
__device__ __attribute__((noinline)) long long engine_bvss_k(args_ref<BfsArgs> a_, int sel, long long qlen,
                                                             long long gwave, long long nwaves, lptr<int> hs) {
  args_ref<BfsArgs> a = uniform_args(a_);
  sel = uniform(sel);
  qlen = uniform(qlen);
  gwave = uniform(gwave);
  nwaves = uniform(nwaves);
  long long work = 0;
  using M = typename MaskOf<SIGMA>::T;
  constexpr int G = 4;
  const gptr<const uint4> qg = a.queue[sel];
  gptr<const SliceT> __restrict__ sl = (gptr<const SliceT>)a.slices;
  gptr<const M> __restrict__ vis = (gptr<const M>)a.vis;
  gptr<uint8_t> __restrict__ mark = a.mark;
  const uint32_t lane = static_cast<uint32_t>(lane_id());
  const bool pre = a.prefilter != 0;
  for (long long base = gwave * G; base < qlen; base += nwaves * G) {
    uint4 dl = make_uint4(0u, 0u, 0u, 0u);
    if (lane < G && base + lane < qlen) dl = qg[base + lane];
    uint32_t st[G], cn[G];
    SliceT al[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      st[g] = __builtin_amdgcn_readlane(dl.x, g);
      cn[g] = __builtin_amdgcn_readlane(dl.y, g);
      al[g] = static_cast<SliceT>(static_cast<uint32_t>(__builtin_amdgcn_readlane(dl.z, g)));
    }
    SliceT w[G][K];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t j = lane + 64u * k;
        work += j < cn[g];
        w[g][k] = (j < cn[g]) ? sl[st[g] + j] : SliceT(0);
      }
    if (pre) {
      M vv[G][K];
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const uint32_t row = static_cast<uint32_t>(w[g][k] >> SliceFmt<SliceT>::kRowShift);
          vv[g][k] = (w[g][k] & al[g]) ? vis[row / SIGMA] : M(~M(0));
        }
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const uint32_t row = static_cast<uint32_t>(w[g][k] >> SliceFmt<SliceT>::kRowShift);
          if (!((vv[g][k] >> (row % SIGMA)) & 1u)) {
            mark[row] = 1;
            if (REC) record_set(hs, row / SIGMA, a.ctl);
          }
        }
    } else {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (w[g][k] & al[g]) {
            const uint32_t row = static_cast<uint32_t>(w[g][k] >> SliceFmt<SliceT>::kRowShift);
            mark[row] = 1;
            if (REC) record_set(hs, row / SIGMA, a.ctl);
          }
    }
  }
  return work;
}

template <int SIGMA, class SliceT, bool REC>
__device__ __forceinline__ long long engine_bvss(args_ref<BfsArgs> a, int sel, long long qlen, long long gwave,
                                                 long long nwaves, lptr<int> hs) {
  switch (a.tau) {
    case 64:
      return engine_bvss_k<SIGMA, SliceT, 1, REC>(a, sel, qlen, gwave, nwaves, hs);
    case 128:
      return engine_bvss_k<SIGMA, SliceT, 2, REC>(a, sel, qlen, gwave, nwaves, hs);
    case 192:
      return engine_bvss_k<SIGMA, SliceT, 3, REC>(a, sel, qlen, gwave, nwaves, hs);
    default:
      return engine_bvss_k<SIGMA, SliceT, 4, REC>(a, sel, qlen, gwave, nwaves, hs);
  }
}

// E0 on the panel-blocked copy, for dense levels. Workgroup b owns panels
// b, b + G, ... (2^rb consecutive rows each) and reads every chunk of its
// panel: 256 slice words, one 16-byte load per lane, plus the chunk's
// 512-byte window of frontier words (one 8-byte load per lane); a lane finds
// the frontier word of each of its slices' sets in the window by two wave
// shuffles. A slice hits when its mask meets that word, and the hit row's
// byte in an LDS byte map is set with a plain store (lazy marking is
// idempotent, so no atomic is needed). Loads of the next batch of chunks are
// issued before the current batch is tested. After the panel, the byte map
// minus the visited words gives the panel's new vertices; the workgroup owns
// those rows, so each new vertex is handled once and no visited word is read
// per hit. Either they are written to the mark bytes (32 rows per pair of
// 16-byte stores) for Stage 2, or (fused, new_level >= 0) the workgroup does
// Stage 2 for its rows itself: it updates the visited words, writes every
// next-frontier word of the panel (buffer sel ^ 1), writes the levels and
// stores its Stage 2 partial counters, so the grid needs no separate Stage 2
// sweep and no second barrier for the level.
// pm: LDS scratch of at least 2^rb bytes, left filled with ones (the
// single-workgroup hash set shares it).
constexpr int kPanelChunk = 256;      // slices per chunk (host layout)
constexpr int kPanelUnroll = 8;       // chunks per wave per batch
static_assert(kPanelUnroll <= kPanelBasePad, "batch bases are read past the last chunk");
constexpr int kPanelMaxBytes = 1 << 15;  // LDS byte map of one panel (rb <= 15)
static_assert(kSingleHash * 4 >= kPanelMaxBytes, "the panel byte map lives in the hash-set slots");
constexpr long long kPanelDenom = 8;  // dense: queued slices >= panel slots / 8

__device__ __forceinline__ bool use_panel(args_ref<BfsArgs> a, const LevelView& v) {
  if (a.npanels <= 0) return false;
  if (a.panel_mode == 2) return true;
  return v.qslices > kSingleMaxMarks && kPanelDenom * v.qslices >= a.panel_slots;
}

struct PanelPtrs {
  gptr<const uint4> words;    // 64 uint4 per chunk
  gptr<const uint2> front8;   // 8 frontier bytes per element
  cptr<const uint32_t> base;  // first set of each chunk (read-only: scalar loads)
};

// Loads chunk c (clamped to the panel's last chunk `cl`, so every load is in
// bounds; the caller skips chunks past the end): this lane's 4 slice words and
// its 8 bytes of the chunk's frontier window.
__device__ __forceinline__ void panel_load(const PanelPtrs& pp, uint32_t c, uint32_t cl, uint32_t lane, uint32_t b,
                                           uint4& w, uint2& f) {
  w = pp.words[static_cast<size_t>(min(c, cl)) * (kPanelChunk / 4) + lane];
  f = pp.front8[(b >> 3) + lane];
}

// Tests the 4 slices of one lane of one chunk; the frontier byte of a slice's
// set is taken from the lane holding it in the chunk's window.
__device__ __forceinline__ void panel_test4(const uint4& w, uint32_t b7, const uint2& f, uint32_t dmask, int rshift,
                                            lptr<uint32_t> pm) {
  const uint32_t s[4] = {w.x, w.y, w.z, w.w};
  uint32_t d[4], lo[4], hi[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    d[q] = ((s[q] >> 8) & dmask) + b7;
    const int src = static_cast<int>(d[q] >> 3);
    lo[q] = static_cast<uint32_t>(__shfl(static_cast<int>(f.x), src, 64));
    hi[q] = static_cast<uint32_t>(__shfl(static_cast<int>(f.y), src, 64));
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t al = (((d[q] >> 2) & 1u) ? hi[q] : lo[q]) >> (8u * (d[q] & 3u));
    if (s[q] & al & 0xffu) reinterpret_cast<lptr<uint8_t>>(pm)[s[q] >> rshift] = 1;
  }
}

// One batch of kPanelUnroll chunks in registers: each chunk's base set, this
// lane's 4 slice words and its 8 bytes of the chunk's frontier window; bit u
// of `valid` (wave-uniform) is set if chunk u lies in the panel.
struct PanelBatch {
  uint32_t b[kPanelUnroll];
  uint4 w[kPanelUnroll];
  uint2 f[kPanelUnroll];
  uint32_t valid;
};

// Bases of the chunks min(c, cl) .. min(c, cl) + U - 1 by scalar loads (c and
// cl wave-uniform; cl = the panel's last chunk). The base array is padded
// with kPanelBasePad zeros, so these loads stay in bounds and a base read
// past the last chunk is set 0, whose window is in bounds too.
__device__ __forceinline__ void panel_bases(const PanelPtrs& pp, uint32_t c, uint32_t cl,
                                            uint32_t (&x)[kPanelUnroll]) {
  const cptr<const uint32_t> b = pp.base + min(c, cl);
#pragma unroll
  for (int u = 0; u < kPanelUnroll; ++u) x[u] = b[u];
}

// Issues the slice and window loads of the batch starting at chunk c, whose
// bases panel_bases read into x. A chunk past cl loads chunk cl's words
// (in bounds) and is left out of the test by `valid`.
__device__ __forceinline__ void panel_issue(const PanelPtrs& pp, PanelBatch& B, uint32_t c, uint32_t cl,
                                            uint32_t lane, const uint32_t (&x)[kPanelUnroll]) {
  B.valid = c > cl ? 0u : (cl - c >= kPanelUnroll - 1 ? (1u << kPanelUnroll) - 1u : (2u << (cl - c)) - 1u);
#pragma unroll
  for (int u = 0; u < kPanelUnroll; ++u) {
    B.b[u] = x[u];
    panel_load(pp, c + u, cl, lane, x[u], B.w[u], B.f[u]);
  }
}

// Tests the chunks of a batch as straight-line code: a chunk outside the
// panel gets an all-zero frontier window, so it hits nothing. With no branch
// in the test, every path to the next batch's loads has waited for exactly
// this batch's loads and no later ones.
__device__ __forceinline__ void panel_test_batch(const PanelBatch& B, uint32_t dmask, int rshift, lptr<uint32_t> pm) {
#pragma unroll
  for (int u = 0; u < kPanelUnroll; ++u) {
    const bool in = (B.valid >> u) & 1u;
    const uint2 f = make_uint2(in ? B.f[u].x : 0u, in ? B.f[u].y : 0u);
    panel_test4(B.w[u], B.b[u] & 7u, f, dmask, rshift, pm);
  }
}

// Stage 2 of one panel (sigma = 8) by the workgroup that owns it: x words of
// its W 32-row groups in pm[8 * j], levels and the counters of finalize_count.
// A lane per vertex, as in finalize_windows: a thread that took its group's 32
// vertices left three quarters of the workgroup idle (128 groups a panel at
// 1 M vertices).
template <int BLOCK>
__device__ __forceinline__ void panel_count_rows(args_ref<BfsArgs> a, lptr<const uint32_t> pm, uint32_t row0,
                                                 uint32_t W, int new_level, uint32_t (&st)[kParts]) {
  constexpr int GB = 8;  // vertices per thread whose loads are issued together
  const gptr<const int32_t> rp = a.rp;
  const gptr<int32_t> levels = a.levels;
  const gptr<const int32_t> orig_id = a.orig_id;
  for (uint32_t base = threadIdx.x; base < 32u * W; base += BLOCK * GB) {
    bool on[GB];
    int r0[GB], r1[GB], id[GB];
#pragma unroll
    for (int j = 0; j < GB; ++j) {
      const uint32_t v = base + j * BLOCK;
      on[j] = v < 32u * W && ((pm[8 * (v >> 5)] >> (v & 31u)) & 1u);
    }
#pragma unroll
    for (int j = 0; j < GB; ++j) {
      const uint32_t u = row0 + base + j * BLOCK;
      r0[j] = r1[j] = id[j] = 0;
      if (on[j]) {
        r0[j] = rp[u];
        r1[j] = rp[u + 1];
        id[j] = orig_id ? orig_id[u] : static_cast<int32_t>(u);
      }
    }
#pragma unroll
    for (int j = 0; j < GB; ++j) {
      if (!on[j]) continue;
      const int d = r1[j] - r0[j];
      levels[id[j]] = new_level;
      st[0] += 1;
      st[2] += static_cast<uint32_t>(d);
      st[3] += d >= 32;
      st[4] += d >= 1024;
      if (d > kLightMax)
        st[6] += (d + kHeavyChunk - 1) / kHeavyChunk;
      else
        st[5] += 1;
    }
  }
}

template <int BLOCK>
__device__ __attribute__((noinline)) long long engine_panel(args_ref<BfsArgs> a_, lptr<uint32_t> pm, int sel,
                                                            int new_level) {
  args_ref<BfsArgs> a = uniform_args(a_);
  sel = uniform(sel);
  new_level = uniform(new_level);
  constexpr int U = kPanelUnroll;
  constexpr uint32_t NW = BLOCK / 64;
  constexpr uint32_t STEP = NW * U;
  const int rb = a.panel_rb;
  const int npanels = a.npanels;
  const uint32_t W = 1u << (rb - 5);  // 32-row groups per panel
  const lptr<u32x4> pm16 = reinterpret_cast<lptr<u32x4>>(pm);
  const lptr<const unsigned long long> pm64 = reinterpret_cast<lptr<const unsigned long long>>(pm);
  const uint32_t dmask = (1u << (24 - rb)) - 1u;
  const int rshift = 32 - rb;
  PanelPtrs pp;
  pp.words = (gptr<const uint4>)a.pwords;
  pp.front8 = (gptr<const uint2>)front_buf(a, sel);
  pp.base = (cptr<const uint32_t>)a.pbase;
  const gptr<const uint32_t> pptr = (gptr<const uint32_t>)a.pptr;
  const gptr<uint32_t> vis32 = (gptr<uint32_t>)a.vis;
  const gptr<uint32_t> next32 = (gptr<uint32_t>)front_buf(a, sel ^ 1);
  const gptr<uint4> mark16 = (gptr<uint4>)a.mark;
  const bool fused = new_level >= 0;
  // fused: the workgroup's Stage 2 counters, summed per panel (kept out of
  // registers during the chunk loop)
  __shared__ uint32_t s_part[kParts];
  if (threadIdx.x < kParts) s_part[threadIdx.x] = 0u;
  const uint32_t lane = static_cast<uint32_t>(lane_id());
  const uint32_t wv = static_cast<uint32_t>(wave_in_block());
  long long work = 0;
  for (int p = blockIdx.x; p < npanels; p += gridDim.x) {
    for (uint32_t j = threadIdx.x; j < 2 * W; j += BLOCK) pm16[j] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    // the chunk range is wave-uniform: scalar registers and scalar branches
    const uint32_t c0 = __builtin_amdgcn_readfirstlane(pptr[p]);
    const uint32_t c1 = __builtin_amdgcn_readfirstlane(pptr[p + 1]);
    const uint32_t cl = c1 - 1;  // used only when the panel has a chunk (c < c1)
    uint32_t c = c0 + __builtin_amdgcn_readfirstlane(wv) * U;
    if (c < c1) {
      // Software pipeline over batches of U chunks in two register sets used
      // in turn: batch k+1 is issued into one set before batch k is tested
      // from the other, so the test waits only for batch k's loads. (A copy
      // from a "next" set into a "current" one would wait for the batch in
      // flight.) The bases of a batch are one vector load, issued a batch
      // ahead and before the slice and window loads it precedes.
      // A counted loop with its exit at the bottom and loads issued
      // unconditionally (past the end they read the clamped last chunk), so
      // the wait before each test is the same on every path: the batch
      // tested has landed while the one issued after it is still in flight.
      // The wave's batches start at c, c + STEP, ...; nb of them hold chunks.
      const uint32_t nb = (c1 - c + STEP - 1) / STEP;
      PanelBatch A, B;
      uint32_t bn[U];
      work += static_cast<long long>(kPanelChunk) * ((nb - 1) * U + min(U, c1 - c - (nb - 1) * STEP));
      // (the scheduling barriers keep each batch's loads together and in
      // this order, so the wait counts below are the same on every path)
      panel_bases(pp, c, cl, bn);
      __builtin_amdgcn_sched_barrier(0);
      panel_issue(pp, A, c, cl, lane, bn);
      panel_bases(pp, c + STEP, cl, bn);
      __builtin_amdgcn_sched_barrier(0);
      panel_issue(pp, B, c + STEP, cl, lane, bn);
      panel_bases(pp, c + 2 * STEP, cl, bn);
      __builtin_amdgcn_sched_barrier(0);
      uint32_t k = 0;
      for (; k + 2 < nb; k += 2) {
        panel_test_batch(A, dmask, rshift, pm);
        __builtin_amdgcn_sched_barrier(0);
        panel_issue(pp, A, c + (k + 2) * STEP, cl, lane, bn);
        panel_bases(pp, c + (k + 3) * STEP, cl, bn);
        __builtin_amdgcn_sched_barrier(0);
        panel_test_batch(B, dmask, rshift, pm);
        __builtin_amdgcn_sched_barrier(0);
        panel_issue(pp, B, c + (k + 3) * STEP, cl, lane, bn);
        panel_bases(pp, c + (k + 4) * STEP, cl, bn);
        __builtin_amdgcn_sched_barrier(0);
      }
      panel_test_batch(A, dmask, rshift, pm);
      if (k + 1 < nb) panel_test_batch(B, dmask, rshift, pm);
    }
    __syncthreads();
    const size_t wb = static_cast<size_t>(p) * W;
    uint32_t st[kParts] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    for (uint32_t j = threadIdx.x; j < W; j += BLOCK) {
      const uint32_t m = gather8(pm64[4 * j]) | (gather8(pm64[4 * j + 1]) << 8) | (gather8(pm64[4 * j + 2]) << 16) |
                         (gather8(pm64[4 * j + 3]) << 24);
      if (fused) {
        uint32_t x = 0;
        if (m) {
          const uint32_t old = vis32[wb + j];
          x = m & ~old;
          if (x) vis32[wb + j] = old | x;
        }
        next32[wb + j] = x;
        pm[8 * j] = x;  // (this thread's own marks, read above)
        if (x) {
          // the group's five slice pointers (slice_ptr is padded on the device)
          const gptr<const uint32_t> sp = a.slice_ptr + 4 * (wb + j);
          const uint32_t tau = static_cast<uint32_t>(a.tau);
          const uint4 s4 = *(gptr<const uint4>)sp;
          const uint32_t spt[5] = {s4.x, s4.y, s4.z, s4.w, sp[4]};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t ns = (x >> (8 * k)) & 0xffu ? spt[k + 1] - spt[k] : 0u;
            st[1] += ns;
            st[7] += (ns + tau - 1) / tau;
          }
        }
        continue;
      }
      if (!m) continue;
      const uint32_t x = m & ~vis32[wb + j];
      if (!x) continue;
      uint32_t q[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t nib = (x >> (4 * k)) & 0xfu;
        q[k] = (nib & 1u) | ((nib & 2u) << 7) | ((nib & 4u) << 14) | ((nib & 8u) << 21);
      }
      mark16[2 * (wb + j)] = make_uint4(q[0], q[1], q[2], q[3]);
      mark16[2 * (wb + j) + 1] = make_uint4(q[4], q[5], q[6], q[7]);
    }
    if (fused) {
      __syncthreads();
      panel_count_rows<BLOCK>(a, pm, static_cast<uint32_t>(p) << rb, W, new_level, st);
#pragma unroll
      for (int f = 0; f < kParts; ++f) {
        const uint32_t t = wave_sum(st[f]);
        if (lane == 0 && t)
          __hip_atomic_fetch_add(&s_part[f], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();
  }
  for (uint32_t j = threadIdx.x; j < 8 * W; j += BLOCK) pm[j] = 0xffffffffu;
  if (fused) {
    // every workgroup stores its partials (zero if it owns no panel)
    __syncthreads();
    if (threadIdx.x < kParts)
      a.part[static_cast<long long>(threadIdx.x) * gridDim.x + blockIdx.x] = s_part[threadIdx.x];
  }
  return lane == 0 ? work : 0;
}

// E1: push over the CSR rows of the frontier vertices.
template <int SIGMA, bool REC>
__device__ __attribute__((noinline)) long long engine_push(args_ref<BfsArgs> a_, int sel, long long nlight,
                                                           long long nheavy, long long gwave, long long nwaves,
                                                           lptr<int> hs) {
  args_ref<BfsArgs> a = uniform_args(a_);
  sel = uniform(sel);
  nlight = uniform(nlight);
  nheavy = uniform(nheavy);
  gwave = uniform(gwave);
  nwaves = uniform(nwaves);
  long long work = 0;
  using M = typename MaskOf<SIGMA>::T;
  gptr<const M> __restrict__ vis = (gptr<const M>)a.vis;
  gptr<const int32_t> __restrict__ rp = a.rp;
  gptr<const int32_t> __restrict__ col = a.col;
  gptr<uint8_t> __restrict__ mark = a.mark;
  const int lane = lane_id();
  gptr<const unsigned long long> __restrict__ heavy = a.fheavy[sel];
  for (long long i = gwave; i < nheavy; i += nwaves) {
    const unsigned long long e = heavy[i];
    const int u = static_cast<int>(e >> 32);
    const row_pos b = rp[u] + static_cast<uint32_t>(e);
    const row_pos end = row_part_end(b, kHeavyChunk, rp[u + 1]);
    for (row_pos p = b + lane; p < end; p += 64) {
      const int v = col[p];
      ++work;
      if (!((vis[v / SIGMA] >> (v % SIGMA)) & 1u)) {
        mark[v] = 1;
        if (REC) record_set(hs, v / SIGMA, a.ctl);
      }
    }
  }
  // Light vertices, 64 per wave step: the wave walks the concatenation of
  // their rows, 64 edges at a time; each lane finds the vertex owning its edge
  // by a binary search over the wave's prefix sums of the degrees, so every
  // lane has an edge (not a vertex's serial chain of loads) in flight.
  gptr<const int32_t> __restrict__ light = a.flight[sel];
  for (long long base = gwave * 64; base < nlight; base += nwaves * 64) {
    const long long i = base + lane;
    int p0 = 0, d = 0;
    if (i < nlight) {
      const int u = light[i];
      p0 = rp[u];
      d = rp[u + 1] - p0;
    }
    const int incl = wave_inclusive_scan(d);
    const int total = __shfl(incl, 63, 64);
    work += lane == 0 ? total : 0;
    for (int e0 = 0; e0 < total; e0 += 64) {
      const int e = e0 + lane;
      int lo = 0;
#pragma unroll
      for (int stp = 32; stp >= 1; stp >>= 1)
        if (__shfl(incl, lo + stp - 1, 64) <= e) lo += stp;
      const int owner = lo & 63;
      const int start = __shfl(incl, owner, 64) - __shfl(d, owner, 64);
      const int op0 = __shfl(p0, owner, 64);
      if (e < total) {
        const int v = col[op0 + (e - start)];
        if (!((vis[v / SIGMA] >> (v % SIGMA)) & 1u)) {
          mark[v] = 1;
          if (REC) record_set(hs, v / SIGMA, a.ctl);
        }
      }
    }
  }
  return work;
}

// E2: bottom-up (Alg. 4). A lane owns a vertex of each of kPullChunks chunks
// of 64 and scans its row to its first frontier neighbour, all chunks together:
// kPullBlocks blocks of four columns are loaded at a time, then their front
// words block by block; a row longer than kPullLight goes over to the whole
// wave, 64 neighbours per step, after kPullTry of them. On small and medium
// graphs the chain of loads of a step (columns, their front words) bounds it,
// times the steps of the longest row in flight, with two waves per SIMD: with a
// chunk at a time, and every long row scanned by the wave from its start, the
// step at which a 1 M vertex R-MAT (30 M arcs) is first searched bottom-up took
// 87 us, with two chunks and the lanes' tries 23. Where most rows are read to
// their end it is the rate of L2 requests (270 G/s: a front word each, and a
// block of columns), and on large graphs the rows in flight, a 128-byte line
// each, push the front words out of the L2. A line is then fetched again for
// every block: a first step on a 2^24-vertex uniform graph (268 M arcs) took
// 1,435 us a block at a time and 1,260 with two; on 2^22 vertices 295 and 275.
// Four blocks: 1,125 and 265, but 46 instead of 43 us at the dense levels of a
// 4 M vertex R-MAT, whose rows end in the first one.
constexpr int kPullLight = 32;
constexpr int kPullTry = 16;
constexpr int kPullChunks = 2;
constexpr int kPullBlocks = 2;

// Scans columns q[k] .. lim[k] of U rows of this lane, each to its first
// neighbour in front; bit k of the result: found, q[k] past the columns
// tested. (One 16-byte load per block of four neighbours: col is padded by 4
// entries, so the load stays in bounds at the end of the array.)
template <int SIGMA, int U>
__device__ __forceinline__ uint32_t pull_scan(gptr<const int32_t> col, gptr<const typename MaskOf<SIGMA>::T> front,
                                              row_pos (&q)[U], const row_pos (&lim)[U]) {
  using M = typename MaskOf<SIGMA>::T;
  constexpr int B = kPullBlocks;
  uint32_t found = 0;
  for (;;) {
    bool more = false;
    int c[U][B][4];
#pragma unroll
    for (int k = 0; k < U; ++k) more |= q[k] < lim[k] && !((found >> k) & 1u);
    if (!__ballot(more)) return found;
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const bool open = !((found >> k) & 1u);
#pragma unroll
      for (int b = 0; b < B; ++b) {
#pragma unroll
        for (int t = 0; t < 4; ++t) c[k][b][t] = 0;
        if (open && row_has(q[k], 4 * b, lim[k]))
          __builtin_memcpy(c[k][b], reinterpret_cast<const int32_t*>(col + (q[k] + 4 * b)), sizeof(c[k][b]));
      }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      bool on[U];
      more = false;
#pragma unroll
      for (int k = 0; k < U; ++k) {
        on[k] = q[k] < lim[k] && !((found >> k) & 1u);
        more |= on[k];
      }
      if (b > 0 && !__ballot(more)) return found;
      M w[U][4];
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          w[k][t] = on[k] && row_has(q[k], t, lim[k]) ? front[static_cast<uint32_t>(c[k][b][t]) / SIGMA] : M(0);
#pragma unroll
      for (int k = 0; k < U; ++k) {
        bool hit = false;
#pragma unroll
        for (int t = 0; t < 4; ++t) hit |= (w[k][t] >> (static_cast<uint32_t>(c[k][b][t]) % SIGMA)) & 1u;
        if (hit) found |= 1u << k;
        if (on[k]) q[k] += 4;
      }
    }
  }
}

// The whole wave scans columns p .. e of one row; whether one is in front.
template <int SIGMA>
__device__ __forceinline__ bool pull_scan_wave(gptr<const int32_t> col, gptr<const typename MaskOf<SIGMA>::T> front,
                                               row_pos p, row_pos e, uint32_t& work) {
  for (; p < e; p += 64) {
    const row_pos i = p + lane_id();
    bool f = false;
    if (i < e) {
      const uint32_t v = static_cast<uint32_t>(col[i]);
      f = (front[v / SIGMA] >> (v % SIGMA)) & 1u;
      ++work;
    }
    if (__ballot(f)) return true;
  }
  return false;
}

template <int SIGMA>
__device__ __attribute__((noinline)) long long engine_pull(args_ref<BfsArgs> a_, int sel, long long gw,
                                                           long long nw) {
  args_ref<BfsArgs> a = uniform_args(a_);
  sel = uniform(sel);
  uint32_t work = 0;
  using M = typename MaskOf<SIGMA>::T;
  constexpr int U = kPullChunks;
  gptr<const M> __restrict__ vis = (gptr<const M>)a.vis;
  gptr<const M> __restrict__ front = (gptr<const M>)front_buf(a, sel);
  gptr<const M> __restrict__ degm = (gptr<const M>)a.degmask_in;
  gptr<const int32_t> __restrict__ rp = a.rp_in;
  gptr<const int32_t> __restrict__ col = a.col_in;
  gptr<uint8_t> __restrict__ mark = a.mark;
  const long long nv = a.nsets * SIGMA;
  const int lane = lane_id();
  // 64-vertex chunks: round k gives the waves chunks k*nw .. k*nw + nw - 1,
  // rotated by k, so chunks with heavy rows that recur with a fixed stride
  // (a relabelling that puts each window's hubs first) spread over all waves
  const int nchunks = static_cast<int>((nv + 63) / 64), waves = uniform(static_cast<int>(nw));
  int turn = uniform(static_cast<int>(gw));
  for (int round0 = 0; round0 < nchunks; round0 += U * waves) {
    uint32_t u[U];
    row_pos p[U], e[U], q[U], lim[U];
    bool cand[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int chunk = round0 + k * waves + turn;
      turn = turn + 1 == waves ? 0 : turn + 1;
      u[k] = static_cast<uint32_t>(chunk) * 64u + static_cast<uint32_t>(lane);
      cand[k] = false;
      if (chunk < nchunks && u[k] < nv) {
        const M unv = static_cast<M>(~vis[u[k] / SIGMA] & degm[u[k] / SIGMA]);
        cand[k] = (unv >> (u[k] % SIGMA)) & 1u;
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      p[k] = e[k] = 0;
      if (cand[k]) {
        p[k] = rp[u[k]];
        e[k] = rp[u[k] + 1];
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      q[k] = p[k];
      lim[k] = e[k] - p[k] > kPullLight ? p[k] + kPullTry : e[k];
    }
    const uint32_t found = pull_scan<SIGMA, U>(col, front, q, lim);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const bool f = (found >> k) & 1u;
      work += min(q[k], lim[k]) - p[k];
      if (f) mark[u[k]] = 1;
      unsigned long long hb = __ballot(!f && lim[k] < e[k]);
      while (hb) {
        const int l = __builtin_ctzll(hb);
        hb &= hb - 1;
        if (pull_scan_wave<SIGMA>(col, front, __builtin_amdgcn_readlane(lim[k], l),
                                  __builtin_amdgcn_readlane(e[k], l), work) &&
            lane == l)
          mark[u[k]] = 1;
      }
    }
  }
  return work;
}

// Runs one engine and adds the adjacency entries it read to the level's
// F_WORK counter (one atomic per block).
// SINGLE: single-workgroup level, marked slice sets are recorded in hs (only
// the BVSS and push engines run there). pm: LDS scratch for the panel-blocked
// BVSS step, which only grid levels take. (Neither pointer is tested: LDS
// offset 0 is a valid address that compares equal to a null pointer.)
// fuse_level >= 0: a panel step also does Stage 2 for that new level.
template <int SIGMA, class SliceT, int BLOCK, bool SINGLE>
__device__ __forceinline__ void run_engine(args_ref<BfsArgs> a, int engine, int sel, int slot, const LevelView& v,
                                           long long gwave, long long nwaves, lptr<int> hs, lptr<uint32_t> pm,
                                           int fuse_level = -1) {
  __shared__ long long lds_work[BLOCK / 64];
  long long work[1];
  constexpr bool kPanelFmt = SIGMA == 8 && sizeof(SliceT) == 4;
  if (kPanelFmt && engine == BLEST_ENGINE_BVSS && !SINGLE && use_panel(a, v))
    work[0] = engine_panel<BLOCK>(a, pm, sel, fuse_level);
  else if (engine == BLEST_ENGINE_BVSS)
    work[0] = engine_bvss<SIGMA, SliceT, SINGLE>(a, sel, v.queue, gwave, nwaves, hs);
  else if (engine == BLEST_ENGINE_PUSH)
    work[0] = engine_push<SIGMA, SINGLE>(a, sel, v.light, v.heavy, gwave, nwaves, hs);
  else
    work[0] = engine_pull<SIGMA>(a, sel, gwave, nwaves);
  if (a.count_work || a.probe) {
    block_sum64<BLOCK, 1>(work, lds_work);
    if (threadIdx.x == 0 && work[0]) add_u64(&a.ctl->acc[slot][F_WORK][0], static_cast<unsigned long long>(work[0]));
  }
}

// ------------------------------------------------------------ Stage 2

// Stage 2 over windows of SPT * BLOCK slice sets; set_at(win, k) gives the set
// handled by this thread in slot k of window win, or -1. MODE:
//  FIN_ATOMIC  marks -> visited/frontier/levels, and the lists, with output
//              space reserved per window by one device atomic per list;
//  FIN_LOCAL   the same with the block-local cursors `local` (one workgroup
//              alone: no atomics; the caller stores the totals);
//  FIN_COUNT   marks -> visited/frontier/levels and counts only: every set's
//              frontier word is rewritten (0 if it gained nothing); no list is
//              written;
//  FIN_EMIT    no state change: the frontier words written by FIN_COUNT give
//              the new vertices, and the lists asked for (want_push,
//              want_queue) are written from the cursors `local`, which the
//              caller presets to this block's offsets.
// The modes that update state add to st[] the level's frontier, queued slices,
// frontier edges, degree >= 32, degree >= 1024, light, heavy and queue entries
// (all below 2^31), whichever lists are written.
//
// A lane reads a set's marks and visited word, but the new vertices are
// handled a lane each: lane i of group j takes bit i % sigma of the word that
// lane j * 64 / sigma + i / sigma holds, so row pointers and input ids of 64
// consecutive vertices are coalesced loads. (A lane that walked its set's
// vertices itself issued 9 + 8 loads and 8 stores of its own per set, 64 cache
// lines each, for 4 sets: 15 us of a 25 to 30 us level of a 1 M vertex graph,
// 64 of whose 256 workgroups had a window.) What remains is a chain of four
// round trips to memory: marks; visited words; slice and row pointers and
// input ids; levels.
// Queue descriptors and heavy edge chunks are written wave-cooperatively: each
// lane finds the run that owns its output index by a binary search over the
// wave's prefix sums, so a hub set with thousands of VSSs costs a few steps.
enum FinMode : int { FIN_ATOMIC = 0, FIN_LOCAL = 1, FIN_COUNT = 2, FIN_EMIT = 3 };

// Slice sets per thread in one window: 1 where that already gives every
// workgroup a window at most (then the windows spread over the most
// workgroups), else 4, whose loads are issued together.
constexpr int kFinSpt = 4;
__device__ __forceinline__ bool fin_wide(args_ref<BfsArgs> a, int block) {
  return a.nsets > 2LL * block * static_cast<long long>(gridDim.x);
}

// The output run that holds index i: the lane whose inclusive prefix sum is
// the first above i.
__device__ __forceinline__ int run_owner(int incl, int i) {
  int lo = 0;
#pragma unroll
  for (int stp = 32; stp >= 1; stp >>= 1)
    if (__shfl(incl, lo + stp - 1, 64) <= i) lo += stp;
  return lo & 63;
}

// Whether a level may be explored by push (the vertex lists are needed).
__device__ __forceinline__ bool push_possible(args_ref<BfsArgs> a) {
  return a.probe || (a.policy != BLEST_POLICY_HEURISTIC && a.policy != BLEST_POLICY_BVSS &&
                     a.policy != BLEST_POLICY_BOTTOM_UP);
}

template <int SIGMA, int BLOCK, int MODE, int SPT, class SetAt>
__device__ __forceinline__ void finalize_windows(args_ref<BfsArgs> a, int new_level, gptr<unsigned long long> acc,
                                                 int sel_out, int win0, int nwin, int wstep, SetAt set_at,
                                                 uint32_t (&st)[kParts], lptr<uint32_t> local, bool want_push,
                                                 bool want_queue) {
  using M = typename MaskOf<SIGMA>::T;
  constexpr bool UPDATE = MODE != FIN_EMIT;
  constexpr int GB = 8;  // groups of 64 vertices whose loads are issued together (a wave's 64 sets have SIGMA)
  __shared__ int lds32[3 * (BLOCK / 64)];
  __shared__ uint32_t bases[3];
  gptr<M> __restrict__ vis = (gptr<M>)a.vis;
  gptr<M> __restrict__ front = (gptr<M>)front_buf(a, sel_out);
  gptr<uint8_t> __restrict__ mark = a.mark;
  gptr<const int32_t> __restrict__ rp = a.rp;
  gptr<const uint32_t> __restrict__ sp = a.slice_ptr;
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  gptr<int32_t> __restrict__ levels = a.levels;
  const gptr<const int32_t> __restrict__ orig_id = a.orig_id;
  const int lane = lane_id();
  const int vbit = lane % SIGMA, vset = lane / SIGMA;  // this lane's vertex in a group: bit, set of the group
  const bool need_sp = UPDATE || want_queue;
  for (int win = win0; win < nwin; win += wstep) {
    M nw[SPT];
    int sset[SPT];
    int nq[SPT];
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      const int s = set_at(win, k);
      sset[k] = s;
      nw[k] = 0;
      nq[k] = 0;
      if (s >= 0) {
        if constexpr (UPDATE)
          nw[k] = load_marks<SIGMA>(mark + static_cast<long long>(s) * SIGMA);
        else
          nw[k] = front[s];
      }
    }
    if constexpr (UPDATE) {
      M old[SPT];
#pragma unroll
      for (int k = 0; k < SPT; ++k) old[k] = nw[k] ? vis[sset[k]] : M(0);
#pragma unroll
      for (int k = 0; k < SPT; ++k) {
        const int s = sset[k];
        if (s < 0) continue;
        const M x = static_cast<M>(nw[k] & ~old[k]);
        if (nw[k]) clear_marks<SIGMA>(mark + static_cast<long long>(s) * SIGMA);
        if (x) vis[s] = static_cast<M>(old[k] | x);
        if (MODE == FIN_COUNT || x) front[s] = x;
        nw[k] = x;
      }
    }
    uint32_t p0[SPT], p1[SPT];
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      p0[k] = p1[k] = 0;
      if (nw[k] && need_sp) {
        p0[k] = sp[sset[k]];
        p1[k] = sp[sset[k] + 1];
      }
    }
    int nl = 0, nh = 0;
    if (UPDATE || want_push) {
#pragma unroll
      for (int k = 0; k < SPT; ++k) {
        if (!__ballot(nw[k] != 0)) continue;
#pragma unroll 1
        for (int j0 = 0; j0 < SIGMA; j0 += GB) {
          bool on[GB];
          int u[GB], r0[GB], r1[GB], id[GB];
#pragma unroll
          for (int j = 0; j < GB; ++j) {
            const int owner = (j0 + j) * (64 / SIGMA) + vset;
            on[j] = (static_cast<uint32_t>(__shfl(static_cast<int>(nw[k]), owner, 64)) >> vbit) & 1u;
            u[j] = __shfl(sset[k], owner, 64) * SIGMA + vbit;
          }
#pragma unroll
          for (int j = 0; j < GB; ++j) {
            r0[j] = r1[j] = id[j] = 0;
            if (on[j]) {
              r0[j] = rp[u[j]];
              r1[j] = rp[u[j] + 1];
              if constexpr (UPDATE) id[j] = orig_id ? orig_id[u[j]] : u[j];
            }
          }
#pragma unroll
          for (int j = 0; j < GB; ++j) {
            if (!on[j]) continue;
            const int d = r1[j] - r0[j];
            if constexpr (UPDATE) {
              levels[id[j]] = new_level;
              st[0] += 1;
              st[2] += static_cast<uint32_t>(d);
              st[3] += d >= 32;
              st[4] += d >= 1024;
            }
            if (d > kLightMax)
              nh += (d + kHeavyChunk - 1) / kHeavyChunk;
            else
              nl += 1;
          }
        }
      }
    }
    int cnt[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      if (nw[k] && need_sp) {
        const uint32_t ns = p1[k] - p0[k];
        nq[k] = static_cast<int>((ns + tau - 1) / tau);
        if constexpr (UPDATE) st[1] += ns;
      }
      cnt[2] += nq[k];
    }
    if constexpr (UPDATE) {
      st[5] += static_cast<uint32_t>(nl);
      st[6] += static_cast<uint32_t>(nh);
      st[7] += static_cast<uint32_t>(cnt[2]);
    }
    if constexpr (MODE == FIN_COUNT) continue;
    if (want_push) {
      cnt[0] = nl;
      cnt[1] = nh;
    }
    if (!__syncthreads_or(cnt[0] | cnt[1] | cnt[2])) continue;
    int ex[3], tot[3];
    block_exclusive_scan<BLOCK, 3>(cnt, ex, tot, lds32);
    if (threadIdx.x < 3) {
      const int f = threadIdx.x;
      const uint32_t t = static_cast<uint32_t>(f == 0 ? tot[0] : f == 1 ? tot[1] : tot[2]);
      if (MODE != FIN_ATOMIC) {
        bases[f] = local[f];
        local[f] += t;
      } else {
        bases[f] = t ? static_cast<uint32_t>(
                           fetch_add_u64(acc + (f == 0 ? F_LIGHT : f == 1 ? F_HEAVY : F_QUEUE) * kPad, t))
                     : 0u;
      }
    }
    __syncthreads();
    if (want_push) {
      // light vertices and heavy edge chunks, group by group
      gptr<int32_t> __restrict__ light = a.flight[sel_out];
      gptr<unsigned long long> __restrict__ heavy = a.fheavy[sel_out];
      uint32_t ol = bases[0] + ex[0], oh = bases[1] + ex[1];
#pragma unroll
      for (int k = 0; k < SPT; ++k) {
        if (!__ballot(nw[k] != 0)) continue;
#pragma unroll 1
        for (int j0 = 0; j0 < SIGMA; j0 += GB) {
          int u[GB], d[GB];
#pragma unroll
          for (int j = 0; j < GB; ++j) {
            const int owner = (j0 + j) * (64 / SIGMA) + vset;
            const bool on = (static_cast<uint32_t>(__shfl(static_cast<int>(nw[k]), owner, 64)) >> vbit) & 1u;
            u[j] = __shfl(sset[k], owner, 64) * SIGMA + vbit;
            d[j] = on ? rp[u[j] + 1] - rp[u[j]] : -1;
          }
#pragma unroll
          for (int j = 0; j < GB; ++j) {
            if (d[j] >= 0 && d[j] <= kLightMax) light[ol++] = u[j];
            const int nch = d[j] > kLightMax ? (d[j] + kHeavyChunk - 1) / kHeavyChunk : 0;
            if (!__ballot(nch != 0)) continue;
            const int incl = wave_inclusive_scan(nch);
            const int total = __builtin_amdgcn_readlane(incl, 63);
            for (int b0 = 0; b0 < total; b0 += 64) {
              const int i = b0 + lane, o = run_owner(incl, i);
              const int c = i - (__shfl(incl, o, 64) - __shfl(nch, o, 64));
              const uint32_t at = static_cast<uint32_t>(__shfl(static_cast<int>(oh), o, 64)) + c;
              const uint32_t ou = static_cast<uint32_t>(__shfl(u[j], o, 64));
              if (i < total)
                heavy[at] = (static_cast<unsigned long long>(ou) << 32) |
                            static_cast<unsigned long long>(c * kHeavyChunk);
            }
            oh += nch;
          }
        }
      }
    }
    if (want_queue) {
      gptr<uint4> __restrict__ queue = a.queue[sel_out];
      uint32_t oq = bases[2] + ex[2];
#pragma unroll
      for (int k = 0; k < SPT; ++k) {
        const int incl = wave_inclusive_scan(nq[k]);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        for (int b0 = 0; b0 < total; b0 += 64) {
          const int i = b0 + lane, o = run_owner(incl, i);
          const uint32_t c = static_cast<uint32_t>(i - (__shfl(incl, o, 64) - __shfl(nq[k], o, 64)));
          const uint32_t at = static_cast<uint32_t>(__shfl(static_cast<int>(oq), o, 64)) + c;
          const uint32_t s0 = static_cast<uint32_t>(__shfl(static_cast<int>(p0[k]), o, 64)) + c * tau;
          const uint32_t end = static_cast<uint32_t>(__shfl(static_cast<int>(p1[k]), o, 64));
          const uint32_t bits = static_cast<uint32_t>(__shfl(static_cast<int>(nw[k]), o, 64));
          const uint32_t s = static_cast<uint32_t>(__shfl(sset[k], o, 64));
          if (i < total) queue[at] = make_uint4(s0, min(tau, end - s0), bits, s);
        }
        oq += nq[k];
      }
    }
    __syncthreads();
  }
}

// Stage 2 of the whole grid (per-stage launches): every slice set, windows
// spread over the blocks, statistics added to the level's slot (block 0 also
// carries the cumulative counts of the previous level).
template <int SIGMA, int BLOCK>
__device__ __forceinline__ void finalize(args_ref<BfsArgs> a, int new_level, int slot_out, int sel_out, long long cumv_in,
                                         long long cume_in) {
  __shared__ uint32_t lds[kParts * (BLOCK / 64)];
  const gptr<unsigned long long> acc = (&a.ctl->acc[slot_out][0][0]);
  uint32_t st[kParts] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  const int nsets = static_cast<int>(a.nsets), tid = threadIdx.x;
  finalize_windows<SIGMA, BLOCK, FIN_ATOMIC, 1>(a, new_level, acc, sel_out, blockIdx.x, (nsets + BLOCK - 1) / BLOCK,
                                                gridDim.x,
                                                [=](int win, int) -> int {
                                                  const int s = win * BLOCK + tid;
                                                  return s < nsets ? s : -1;
                                                },
                                                st, nullptr, push_possible(a), true);
  const uint32_t t = block_sum32<BLOCK, kParts>(st, to_lds(lds));
  if (tid < 5) {
    constexpr int f[5] = {F_FRONTIER, F_QSLICES, F_FEDGES, F_DEG32, F_DEG1024};
    if (t) add_u64(acc + f[tid] * kPad, t);
    const int cum = tid == 0 ? F_CUMV : F_CUME;
    const long long in = blockIdx.x ? 0 : tid == 0 ? cumv_in : cume_in;
    if ((tid == 0 || tid == 2) && (t || in)) add_u64(acc + cum * kPad, t + static_cast<unsigned long long>(in));
  }
}

// ------------------------------------------------- two-phase grid Stage 2
//
// In the persistent kernel a grid level's Stage 2 runs in two phases with no
// device atomics. Count: every workgroup sweeps its windows (marks ->
// visited/frontier/levels) and stores its partial counters with plain stores.
// After the barrier every workgroup sums the partials in the same order, so
// all of them hold the same level statistics and pick the same engine for
// the next level, and each knows the sum of the list sizes of the workgroups
// before it. Emit: only when that engine reads a list (the VSS queue for BVSS
// over the queue, the vertex lists for push; all lists in probe mode) do the
// workgroups sweep again and write it at those offsets, behind one more
// barrier. Bottom-up and panel levels skip the emit phase.

// MODE = FIN_COUNT (counts only) or FIN_ATOMIC (lists too, output space
// reserved with one device atomic per window and list on the cursors of
// slot `slot_out`); either way the level statistics go to the partials
// (field f of workgroup b at f * gridDim.x + b, so that a wave reads a field
// of all workgroups with coalesced loads).
template <int SIGMA, int BLOCK, int MODE, int SPT>
__device__ __attribute__((noinline)) void finalize_count(args_ref<BfsArgs> a_, int new_level, int slot_out,
                                                         int sel_out) {
  args_ref<BfsArgs> a = uniform_args(a_);
  new_level = uniform(new_level);
  slot_out = uniform(slot_out);
  sel_out = uniform(sel_out);
  constexpr int WIN = BLOCK * SPT;
  __shared__ uint32_t lds[kParts * (BLOCK / 64)];
  uint32_t st[kParts] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  const int nsets = static_cast<int>(a.nsets), tid = threadIdx.x;
  finalize_windows<SIGMA, BLOCK, MODE, SPT>(a, new_level, (&a.ctl->acc[slot_out][0][0]), sel_out, blockIdx.x,
                                            (nsets + WIN - 1) / WIN, gridDim.x,
                                            [=](int win, int k) -> int {
                                              const int s = win * WIN + k * BLOCK + tid;
                                              return s < nsets ? s : -1;
                                            },
                                            st, nullptr, push_possible(a), true);
  const uint32_t t = block_sum32<BLOCK, kParts>(st, to_lds(lds));
  if (tid < kParts) a.part[static_cast<long long>(tid) * gridDim.x + blockIdx.x] = t;
}

// The view of the level after v from its counters (kParts fields).
__device__ __forceinline__ LevelView next_view(const LevelView& v, const uint32_t (&t)[kParts]) {
  return LevelView{t[0], t[7], t[1], t[2], t[3], t[4], t[5], t[6], v.cumv + t[0], v.cume + t[2]};
}

// Sums the partial counters of all workgroups (after the barrier that follows
// finalize_count). before[] = light, heavy and queue entries of the
// workgroups with a smaller index (this workgroup's list offsets).
template <int BLOCK>
__device__ __forceinline__ void reduce_parts(args_ref<BfsArgs> a, uint32_t (&tot)[kParts], uint32_t (&before)[3]) {
  __shared__ uint32_t s_tot[kParts], s_bef[3];
  const gptr<const uint32_t> part = a.part;
  const int nb = static_cast<int>(gridDim.x);
  const int me = static_cast<int>(blockIdx.x);
  const int lane = lane_id(), w = wave_in_block();
  for (int f = w; f < kParts; f += BLOCK / 64) {
    uint32_t t = 0, bs = 0;
    for (int b0 = 0; b0 < nb; b0 += 256) {
      uint32_t x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int b = b0 + j * 64 + lane;
        x[j] = b < nb ? part[static_cast<long long>(f) * nb + b] : 0u;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        t += x[j];
        bs += b0 + j * 64 + lane < me ? x[j] : 0u;
      }
    }
    t = wave_sum(t);
    bs = wave_sum(bs);
    if (lane == 0) {
      s_tot[f] = t;
      if (f >= 5) s_bef[f - 5] = bs;
    }
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < kParts; ++f) tot[f] = static_cast<uint32_t>(uniform(static_cast<int>(s_tot[f])));
#pragma unroll
  for (int f = 0; f < 3; ++f) before[f] = static_cast<uint32_t>(uniform(static_cast<int>(s_bef[f])));
  __syncthreads();
}

// The lists of the windows (or, panel_part, of the panels) whose counts this
// workgroup stored, at its offsets. panel_part: the counts came from the fused
// panel step, so each workgroup emits the lists of the slice sets of its own
// panels (the partition its partial counters, and hence its offsets, were
// computed over); otherwise the window partition of finalize_count.
template <int SIGMA, int BLOCK, int SPT>
__device__ __attribute__((noinline)) void finalize_emit(args_ref<BfsArgs> a_, int sel_out, uint32_t before_light,
                                                        uint32_t before_heavy, uint32_t before_queue, bool want_push,
                                                        bool want_queue, bool panel_part) {
  args_ref<BfsArgs> a = uniform_args(a_);
  sel_out = uniform(sel_out);
  constexpr int WIN = BLOCK * SPT;
  __shared__ uint32_t cursor[3];
  const int tid = threadIdx.x;
  if (tid < 3) cursor[tid] = tid == 0 ? before_light : tid == 1 ? before_heavy : before_queue;
  __syncthreads();
  uint32_t st[kParts] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  const int nsets = static_cast<int>(a.nsets);
  const gptr<unsigned long long> acc0 = (&a.ctl->acc[0][0][0]);
  // panel_part: panel p holds sets [p * sp, (p + 1) * sp); this workgroup owns
  // panels blockIdx.x, blockIdx.x + G, ...; window w is window w % wpp of its
  // (w / wpp)-th panel
  const int sp = panel_part ? 1 << (a.panel_rb - 3) : nsets;
  const int b = blockIdx.x, G = gridDim.x;
  const int wpp = (sp + WIN - 1) / WIN;
  const int mine = !panel_part ? 0 : a.npanels > b ? (a.npanels - 1 - b) / G + 1 : 0;
  finalize_windows<SIGMA, BLOCK, FIN_EMIT, SPT>(a, 0, acc0, sel_out, panel_part ? 0 : b, panel_part ? mine * wpp : wpp,
                                                panel_part ? 1 : G,
                                                [=](int win, int k) -> int {
                                                  const int p = panel_part ? b + (win / wpp) * G : 0;
                                                  const int w = panel_part ? win % wpp : win;
                                                  const int i = w * WIN + k * BLOCK + tid;  // in the panel
                                                  const long long s = static_cast<long long>(p) * sp + i;
                                                  return i < sp && s < nsets ? static_cast<int>(s) : -1;
                                                },
                                                st, to_lds(cursor), want_push, want_queue);
}

// ------------------------------------------------- single-workgroup levels
//
// A level whose Stage 1 can mark at most kSingleMaxMarks rows (BVSS: queued
// slices; push: frontier edges) is run by workgroup 0 alone: the engine
// records every slice set it marks in an LDS hash set, and Stage 2 finalises
// only those sets, with workgroup barriers instead of device-wide ones. The
// other workgroups wait on a flag until workgroup 0 reaches a level that is
// not small (or the end), then all continue together.

__device__ __forceinline__ bool single_eligible(args_ref<BfsArgs> a, int engine, const LevelView& v) {
  if (!a.single_block || a.probe) return false;
  if (engine == BLEST_ENGINE_BVSS) return v.qslices <= kSingleMaxMarks && !(a.npanels > 0 && a.panel_mode == 2);
  if (engine == BLEST_ENGINE_PUSH) return v.fedges <= kSingleMaxMarks;
  return false;
}

// Stage 2 of one workgroup over the sets recorded during Stage 1 (the LDS
// list after the hash set); empties both. Output cursors are block-local; the
// level's counters go to tot (LDS) and to the level's slot.
template <int SIGMA, int BLOCK>
__device__ __attribute__((noinline)) void finalize_list(args_ref<BfsArgs> a_, int new_level, int slot_out,
                                                        int sel_out, uint32_t cumv_in, uint32_t cume_in,
                                                        lptr<int> hs, lptr<uint32_t> tot) {
  args_ref<BfsArgs> a = uniform_args(a_);
  new_level = uniform(new_level);
  slot_out = uniform(slot_out);
  sel_out = uniform(sel_out);
  __shared__ uint32_t local[3];
  __shared__ uint32_t lds[kParts * (BLOCK / 64)];
  const int tid = threadIdx.x;
  const gptr<unsigned long long> acc = (&a.ctl->acc[slot_out][0][0]);
  if (tid < 3) local[tid] = 0u;
  __syncthreads();
  const int count = uniform(hs[kSingleHash]);
  const lptr<const int> list = hs + kSingleHash + 1;
  uint32_t st[kParts] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  finalize_windows<SIGMA, BLOCK, FIN_LOCAL, 1>(a, new_level, acc, sel_out, 0, (count + BLOCK - 1) / BLOCK, 1,
                                               [=](int win, int) -> int {
                                                 const int i = win * BLOCK + tid;
                                                 return i < count ? list[i] : -1;
                                               },
                                               st, to_lds(local), push_possible(a), true);
  const uint32_t t = block_sum32<BLOCK, kParts>(st, to_lds(lds));
  for (int i = tid; i < kSingleHash + 1; i += BLOCK) hs[i] = (i == kSingleHash) ? 0 : -1;
  auto put = [&](int f, unsigned long long v) {
    __hip_atomic_store(acc + f * kPad, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (tid < kParts) {
    constexpr int f[kParts] = {F_FRONTIER, F_QSLICES, F_FEDGES, F_DEG32, F_DEG1024, F_LIGHT, F_HEAVY, F_QUEUE};
    tot[tid] = t;
    put(f[tid], t);
    if (tid == 0) put(F_CUMV, static_cast<unsigned long long>(cumv_in) + t);
    if (tid == 2) put(F_CUME, static_cast<unsigned long long>(cume_in) + t);
  }
}

// ------------------------------------------------------- init and seeding

template <int SIGMA>
// seeded: the threads that clear the source's visited/frontier word and
// level write the source's values instead (level 0), so no barrier is needed
// between the clear and those writes.
__device__ __forceinline__ void clear_state(args_ref<BfsArgs> a, long long gtid, long long nthreads, bool seeded = false) {
  using M = typename MaskOf<SIGMA>::T;
  const gptr<M> vis = (gptr<M>)a.vis;
  const gptr<M> front0 = (gptr<M>)front_buf(a, 0), front1 = (gptr<M>)front_buf(a, 1);
  const long long src_set = seeded ? a.src / SIGMA : -1;
  const M src_bit = static_cast<M>(M(1) << (a.src % SIGMA));
  const long long src_in = seeded ? (a.orig_id ? a.orig_id[a.src] : a.src) : -1;
  for (long long i = gtid; i < a.n; i += nthreads) a.levels[i] = i == src_in ? 0 : -1;
  for (long long s = gtid; s < a.nsets; s += nthreads) {
    vis[s] = s == src_set ? src_bit : M(0);
    front0[s] = s == src_set ? src_bit : M(0);
    front1[s] = 0;
  }
  if (blockIdx.x == 0)
    for (int t = threadIdx.x; t < kStatSlots * kStatFields; t += blockDim.x)
      a.ctl->acc[t / kStatFields][t % kStatFields][0] = 0ULL;
}

// Level 0: frontier = {src}, queue = the VSSs of src's slice set. One block.
template <int SIGMA>
// lists_only: clear_state(seeded) already wrote the visited/frontier bit and level.
__device__ __forceinline__ void seed_source(args_ref<BfsArgs> a, bool lists_only = false) {
  using M = typename MaskOf<SIGMA>::T;
  const long long src = a.src;
  const long long s = src / SIGMA;
  const M bit = static_cast<M>(M(1) << (src % SIGMA));
  const uint32_t s0 = a.slice_ptr[s], ns = a.slice_ptr[s + 1] - s0;
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  const uint32_t nq = (ns + tau - 1) / tau;
  const int d = a.rp[src + 1] - a.rp[src];
  for (uint32_t k = threadIdx.x; k < nq; k += blockDim.x)
    a.queue[0][k] = make_uint4(s0 + k * tau, min(tau, ns - k * tau), static_cast<uint32_t>(bit), static_cast<uint32_t>(s));
  const int nh = d > kLightMax ? (d + kHeavyChunk - 1) / kHeavyChunk : 0;
  for (int c = threadIdx.x; c < nh; c += blockDim.x)
    a.fheavy[0][c] = (static_cast<unsigned long long>(src) << 32) | static_cast<unsigned long long>(c * kHeavyChunk);
  if (threadIdx.x == 0) {
    if (!lists_only) {
      ((gptr<M>)a.vis)[s] = bit;
      ((gptr<M>)front_buf(a, 0))[s] = bit;
      a.levels[a.orig_id ? a.orig_id[src] : src] = 0;
    }
    if (nh == 0) a.flight[0][0] = static_cast<int32_t>(src);
    const gptr<unsigned long long> acc = &a.ctl->acc[0][0][0];
    acc[F_FRONTIER * kPad] = 1;
    acc[F_QUEUE * kPad] = nq;
    acc[F_QSLICES * kPad] = ns;
    acc[F_FEDGES * kPad] = static_cast<unsigned long long>(d);
    acc[F_DEG32 * kPad] = d >= 32;
    acc[F_DEG1024 * kPad] = d >= 1024;
    acc[F_LIGHT * kPad] = nh == 0 ? 1 : 0;
    acc[F_HEAVY * kPad] = static_cast<unsigned long long>(nh);
    acc[F_CUMV * kPad] = 1;
    acc[F_CUME * kPad] = static_cast<unsigned long long>(d);
  }
}

// Stamps the start of a level's step (one lane of workgroup 0).
__device__ __forceinline__ void log_begin(args_ref<BfsArgs> a, int level) {
  if (level < a.log_cap) a.log[level].t_begin = dev_ticks();
}

// ------------------------------------------------------ persistent kernel

// Waits until every wave of the block has its memory operations performed,
// then synchronises the block.
__device__ __forceinline__ void block_sync_mem() {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
}

// Waits until workgroup 0 has finished its episode (one thread per waiting
// workgroup), bounded like a barrier; the bound restarts whenever the episode
// finishes a level, so it measures a stall, not the length of a long run of
// small levels. Returns the level it stopped at, or -1. The polls are a
// microsecond apart: they go to the memory that workgroup 0 works in.
__device__ __forceinline__ int wait_episode(args_ref<BfsArgs> a, unsigned episodes) {
  const gptr<Ctl> ctl = a.ctl;
  unsigned long long t0 = dev_ticks();
  int seen = -1;
  bool ok = true;
  while (__hip_atomic_load(&ctl->single_gen[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < episodes) {
    if (__hip_atomic_load(&ctl->error[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
      ok = false;
      break;
    }
    const int prog = __hip_atomic_load(&ctl->single_progress[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (prog != seen) {
      seen = prog;
      t0 = dev_ticks();
    }
    if (dev_ticks() - t0 > a.timeout_ticks) {
      __hip_atomic_store(&ctl->error[0], static_cast<int>(BLEST_ERR_TIMEOUT), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      ok = false;
      break;
    }
    __builtin_amdgcn_s_sleep(16);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return ok ? __hip_atomic_load(&ctl->single_level[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : -1;
}

// Workgroup 0 runs consecutive small levels alone, starting at `level` with
// its view, chosen engine and features. Returns the first level it did not
// run (its slot holds that level's statistics).
template <int SIGMA, class SliceT, int BLOCK>
__device__ __attribute__((noinline)) int single_episode(args_ref<BfsArgs> a_, int level, int engine, LevelView v,
                                                        lptr<const float> s_mlp, bool learned, lptr<int> hs) {
  args_ref<BfsArgs> a = uniform_args(a_);
  level = uniform(level);
  engine = uniform(engine);
  const long long gwave = wave_in_block(), nwaves = BLOCK / 64;
  __shared__ uint32_t s_tot[kParts];
  for (;;) {
    const int slot = level % kStatSlots, nslot = (level + 1) % kStatSlots;
    if (threadIdx.x == 0) log_begin(a, level);
    // (the next level's work counter; its other fields are stored by Stage 2)
    if (threadIdx.x == 0)
      __hip_atomic_store(&a.ctl->acc[nslot][F_WORK][0], 0ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    run_engine<SIGMA, SliceT, BLOCK, true>(a, engine, level & 1, slot, v, gwave, nwaves, hs, (lptr<uint32_t>)hs);
    block_sync_mem();
    if (threadIdx.x == 0 && level < a.log_cap) a.log[level].t_mid = dev_ticks();
    finalize_list<SIGMA, BLOCK>(a, level + 1, nslot, (level & 1) ^ 1, v.cumv, v.cume, hs, to_lds(s_tot));
    block_sync_mem();
    if (threadIdx.x == 0 && level < a.log_cap) {
      a.log[level].t_end = dev_ticks();
      a.log[level].work = static_cast<long long>(ld_relaxed_u64(&a.ctl->acc[slot][F_WORK][0]));
    }
    ++level;
    // progress for the waiting workgroups: their time bound restarts with every level
    if (threadIdx.x == 0)
      __hip_atomic_store(&a.ctl->single_progress[0], level, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t tot[kParts];
#pragma unroll
    for (int f = 0; f < kParts; ++f) tot[f] = static_cast<uint32_t>(uniform(static_cast<int>(s_tot[f])));
    v = next_view(v, tot);
    if (v.frontier == 0) return level;
    if (__hip_atomic_load(&a.ctl->error[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return level;
    engine = decide_level<false>(a, v, level, s_mlp, learned);
    if (!single_eligible(a, engine, v)) return level;
  }
}

template <int SIGMA, class SliceT, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_bfs_persistent(BfsArgs args) {
  args_ref<BfsArgs> a = kernel_args(args);
  extern __shared__ float s_mlp[];
  __shared__ __attribute__((aligned(16))) int hs[kSingleLds];
  __shared__ int s_level;
  const unsigned nblocks = gridDim.x;
  const long long nthreads = static_cast<long long>(nblocks) * BLOCK;
  const long long gtid = static_cast<long long>(blockIdx.x) * BLOCK + threadIdx.x;
  const long long gwave = static_cast<long long>(blockIdx.x) * (BLOCK / 64) + wave_in_block();
  const long long nwaves = static_cast<long long>(nblocks) * (BLOCK / 64);
  const bool learned = a.policy == BLEST_POLICY_LEARNED && a.mlp != nullptr && a.mlp->valid;
  const lptr<const float> mlp = to_lds((const float*)s_mlp);
  if (learned) mlp_to_lds((const MlpDev*)a.mlp, s_mlp);
  for (int i = threadIdx.x; i < kSingleHash + 1; i += BLOCK) hs[i] = (i == kSingleHash) ? 0 : -1;
  // state clear and level-0 seed before the registration barrier, which also
  // publishes them (one device-wide barrier at kernel start)
  clear_state<SIGMA>(a, gtid, nthreads, true);
  if (blockIdx.x == 0) {
    __syncthreads();  // block 0's counter clear before its seed counters
    seed_source<SIGMA>(a, true);
    if (threadIdx.x == 0) {
      a.ctl->single_gen[0] = 0u;
      host_status_begin(a.hstat);
    }
  }
  BarrierCtx bc;
  if (!barrier_register((Ctl*)a.ctl, &bc, a.timeout_ticks)) return;
  unsigned episodes = 0;
  int level = 0;
  constexpr bool kPanelFmt = SIGMA == 8 && sizeof(SliceT) == 4;
  LevelView v = read_level(a.ctl, 0);
  long long prev_frontier = 0;
  bool decided = false;  // engine already chosen for `level`
  int engine = 0;
  for (;;) {
    const int slot = level % kStatSlots;
    if (v.frontier == 0) break;
    if (!decided) engine = decide_level<false>(a, v, level, mlp, learned);
    decided = false;
    if (single_eligible(a, engine, v)) {
      ++episodes;
      if (blockIdx.x == 0) {
        const int next = uniform(single_episode<SIGMA, SliceT, BLOCK>(a, level, engine, v, mlp, learned, to_lds(hs)));
        block_sync_mem();
        if (threadIdx.x == 0) {
          __hip_atomic_store(&a.ctl->single_level[0], next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&a.ctl->single_gen[0], episodes, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
          // counters were updated by device atomics during the episode; drop
          // any cached copies before the plain loads of grid mode
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          s_level = next;
        }
      } else if (threadIdx.x == 0) {
        s_level = wait_episode(a, episodes);
      }
      __syncthreads();
      if (s_level < 0 || __hip_atomic_load(&a.ctl->error[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
        return;
      level = uniform(s_level);
      v = read_level(a.ctl, level % kStatSlots);
      prev_frontier = level > 0 ? read_level(a.ctl, (level + kStatSlots - 1) % kStatSlots).frontier : 0;
      continue;
    }
    if (blockIdx.x == 0) {
      if (threadIdx.x == 0) log_begin(a, level);
      const int nslot = (level + 1) % kStatSlots;
      for (int t = threadIdx.x; t < kStatFields; t += BLOCK) a.ctl->acc[nslot][t][0] = 0ULL;
    }
    const int sel = level & 1;
    // A BVSS step over the panel copy does Stage 2 itself (two-phase modes):
    // its partial counters are ready after the Stage 1 barrier.
    const bool fused = !a.probe && a.count_first != 0 && engine == BLEST_ENGINE_BVSS && kPanelFmt && use_panel(a, v);
    if (a.probe) {
      for (int e = 0; e < 3; ++e) {
        const unsigned long long t0 = dev_ticks();
        run_engine<SIGMA, SliceT, BLOCK, false>(a, e, sel, slot, v, gwave, nwaves, to_lds(hs),
                                         to_lds(reinterpret_cast<uint32_t*>(hs)));
        if (!grid_barrier((Ctl*)a.ctl, bc)) return;
        if (blockIdx.x == 0 && threadIdx.x == 0 && level < a.log_cap) a.log[level].t_engine[e] = dev_ticks() - t0;
      }
    } else {
      run_engine<SIGMA, SliceT, BLOCK, false>(a, engine, sel, slot, v, gwave, nwaves, to_lds(hs),
                                       to_lds(reinterpret_cast<uint32_t*>(hs)), fused ? level + 1 : -1);
      if (!grid_barrier((Ctl*)a.ctl, bc)) return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && level < a.log_cap) a.log[level].t_mid = dev_ticks();
    // Stage 2. When the next level is likely dense (this step was BVSS over
    // the panel copy, or bottom-up on a frontier that did not shrink, or the
    // frontier's mean degree is at least 8, so the next frontier will be much
    // larger) it will likely read no list: the two-phase form counts first
    // and writes lists only if the chosen engine needs them. Otherwise (a
    // shrinking bottom-up tail is usually followed by a small queue step)
    // the lists are built in the same pass (one device atomic per window and
    // list), which saves a barrier.
    // The level statistics come from the per-workgroup partials either way.
    const bool dense_next = (engine == BLEST_ENGINE_BOTTOM_UP && v.frontier >= prev_frontier) ||
                            (engine == BLEST_ENGINE_BVSS && kPanelFmt && use_panel(a, v)) ||
                            v.fedges >= 8LL * v.frontier;
    const bool two_phase = fused || (!a.probe && (a.count_first == 2 || (a.count_first == 1 && dense_next)));
    LevelView nv;
    bool emitted = false;
    uint32_t before[3] = {0u, 0u, 0u};
    const bool wide = fin_wide(a, BLOCK);
    {
      if (!fused) {
        const int ns = (level + 1) % kStatSlots;
        if (two_phase && wide)
          finalize_count<SIGMA, BLOCK, FIN_COUNT, kFinSpt>(a, level + 1, ns, sel ^ 1);
        else if (two_phase)
          finalize_count<SIGMA, BLOCK, FIN_COUNT, 1>(a, level + 1, ns, sel ^ 1);
        else if (wide)
          finalize_count<SIGMA, BLOCK, FIN_ATOMIC, kFinSpt>(a, level + 1, ns, sel ^ 1);
        else
          finalize_count<SIGMA, BLOCK, FIN_ATOMIC, 1>(a, level + 1, ns, sel ^ 1);
        if (!grid_barrier((Ctl*)a.ctl, bc)) return;
      }
      uint32_t tot[kParts];
      reduce_parts<BLOCK>(a, tot, before);
      nv = next_view(v, tot);
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (level < a.log_cap) a.log[level].t_count = dev_ticks();
        // the level's counters, for a single-workgroup episode that may follow
        const gptr<unsigned long long> acc = &a.ctl->acc[(level + 1) % kStatSlots][0][0];
        const long long vals[10] = {nv.frontier, nv.queue, nv.qslices, nv.fedges, nv.deg32,
                                    nv.deg1024,  nv.light, nv.heavy,   nv.cumv,   nv.cume};
        for (int f = 0; f < 10; ++f)
          __hip_atomic_store(acc + f * kPad, static_cast<unsigned long long>(vals[f]), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (nv.frontier > 0) {
      engine = decide_level<false>(a, nv, level + 1, mlp, learned);
      decided = true;
      if (two_phase) {
        const bool want_queue = engine == BLEST_ENGINE_BVSS && !(kPanelFmt && use_panel(a, nv));
        const bool want_push = engine == BLEST_ENGINE_PUSH;
        if (want_queue || want_push) {
          if (wide)
            finalize_emit<SIGMA, BLOCK, kFinSpt>(a, sel ^ 1, before[0], before[1], before[2], want_push, want_queue,
                                                 fused);
          else
            finalize_emit<SIGMA, BLOCK, 1>(a, sel ^ 1, before[0], before[1], before[2], want_push, want_queue, fused);
          emitted = true;
        }
      }
    }
    if (emitted && !grid_barrier((Ctl*)a.ctl, bc)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0 && level < a.log_cap) {
      a.log[level].t_end = dev_ticks();
      a.log[level].work = static_cast<long long>(a.ctl->acc[slot][F_WORK][0]);
    }
    prev_frontier = v.frontier;
    v = nv;
    ++level;
  }
  if (blockIdx.x == 0) {
    // Nothing reads the XCD registration after barrier_register; clear it
    // for the next launch.
    if (threadIdx.x < 8) a.ctl->xcd_blocks[threadIdx.x][0] = 0u;
    if (threadIdx.x == 8) a.ctl->xcd_active[0] = 0u;
    if (threadIdx.x == 0) {
      a.ctl->nlevels[0] = level;
      host_status_end(a.hstat, a.ctl, level);
    }
  }
}

// ------------------------------------------- eager vertex updates (Alg. 2)
//
// Alg. 2 (Section "Compute Mechanics") updates a vertex as soon as a slice
// hits it: the level is written, the vertex's bit is ORed into the next
// frontier word by an atomic whose returned value identifies the first
// writer of each slice set, and that writer enqueues the set's VSSs. There is
// no Stage 2 sweep and one device-wide barrier per level, which suits graphs
// whose rows inside a VSS are clustered (update divergence at most 25,000,
// Section "Ablation Studies"): there the scattered updates that the lazy
// scheme defers are cheap, and its per-level Stage 2 pass is what dominates
// thousands of small levels.
//
// Buffers rotate over three levels. Level l reads the frontier words F_l and
// the queue Q_l (buffers l mod 3), builds F_{l+1} and Q_{l+1} (buffers
// (l + 1) mod 3, all-zero words when the level starts), ORs F_l into the
// visited words walking Q_l, and zeroes the words of F_{l-1} walking Q_{l-1},
// which makes that buffer clean for level l + 1. (A slice set without slices,
// of vertices without out-arcs in a directed graph, is in no queue: its vertices
// enter the visited words when they are found, and the bits they leave in the
// frontier words are read by nothing, as no row has them as in-neighbours.) Visited words therefore hold
// every vertex of levels < l and possibly some of level l, so a vertex was
// reached before level l + 1 iff its bit is set in visited | F_l, whichever
// of the two copies a wave reads. The statistics of level l + 1 (the inputs
// of Eq. 3 and of the switch network) are summed by device atomics into the
// rotating counter slot (l + 1) mod 3, which level l - 1 zeroed.

__device__ __forceinline__ gptr<void> eager_front(args_ref<BfsArgs> a, int b) {
  return (gptr<char>)a.front + static_cast<long long>(b) * a.fstride;
}

// Atomic OR of a sigma-bit word (8- and 16-bit words through the aligned
// 32-bit word that holds them); returns the word's previous value.
template <int SIGMA>
__device__ __forceinline__ typename MaskOf<SIGMA>::T atomic_or_word(gptr<typename MaskOf<SIGMA>::T> p,
                                                                    typename MaskOf<SIGMA>::T bits) {
  using M = typename MaskOf<SIGMA>::T;
  if constexpr (SIGMA == 32) {
    return __hip_atomic_fetch_or(p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    const uintptr_t addr = (uintptr_t)p;
    const gptr<uint32_t> w = (gptr<uint32_t>)(addr & ~uintptr_t(3));
    const uint32_t sh = static_cast<uint32_t>(addr & 3u) * 8u;
    const uint32_t old =
        __hip_atomic_fetch_or(w, static_cast<uint32_t>(bits) << sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return static_cast<M>(old >> sh);
  }
}

constexpr int kEpList = 1024;       // vertices a frontier may have: a level of one workgroup costs 12 ns a vertex,
                                    // one of the grid 13 us (2048 x 2048 grid, 2,492 levels, kernel time of one
                                    // run: 38.3 ms with 512, 36.4 with 1024)
constexpr int kEpLog2Slots = 11, kEpSlots = 1 << kEpLog2Slots;  // table slots: at most half full
constexpr uint32_t kEpEdges = 4096;  // a level's frontier edges (so the new vertices fit the list)

struct EpisodeLds {
  int tab[kEpSlots];      // slice set, -1 empty
  uint32_t list[kEpEdges];
  uint32_t sum[2][6];     // statistics of the new level, by level parity
  int count[2];           // vertices found, by level parity
  int queued;             // VSSs exported
  // a grid level's new vertices (list, their number in found; bit 31: first of its set)
  int found;
  unsigned long long base;
};

// Per-lane counts of a level's new vertices, summed per workgroup at the end
// (each count is below 2^31, see LevelView).
struct EagerStats {
  uint32_t frontier = 0, qslices = 0, fedges = 0, deg32 = 0, deg1024 = 0, work = 0;
};

// A vertex reached at this level, by the lane that reached it first: into the
// workgroup's list (its levels, statistics and queue entries follow at the end
// of the step, for all of them together).
// A vertex without an out-arc (directed graphs only) goes into the visited words
// here: where its whole set has none, the set has no slice, so no queue brings
// its word there at the next level.
__device__ __forceinline__ void eager_write(args_ref<BfsArgs> a, uint32_t u, int new_level, EagerStats& st) {
  const int32_t deg = a.rp[u + 1] - a.rp[u];
  a.levels[a.orig_id ? a.orig_id[u] : static_cast<int32_t>(u)] = new_level;
  if (deg == 0)
    __hip_atomic_fetch_or((gptr<uint32_t>)a.vis + (u >> 5), 1u << (u & 31u), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT);
  st.frontier += 1;
  st.fedges += static_cast<uint32_t>(deg);
  st.deg32 += deg >= 32;
  st.deg1024 += deg >= 1024;
}

__device__ __forceinline__ void eager_found(args_ref<BfsArgs> a, uint32_t u, bool first, int level,
                                            lptr<EpisodeLds> L, EagerStats& st);

// The end of a step: the listed vertices' levels, statistics and, for the
// first of each set, its VSSs, with one queue reservation and one set of
// counter atomics per workgroup (one per new set and per wave, on the same
// few addresses at the memory side, took most of a level of 1,700 vertices).
template <int SIGMA, int BLOCK>
__device__ __forceinline__ void eager_finish(args_ref<BfsArgs> a, int level, lptr<EpisodeLds> L, EagerStats st) {
  __shared__ int lds32[BLOCK / 64];
  const int nslot = (level + 1) % kStatSlots;
  const gptr<uint4> q = a.queue[(level + 1) % 3];
  const gptr<const uint32_t> slp = a.slice_ptr;
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  __syncthreads();
  const int found = uniform(min(L->found, static_cast<int>(kEpEdges)));
  for (int b = 0; b < found; b += BLOCK) {
    const int i = b + static_cast<int>(threadIdx.x);
    uint32_t s = 0, s0 = 0, ns = 0;
    int nv[1] = {0}, ex[1], tot[1];
    if (i < found) {
      const uint32_t e = L->list[i], u = e & 0x7fffffffu;
      s = u / SIGMA;
      if (e >> 31) {
        s0 = slp[s];
        ns = slp[s + 1] - s0;
      }
      eager_write(a, u, level + 1, st);
      nv[0] = static_cast<int>((ns + tau - 1) / tau);
      st.qslices += ns;
    }
    block_exclusive_scan<BLOCK, 1>(nv, ex, tot, lds32);
    if (threadIdx.x == 0) L->base = tot[0] ? fetch_add_u64(&a.ctl->acc[nslot][F_QUEUE][0], tot[0]) : 0ULL;
    __syncthreads();
    const unsigned long long o = L->base + ex[0];
    for (int k = 0; k < nv[0]; ++k)
      q[o + k] = make_uint4(s0 + k * tau, min(tau, ns - k * tau), 0u, s);
    __syncthreads();
  }
  if (found) {
    const uint32_t v[5] = {st.frontier, st.qslices, st.fedges, st.deg32, st.deg1024};
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const uint32_t t = wave_sum(v[k]);
      if (lane_id() == 0 && t)
        __hip_atomic_fetch_add(&L->sum[0][k], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    if (threadIdx.x < 5) {
      constexpr int f[5] = {F_FRONTIER, F_QSLICES, F_FEDGES, F_DEG32, F_DEG1024};
      const uint32_t t = L->sum[0][threadIdx.x];
      if (t) add_u64(&a.ctl->acc[nslot][f[threadIdx.x]][0], t);
      L->sum[0][threadIdx.x] = 0u;
    }
    if (threadIdx.x == 0) L->found = 0;
  }
  if (a.count_work || a.probe) {
    const unsigned long long w = wave_sum(static_cast<unsigned long long>(st.work));
    if (lane_id() == 0 && w) add_u64(&a.ctl->acc[level % kStatSlots][F_WORK][0], w);
  }
}

__device__ __forceinline__ void eager_found(args_ref<BfsArgs> a, uint32_t u, bool first, int level,
                                            lptr<EpisodeLds> L, EagerStats& st) {
  const int i = __hip_atomic_fetch_add(&L->found, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if (i < static_cast<int>(kEpEdges)) {
    L->list[i] = u | (first ? 0x80000000u : 0u);
    return;
  }
  // the list is full: this vertex on its own (its statistics still go with
  // the workgroup's)
  eager_write(a, u, level + 1, st);
  if (!first) return;
  const uint32_t s = u / static_cast<uint32_t>(a.sigma), tau = static_cast<uint32_t>(a.tau);
  const uint32_t s0 = a.slice_ptr[s], ns = a.slice_ptr[s + 1] - s0, nv = (ns + tau - 1) / tau;
  st.qslices += ns;
  if (nv == 0) return;
  const unsigned long long o = fetch_add_u64(&a.ctl->acc[(level + 1) % kStatSlots][F_QUEUE][0], nv);
  for (uint32_t k = 0; k < nv; ++k)
    a.queue[(level + 1) % 3][o + k] = make_uint4(s0 + k * tau, min(tau, ns - k * tau), 0u, s);
}

// Top-down step of Alg. 2: a wave takes G queued VSSs at a time, reads their
// sets' frontier words from F_l and all their slices, then handles the hits.
template <int SIGMA, class SliceT, int K, int BLOCK>
__device__ __attribute__((noinline)) void eager_td_k(args_ref<BfsArgs> a_, int level, long long qlen, long long gwave,
                                                     long long nwaves, lptr<EpisodeLds> L) {
  args_ref<BfsArgs> a = uniform_args(a_);
  level = uniform(level);
  qlen = uniform(qlen);
  gwave = uniform(gwave);
  nwaves = uniform(nwaves);
  EagerStats st;
  using M = typename MaskOf<SIGMA>::T;
  constexpr int G = 4;
  const int cb = level % 3, nb = (level + 1) % 3;
  const gptr<const uint4> qg = a.queue[cb];
  gptr<const SliceT> __restrict__ sl = (gptr<const SliceT>)a.slices;
  gptr<const M> vis = (gptr<const M>)a.vis;
  gptr<const M> fc = (gptr<const M>)eager_front(a, cb);
  const gptr<M> fn = (gptr<M>)eager_front(a, nb);
  const uint32_t lane = static_cast<uint32_t>(lane_id());
  for (long long base = gwave * G; base < qlen; base += nwaves * G) {
    uint4 dl = make_uint4(0u, 0u, 0u, 0u);
    uint32_t al_l = 0;
    if (lane < G && base + lane < qlen) {
      dl = qg[base + lane];
      al_l = static_cast<uint32_t>(fc[dl.w]);
    }
    uint32_t s0[G], cn[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      s0[g] = __builtin_amdgcn_readlane(dl.x, g);
      cn[g] = __builtin_amdgcn_readlane(dl.y, g);
    }
    SliceT w[G][K];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t j = lane + 64u * k;
        st.work += j < cn[g];
        w[g][k] = (j < cn[g]) ? sl[s0[g] + j] : SliceT(0);
      }
    // (the frontier words are waited for only here, with the slices)
    SliceT al[G];
#pragma unroll
    for (int g = 0; g < G; ++g) al[g] = static_cast<SliceT>(static_cast<uint32_t>(__builtin_amdgcn_readlane(al_l, g)));
    // visited | F_l of every hit row, all loads issued before any test
    M seen[G][K];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t row = static_cast<uint32_t>(w[g][k] >> SliceFmt<SliceT>::kRowShift);
        seen[g][k] = (w[g][k] & al[g]) ? static_cast<M>(vis[row / SIGMA] | fc[row / SIGMA]) : M(~M(0));
      }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t row = static_cast<uint32_t>(w[g][k] >> SliceFmt<SliceT>::kRowShift);
        const M bit = static_cast<M>(M(1) << (row % SIGMA));
        if (!(seen[g][k] & bit)) {
          const M old = atomic_or_word<SIGMA>(fn + row / SIGMA, bit);
          if (!(old & bit)) eager_found(a, row, old == 0, level, L, st);
        }
      }
  }
  eager_finish<SIGMA, BLOCK>(a, level, L, st);
}

template <int SIGMA, class SliceT, int BLOCK>
__device__ __forceinline__ void eager_td(args_ref<BfsArgs> a, int level, long long qlen, long long gwave,
                                         long long nwaves, lptr<EpisodeLds> L) {
  switch (a.tau) {
    case 64:
      return eager_td_k<SIGMA, SliceT, 1, BLOCK>(a, level, qlen, gwave, nwaves, L);
    case 128:
      return eager_td_k<SIGMA, SliceT, 2, BLOCK>(a, level, qlen, gwave, nwaves, L);
    case 192:
      return eager_td_k<SIGMA, SliceT, 3, BLOCK>(a, level, qlen, gwave, nwaves, L);
    default:
      return eager_td_k<SIGMA, SliceT, 4, BLOCK>(a, level, qlen, gwave, nwaves, L);
  }
}

// Bottom-up step (Alg. 4) with eager updates: a lane owns a vertex, an
// unvisited vertex scans its row (the whole wave scans rows longer than
// kPullLight) for a neighbour in F_l. The wave owns all sigma vertices of each
// of its sets, so it writes their F_{l+1} words with plain stores and
// enqueues the sets that gained vertices.
template <int SIGMA, int BLOCK>
__device__ __attribute__((noinline)) void eager_bu(args_ref<BfsArgs> a_, int level, long long gwave, long long nwaves,
                                                   lptr<EpisodeLds> L) {
  args_ref<BfsArgs> a = uniform_args(a_);
  level = uniform(level);
  gwave = uniform(gwave);
  nwaves = uniform(nwaves);
  EagerStats st;
  using M = typename MaskOf<SIGMA>::T;
  const int cb = level % 3, nb = (level + 1) % 3;
  gptr<const M> vis = (gptr<const M>)a.vis;
  gptr<const M> fc = (gptr<const M>)eager_front(a, cb);
  gptr<const M> degm = (gptr<const M>)a.degmask_in;
  const gptr<M> fn = (gptr<M>)eager_front(a, nb);
  gptr<const int32_t> rp = a.rp_in;
  gptr<const int32_t> col = a.col_in;
  const long long nv = a.nsets * SIGMA;
  const int lane = lane_id();
  const int nchunks = static_cast<int>((nv + 63) / 64), waves = static_cast<int>(nwaves);
  // 64-vertex chunks, round k rotated by k (as in the lazy bottom-up engine)
  int turn = static_cast<int>(gwave);
  for (int round0 = 0; round0 < nchunks; round0 += waves) {
    const int chunk = round0 + turn;
    turn = turn + 1 == waves ? 0 : turn + 1;
    if (chunk >= nchunks) continue;
    const long long u = chunk * 64LL + lane;
    bool cand = false;
    row_pos p = 0, e = 0;
    if (u < nv) {
      const long long s = u / SIGMA;
      const M unv = static_cast<M>(~(vis[s] | fc[s]) & degm[s]);
      cand = (unv >> (u % SIGMA)) & 1u;
    }
    if (!__ballot(cand)) continue;
    if (cand) {
      p = rp[u];
      e = rp[u + 1];
    }
    row_pos q[1] = {p};
    const row_pos lim[1] = {e - p > kPullLight ? p + kPullTry : e};
    bool found = pull_scan<SIGMA, 1>(col, fc, q, lim) != 0;
    st.work += min(q[0], lim[0]) - p;
    unsigned long long hb = __ballot(!found && lim[0] < e);
    while (hb) {
      const int l = __builtin_ctzll(hb);
      hb &= hb - 1;
      if (pull_scan_wave<SIGMA>(col, fc, __builtin_amdgcn_readlane(lim[0], l), __builtin_amdgcn_readlane(e, l),
                                st.work) &&
          lane == l)
        found = true;
    }
    const unsigned long long got = __ballot(found);
    if (!got) continue;
    if (lane % SIGMA == 0) {
      const M bits = static_cast<M>(got >> lane);
      if (bits) fn[u / SIGMA] = bits;
    }
    if (found) {
      const M below = static_cast<M>((got >> (lane & ~(SIGMA - 1))) & ((1ULL << (lane % SIGMA)) - 1ULL));
      eager_found(a, static_cast<uint32_t>(u), below == 0, level, L, st);
    }
  }
  eager_finish<SIGMA, BLOCK>(a, level, L, st);
}

// ---------------------------------------- eager levels of one workgroup
//
// A run of small levels on workgroup 0 alone, the frontier kept in registers
// and LDS. What bounds such a level on the whole grid is not its work but its
// chain of dependent loads from memory that no cache holds after a device-wide
// barrier, plus the barrier itself. Here the chain stays in one compute unit
// and its L2: a vertex's columns, their visited words, an atomic OR on those
// not visited (performed in the L2: no other workgroup touches the visited
// words meanwhile), the new vertices' row pointers. A level reads the rows of
// its frontier vertices (the columns that the hits of the queued slices stand
// for; a queued set of a grid graph has 18 slices for 1 to 3 frontier
// vertices).
// Measured on a 2048 x 2048 grid graph (2,492 levels of up to 3,312 vertices):
// 51.5 ms a call when one workgroup ran levels of up to 256 queued slices
// through the grid's own functions and arguments were read from the stack, 34.3
// now (one box); 773 levels here, 6.2 us each and 12 ns a frontier vertex, 1,719
// on the grid, 13.2 us each.
// Phase A walks the rows and collects the new vertices in LDS, phase B loads
// their row and slice pointers, writes levels and sums the statistics; a hash
// table of the new vertices' slice sets tells the first vertex of a set.
// Adds set s to the table; its slot if it was not there, else -1.
__device__ __forceinline__ int ep_claim(lptr<int> tab, int s) {
  uint32_t h = (static_cast<uint32_t>(s) * 2654435761u) >> (32 - kEpLog2Slots);
  for (int probe = 0; probe < kEpSlots; ++probe, h = (h + 1) & (kEpSlots - 1)) {
    int old = -1;
    if (__hip_atomic_compare_exchange_strong(tab + h, &old, s, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP))
      return static_cast<int>(h);
    if (old == s) return -1;
  }
  return -1;
}

// Frontier vertex u into the grid scheme's words and queue (cursor in LDS);
// the first of its set adds the set's VSSs and slices to st[0], st[1]. The
// words are this workgroup's alone meanwhile, so the OR stays in its L2.
template <int SIGMA>
__device__ __forceinline__ void ep_export(gptr<typename MaskOf<SIGMA>::T> fo, gptr<uint4> qo,
                                          gptr<const uint32_t> slp, int u, uint32_t tau, lptr<int> queued,
                                          uint32_t* st) {
  using M = typename MaskOf<SIGMA>::T;
  const uint32_t s = static_cast<uint32_t>(u) / SIGMA;
  const uint32_t old = __hip_atomic_fetch_or((gptr<uint32_t>)fo + (u >> 5), 1u << (u & 31), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
  if (static_cast<M>(old >> ((s * SIGMA) & 31))) return;
  const uint32_t b0 = slp[s], ns = slp[s + 1] - b0, nv = (ns + tau - 1) / tau;
  const int off = __hip_atomic_fetch_add(queued, static_cast<int>(nv), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  for (uint32_t k = 0; k < nv; ++k) qo[off + k] = make_uint4(b0 + k * tau, min(tau, ns - k * tau), 0u, s);
  st[0] += nv;
  st[1] += ns;
}

// Whether workgroup 0 may run the level alone (the same in every workgroup).
__device__ __forceinline__ bool episode_eligible(args_ref<BfsArgs> a, const LevelView& v, int engine) {
  return a.single_block && engine == BLEST_ENGINE_BVSS && v.frontier <= kEpList && v.fedges <= kEpEdges;
}

// Runs levels from `level` (view v, queue Q_level and words F_level of the
// grid scheme; prev_queue VSSs of the level before) until one is not
// eligible, its frontier is empty or has more than kEpList vertices, and
// leaves the grid scheme's state for the level it returns, with no word of
// the level before it left in the frontier buffers. Called by workgroup 0.
typedef int i32x4_word_aligned __attribute__((ext_vector_type(4), aligned(4)));

template <int SIGMA, int BLOCK>
__device__ __attribute__((noinline)) int eager_episode(args_ref<BfsArgs> a_, int level, LevelView v,
                                                       uint32_t prev_queue, lptr<const float> s_mlp, bool learned,
                                                       lptr<EpisodeLds> L) {
  using M = typename MaskOf<SIGMA>::T;
  args_ref<BfsArgs> a = uniform_args(a_);
  level = uniform(level);
  prev_queue = uniform(static_cast<int>(prev_queue));
  constexpr int EPT = (kEpList + BLOCK - 1) / BLOCK;  // frontier vertices per thread
  const int tid = static_cast<int>(threadIdx.x), lane = lane_id();
  const gptr<const int32_t> rp = a.rp, col = a.col, orig_id = a.orig_id;
  const gptr<const uint32_t> slp = a.slice_ptr;
  const gptr<uint32_t> vis32 = (gptr<uint32_t>)a.vis;  // bit u % 32 of word u / 32, whatever sigma
  const gptr<int32_t> levels = a.levels;
  const uint32_t tau = static_cast<uint32_t>(a.tau);
  const lptr<int> tab = &L->tab[0];

  // take over the grid scheme's frontier: F_level into the list and the
  // visited words, out of the frontier buffers
  for (int i = tid; i < kEpSlots; i += BLOCK) tab[i] = -1;
  if (tid < 2) L->count[tid] = 0;
  if (tid < 12) L->sum[0][tid] = 0u;
  __syncthreads();
  {
    const gptr<M> fc = (gptr<M>)eager_front(a, level % 3), fp = (gptr<M>)eager_front(a, (level + 2) % 3);
    const gptr<const uint4> qc = a.queue[level % 3], qp = a.queue[(level + 2) % 3];
    const gptr<M> vis = (gptr<M>)a.vis;
    for (uint32_t i = tid; i < prev_queue; i += BLOCK) fp[qp[i].w] = 0;
    for (uint32_t i = tid; i < v.queue; i += BLOCK) {
      const uint32_t s = qc[i].w;
      const M bits = fc[s];
      if (bits && ep_claim(tab, static_cast<int>(s)) >= 0) {
        vis[s] = static_cast<M>(vis[s] | bits);
        for (uint32_t t = bits; t; t &= t - 1) {
          const int k = __hip_atomic_fetch_add(&L->count[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          L->list[k] = s * SIGMA + __builtin_ctz(t);
        }
      }
    }
    block_sync_mem();
    for (uint32_t i = tid; i < v.queue; i += BLOCK) fc[qc[i].w] = 0;
  }
  int cnt = uniform(L->count[0]);
  int eu[EPT], ep[EPT], ed[EPT], es[EPT];  // this thread's frontier vertices: id, first column, degree, table slot
#pragma unroll
  for (int g = 0; g < EPT; ++g) {
    const int i = g * BLOCK + tid;
    eu[g] = i < cnt ? static_cast<int>(L->list[i]) : -1;
    ep[g] = ed[g] = 0;
    es[g] = -1;
    if (eu[g] >= 0) {
      ep[g] = rp[eu[g]];
      ed[g] = rp[eu[g] + 1] - ep[g];
    }
  }
  for (int i = tid; i < kEpSlots; i += BLOCK) tab[i] = -1;
  block_sync_mem();
  if (tid == 0) L->count[0] = L->queued = 0;
  __syncthreads();
  bool big = false;
  for (int done_levels = 0;; ++done_levels) {
    const int par = done_levels & 1;
    if (tid == 0) log_begin(a, level);
    // phase A: the rows of the frontier, four columns per lane at a time
    const lptr<int> count = &L->count[par];
    auto visit = [&](const bool (&want)[4], const int (&c)[4]) {
      uint32_t w[4];
      bool on[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = want[j] ? vis32[c[j] >> 5] : ~0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        on[j] = !((w[j] >> (c[j] & 31)) & 1u);
        if (on[j])
          w[j] = __hip_atomic_fetch_or(vis32 + (c[j] >> 5), 1u << (c[j] & 31), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      unsigned long long b[4];
      int total = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        on[j] = on[j] && !((w[j] >> (c[j] & 31)) & 1u);
        b[j] = __ballot(on[j]);
        total += __popcll(b[j]);
      }
      if (total == 0) return;
      int k = 0;
      if (lane == 0) k = __hip_atomic_fetch_add(count, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      k = uniform(k);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = k + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                              static_cast<uint32_t>(b[j] >> 32),
                              __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b[j]), 0u)));
        if (on[j]) L->list[i] = static_cast<uint32_t>(c[j]);  // at most kEpEdges of them
        k += __popcll(b[j]);
      }
    };
#pragma unroll
    for (int g = 0; g < EPT; ++g) {
      if (g * BLOCK >= cnt) break;
      const int d = ed[g], p = ep[g];
      // a table slot claimed for this level's frontier is free again
      if (es[g] >= 0) tab[es[g]] = -1;
      if (!__ballot(d > 8)) {
        // short rows: a lane each (col is padded by 4 entries)
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
          if (!__ballot(d > h)) break;
          i32x4_word_aligned q = {0, 0, 0, 0};
          if (d > h) q = *(gptr<const i32x4_word_aligned>)(col + p + h);
          const bool want[4] = {d > h, d > h + 1, d > h + 2, d > h + 3};
          const int c[4] = {q.x, q.y, q.z, q.w};
          visit(want, c);
        }
      } else {
        // 256 columns of the wave's concatenated rows at a time; a lane finds
        // the row of each of its four by a binary search over the degrees'
        // prefix sums
        const int incl = wave_inclusive_scan(d);
        const int total = __shfl(incl, 63, 64);
        for (int e0 = 0; e0 < total; e0 += 256) {
          bool want[4];
          int c[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int e = e0 + 64 * j + lane;
            int lo = 0;
#pragma unroll
            for (int stp = 32; stp >= 1; stp >>= 1)
              if (__shfl(incl, lo + stp - 1, 64) <= e) lo += stp;
            const int owner = lo & 63;
            const int at = __shfl(p - (incl - d), owner, 64) + e;
            want[j] = e < total;
            c[j] = want[j] ? col[at] : 0;
          }
          visit(want, c);
        }
      }
    }
    __syncthreads();
    cnt = uniform(*count);
    big = cnt > kEpList;
    const lptr<uint32_t> sum = &L->sum[par][0];
    if (tid < 6) L->sum[par ^ 1][tid] = 0u;
    if (tid == 0) L->count[par ^ 1] = 0;
    uint32_t st[5] = {0u, 0u, 0u, 0u, 0u};  // queued VSSs, slices, frontier edges, degree >= 32, >= 1024
    const int new_level = level + 1;
    if (big) {
      // more vertices than this workgroup keeps: the grid goes on from here
      const gptr<M> fo = (gptr<M>)eager_front(a, new_level % 3);
      const gptr<uint4> qo = a.queue[new_level % 3];
      for (int i = tid; i < cnt; i += BLOCK) {
        const int u = static_cast<int>(L->list[i]);
        const int d = rp[u + 1] - rp[u];
        levels[orig_id ? orig_id[u] : u] = new_level;
        st[2] += static_cast<uint32_t>(d);
        st[3] += d >= 32;
        st[4] += d >= 1024;
        ep_export<SIGMA>(fo, qo, slp, u, tau, &L->queued, st);
      }
    } else {
      // phase B: the new vertices
      uint32_t s0[EPT], s1[EPT];
      int oid[EPT];
#pragma unroll
      for (int g = 0; g < EPT; ++g) {
        eu[g] = es[g] = -1;
        ep[g] = ed[g] = 0;
        s0[g] = s1[g] = 0u;
        oid[g] = 0;
        const int i = g * BLOCK + tid;
        if (i < cnt) {
          const int u = static_cast<int>(L->list[i]);
          eu[g] = oid[g] = u;
          ep[g] = rp[u];
          ed[g] = rp[u + 1];
          if (orig_id) oid[g] = orig_id[u];
          es[g] = ep_claim(tab, u / SIGMA);
          if (es[g] >= 0) {
            s0[g] = slp[u / SIGMA];
            s1[g] = slp[u / SIGMA + 1];
          }
        }
      }
#pragma unroll
      for (int g = 0; g < EPT; ++g) {
        if (eu[g] < 0) continue;
        levels[oid[g]] = new_level;
        ed[g] -= ep[g];
        const uint32_t ns = s1[g] - s0[g];
        st[0] += (ns + tau - 1) / tau;
        st[1] += ns;
        st[2] += static_cast<uint32_t>(ed[g]);
        st[3] += ed[g] >= 32;
        st[4] += ed[g] >= 1024;
      }
    }
    if (wave_in_block() * 64 < cnt) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        const uint32_t t = wave_sum(st[f]);
        if (lane == 0 && t) __hip_atomic_fetch_add(sum + f, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();
    const uint32_t work = v.fedges;
    v.frontier = static_cast<uint32_t>(cnt);
    v.queue = uniform(static_cast<int>(sum[0]));
    v.qslices = uniform(static_cast<int>(sum[1]));
    v.fedges = uniform(static_cast<int>(sum[2]));
    v.deg32 = uniform(static_cast<int>(sum[3]));
    v.deg1024 = uniform(static_cast<int>(sum[4]));
    v.light = v.heavy = 0u;
    v.cumv += v.frontier;
    v.cume += v.fedges;
    if (tid == 0 && level < a.log_cap) {
      const unsigned long long t = dev_ticks();
      a.log[level].t_mid = t;
      a.log[level].t_end = t;
      if (a.count_work) a.log[level].work = work;
    }
    ++level;
    // progress for the waiting workgroups: their time bound restarts with every level
    if (tid == 0) __hip_atomic_store(&a.ctl->single_progress[0], level, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v.frontier == 0 || big) break;
    if ((level & 255) == 0 && __hip_atomic_load(&a.ctl->error[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
      break;
    const int engine = decide_level<true>(a, v, level, s_mlp, learned);
    if (!episode_eligible(a, v, engine)) break;
  }
  // hand over: F_level and Q_level in the grid scheme's buffers (all frontier
  // words were zero), its statistics in the slot of its level
  if (!big) {
    const gptr<M> fo = (gptr<M>)eager_front(a, level % 3);
    uint32_t st[2] = {0u, 0u};
#pragma unroll
    for (int g = 0; g < EPT; ++g)
      if (eu[g] >= 0) ep_export<SIGMA>(fo, a.queue[level % 3], slp, eu[g], tau, &L->queued, st);
  }
  auto put = [&](int sl, int f, unsigned long long x) {
    __hip_atomic_store(&a.ctl->acc[sl % kStatSlots][f][0], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (tid < kStatFields) {
    put(level + 1, tid, 0ULL);
    put(level + 2, tid, 0ULL);
  }
  if (tid == 0) {
    put(level, F_FRONTIER, v.frontier);
    put(level, F_QUEUE, v.queue);
    put(level, F_QSLICES, v.qslices);
    put(level, F_FEDGES, v.fedges);
    put(level, F_DEG32, v.deg32);
    put(level, F_DEG1024, v.deg1024);
    put(level, F_CUMV, v.cumv);
    put(level, F_CUME, v.cume);
    put(level, F_WORK, 0ULL);
  }
  return level;
}

// One level of the eager scheme by the whole grid: bookkeeping, the engine and its counters. The caller
// synchronises afterwards.
template <int SIGMA, class SliceT, int BLOCK>
__device__ __forceinline__ void eager_level(args_ref<BfsArgs> a, int level, const LevelView& v, uint32_t prev_queue,
                                            int engine, long long gtid, long long nthreads, long long gwave,
                                            long long nwaves, lptr<EpisodeLds> L) {
  using M = typename MaskOf<SIGMA>::T;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) log_begin(a, level);
    // the slot level + 2 accumulates into during the next level
    const int zslot = (level + 2) % kStatSlots;
    for (int t = threadIdx.x; t < kStatFields; t += BLOCK)
      __hip_atomic_store(&a.ctl->acc[zslot][t][0], 0ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  {
    // F_l into the visited words (walking Q_l); F_{l-1} cleared (walking Q_{l-1}).
    // In a directed graph eager_write ORs vertices into the same 32-bit words
    // meanwhile, so both do it by atomics.
    const bool atomic = a.rp_in != a.rp;
    const gptr<const uint4> qc = a.queue[level % 3];
    const gptr<const uint4> qp = a.queue[(level + 2) % 3];
    gptr<M> vis = (gptr<M>)a.vis;
    const gptr<const M> fc = (gptr<const M>)eager_front(a, level % 3);
    gptr<M> fp = (gptr<M>)eager_front(a, (level + 2) % 3);
    for (long long i = gtid; i < v.queue; i += nthreads) {
      const uint32_t s = qc[i].w;
      const M old = vis[s], bits = fc[s];
      if (!atomic)
        vis[s] = static_cast<M>(old | bits);
      else if (bits & ~old)
        atomic_or_word<SIGMA>(vis + s, bits);
    }
    for (long long i = gtid; i < prev_queue; i += nthreads) fp[qp[i].w] = 0;
  }
  if (engine == BLEST_ENGINE_BOTTOM_UP)
    eager_bu<SIGMA, BLOCK>(a, level, gwave, nwaves, L);
  else
    eager_td<SIGMA, SliceT, BLOCK>(a, level, v.queue, gwave, nwaves, L);
}

template <int SIGMA, class SliceT, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_bfs_eager(BfsArgs args) {
  args_ref<BfsArgs> a = kernel_args(args);
  extern __shared__ float s_mlp[];
  __shared__ int s_level;
  __shared__ EpisodeLds s_ep;
  using M = typename MaskOf<SIGMA>::T;
  const unsigned nblocks = gridDim.x;
  const long long nthreads = static_cast<long long>(nblocks) * BLOCK;
  const long long gtid = static_cast<long long>(blockIdx.x) * BLOCK + threadIdx.x;
  const long long gwave = static_cast<long long>(blockIdx.x) * (BLOCK / 64) + wave_in_block();
  const long long nwaves = static_cast<long long>(nblocks) * (BLOCK / 64);
  const bool learned = a.policy == BLEST_POLICY_LEARNED && a.mlp != nullptr && a.mlp->valid;
  const lptr<const float> mlp = to_lds((const float*)s_mlp);
  if (threadIdx.x == 0) s_ep.found = 0;
  if (threadIdx.x < 12) s_ep.sum[0][threadIdx.x] = 0u;
  if (learned) mlp_to_lds((const MlpDev*)a.mlp, s_mlp);
  // levels, visited words and F_0, F_1 as in the lazy scheme, plus F_2; the
  // registration barrier publishes them with the level-0 counters and queue
  clear_state<SIGMA>(a, gtid, nthreads, true);
  {
    const gptr<M> f2 = (gptr<M>)eager_front(a, 2);
    for (long long s = gtid; s < a.nsets; s += nthreads) f2[s] = 0;
  }
  if (blockIdx.x == 0) {
    __syncthreads();  // block 0's counter clear before its seed counters
    seed_source<SIGMA>(a, true);
    if (threadIdx.x == 0) {
      a.ctl->single_gen[0] = 0u;
      host_status_begin(a.hstat);
    }
  }
  BarrierCtx bc;
  if (!barrier_register((Ctl*)a.ctl, &bc, a.timeout_ticks)) return;
  int level = 0;
  unsigned episodes = 0;
  LevelView v = read_level(a.ctl, 0);
  uint32_t prev_queue = 0;
  while (v.frontier != 0) {
    const int engine = decide_level<true>(a, v, level, mlp, learned);
    if (episode_eligible(a, v, engine)) {
      // workgroup 0 runs levels alone; the others wait for the level it stops
      // at. It leaves no word of the level before behind, so prev_queue is 0.
      ++episodes;
      if (blockIdx.x == 0) {
        const int next = uniform(eager_episode<SIGMA, BLOCK>(a, level, v, prev_queue, mlp, learned, to_lds(&s_ep)));
        block_sync_mem();
        if (threadIdx.x == 0) {
          __hip_atomic_store(&a.ctl->single_level[0], next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&a.ctl->single_gen[0], episodes, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
          // counters were updated by device atomics during the episode; drop
          // any cached copies before the plain loads of grid mode
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          s_level = next;
        }
      } else if (threadIdx.x == 0) {
        s_level = wait_episode(a, episodes);
      }
      __syncthreads();
      if (s_level < 0 || __hip_atomic_load(&a.ctl->error[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
        return;
      level = uniform(s_level);
      if (threadIdx.x == 0) s_ep.found = 0;
      if (threadIdx.x < 12) s_ep.sum[0][threadIdx.x] = 0u;
      __syncthreads();  // s_level is read before the next episode writes it
      v = read_level(a.ctl, level % kStatSlots);
      v.light = v.heavy = 0;
      prev_queue = 0;
      continue;
    }
    eager_level<SIGMA, SliceT, BLOCK>(a, level, v, prev_queue, engine, gtid, nthreads, gwave, nwaves, to_lds(&s_ep));
    if (!grid_barrier((Ctl*)a.ctl, bc)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0 && level < a.log_cap) {
      const unsigned long long t = dev_ticks();
      a.log[level].t_mid = t;
      a.log[level].t_end = t;
      a.log[level].work = static_cast<long long>(a.ctl->acc[level % kStatSlots][F_WORK][0]);
    }
    LevelView nv = read_level(a.ctl, (level + 1) % kStatSlots);
    nv.light = 0;
    nv.heavy = 0;
    nv.cumv = v.cumv + nv.frontier;
    nv.cume = v.cume + nv.fedges;
    prev_queue = v.queue;
    v = nv;
    ++level;
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x < 8) a.ctl->xcd_blocks[threadIdx.x][0] = 0u;
    if (threadIdx.x == 8) a.ctl->xcd_active[0] = 0u;
    if (threadIdx.x == 0) {
      a.ctl->nlevels[0] = level;
      host_status_end(a.hstat, a.ctl, level);
    }
  }
}

// ------------------------------------------------------ per-stage kernels

template <int SIGMA, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_bfs_clear(BfsArgs args) {
  args_ref<BfsArgs> a = kernel_args(args);
  const long long nthreads = static_cast<long long>(gridDim.x) * BLOCK;
  clear_state<SIGMA>(a, static_cast<long long>(blockIdx.x) * BLOCK + threadIdx.x, nthreads);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.ctl->done[0] = 0;
    host_status_begin(a.hstat);  // (stays 0: the host reads the control block after per-stage launches)
  }
}

template <int SIGMA, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_bfs_seed(BfsArgs args) {
  args_ref<BfsArgs> a = kernel_args(args);
  seed_source<SIGMA>(a);
}

template <int SIGMA, class SliceT, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_bfs_stage1(BfsArgs args, int level, long long prev_slot_frontier_unused) {
  args_ref<BfsArgs> a = kernel_args(args);
  extern __shared__ float s_mlp[];
  if (a.ctl->done[0]) return;
  const long long gwave = static_cast<long long>(blockIdx.x) * (BLOCK / 64) + wave_in_block();
  const long long nwaves = static_cast<long long>(gridDim.x) * (BLOCK / 64);
  const LevelView v = read_level(a.ctl, level % kStatSlots);
  if (v.frontier == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.ctl->done[0] = 1;
      a.ctl->nlevels[0] = level;
    }
    return;
  }
  const bool learned = a.policy == BLEST_POLICY_LEARNED && a.mlp != nullptr && a.mlp->valid;
  if (learned) {
    mlp_to_lds((const MlpDev*)a.mlp, s_mlp);
    __syncthreads();
  }
  const int engine = decide_level<false>(a, v, level, to_lds((const float*)s_mlp), learned);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) log_begin(a, level);
    const int nslot = (level + 1) % kStatSlots;
    for (int t = threadIdx.x; t < kStatFields; t += BLOCK) a.ctl->acc[nslot][t][0] = 0ULL;
  }
  __shared__ __attribute__((aligned(16))) uint32_t pm[kPanelMaxBytes / 4];
  run_engine<SIGMA, SliceT, BLOCK, false>(a, engine, level & 1, level % kStatSlots, v, gwave, nwaves, (lptr<int>)to_lds(pm),
                                   to_lds(pm));
}

template <int SIGMA, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_bfs_stage2(BfsArgs args, int level) {
  args_ref<BfsArgs> a = kernel_args(args);
  if (a.ctl->done[0]) return;
  const LevelView v = read_level(a.ctl, level % kStatSlots);
  if (v.frontier == 0) return;
  if (blockIdx.x == 0 && threadIdx.x == 0 && level < a.log_cap) a.log[level].t_mid = dev_ticks();
  finalize<SIGMA, BLOCK>(a, level + 1, (level + 1) % kStatSlots, (level & 1) ^ 1, v.cumv, v.cume);
  if (blockIdx.x == 0 && threadIdx.x == 0 && level < a.log_cap) {
    a.log[level].t_end = dev_ticks();
    a.log[level].work = static_cast<long long>(a.ctl->acc[level % kStatSlots][F_WORK][0]);
  }
}

// ------------------------------------------------------------ host side

namespace {

template <int SIGMA, class SliceT, int BLOCK>
const void* persistent_fn() {
  return reinterpret_cast<const void*>(&k_bfs_persistent<SIGMA, SliceT, BLOCK>);
}

template <int SIGMA, class SliceT, int BLOCK>
const void* eager_fn() {
  return reinterpret_cast<const void*>(&k_bfs_eager<SIGMA, SliceT, BLOCK>);
}

template <int SIGMA, class SliceT, int BLOCK>
hipError_t run_t(const DevGraph& g, BfsArgs& a, hipStream_t st) {
  const size_t shmem = (a.policy == BLEST_POLICY_LEARNED) ? kLdsMlpFloats * sizeof(float) : 0;
  if (g.eager && !a.probe) {
    void* args[] = {static_cast<void*>(&a)};
    return hipLaunchCooperativeKernel(eager_fn<SIGMA, SliceT, BLOCK>(), dim3(g.grid_eager), dim3(BLOCK), args,
                                      static_cast<unsigned>(shmem), st);
  }
  if (g.persistent || a.probe) {
    void* args[] = {static_cast<void*>(&a)};
    return hipLaunchCooperativeKernel(persistent_fn<SIGMA, SliceT, BLOCK>(), dim3(g.grid), dim3(BLOCK), args,
                                      static_cast<unsigned>(shmem), st);
  }
  hipLaunchKernelGGL((k_bfs_clear<SIGMA, BLOCK>), dim3(g.grid), dim3(BLOCK), 0, st, a);
  hipLaunchKernelGGL((k_bfs_seed<SIGMA, BLOCK>), dim3(1), dim3(BLOCK), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int level = 0;
  int batch = 4;
  for (;;) {
    for (int i = 0; i < batch; ++i, ++level) {
      hipLaunchKernelGGL((k_bfs_stage1<SIGMA, SliceT, BLOCK>), dim3(g.grid), dim3(BLOCK), shmem, st, a, level, 0LL);
      hipLaunchKernelGGL((k_bfs_stage2<SIGMA, BLOCK>), dim3(g.grid), dim3(BLOCK), 0, st, a, level);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(g.host_flags, &g.ctl->done[0], sizeof(int), hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    if (g.host_flags[0]) break;
    if (level > g.n + 2) return hipErrorUnknown;
    batch = batch < 64 ? batch * 2 : 64;
  }
  return hipSuccess;
}

template <int SIGMA, class SliceT>
hipError_t run_block(const DevGraph& g, BfsArgs& a, hipStream_t st) {
  switch (g.block) {
    case 256:
      return run_t<SIGMA, SliceT, 256>(g, a, st);
    case 1024:
      return run_t<SIGMA, SliceT, 1024>(g, a, st);
    default:
      return run_t<SIGMA, SliceT, 512>(g, a, st);
  }
}

template <int SIGMA, class SliceT>
hipError_t occupancy_block(const DevGraph& g, size_t shmem, int* nb) {
  switch (g.block) {
    case 256:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, persistent_fn<SIGMA, SliceT, 256>(), 256, shmem);
    case 1024:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, persistent_fn<SIGMA, SliceT, 1024>(), 1024, shmem);
    default:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, persistent_fn<SIGMA, SliceT, 512>(), 512, shmem);
  }
}

template <int SIGMA, class SliceT>
hipError_t occupancy_eager(const DevGraph& g, size_t shmem, int* nb) {
  switch (g.block) {
    case 256:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, eager_fn<SIGMA, SliceT, 256>(), 256, shmem);
    case 1024:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, eager_fn<SIGMA, SliceT, 1024>(), 1024, shmem);
    default:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, eager_fn<SIGMA, SliceT, 512>(), 512, shmem);
  }
}

}  // namespace

hipError_t bfs_grid_size_eager(const DevGraph& g, int blocks_per_cu, int* grid) {
  // sized with the switch network's LDS, which the learned policy adds
  const size_t shmem = kLdsMlpFloats * sizeof(float);
  int nb = 0;
  hipError_t e;
  if (g.sigma == 8 && !g.wide)
    e = occupancy_eager<8, uint32_t>(g, shmem, &nb);
  else if (g.sigma == 8)
    e = occupancy_eager<8, uint64_t>(g, shmem, &nb);
  else if (g.sigma == 16)
    e = occupancy_eager<16, uint64_t>(g, shmem, &nb);
  else
    e = occupancy_eager<32, uint64_t>(g, shmem, &nb);
  if (e != hipSuccess) return e;
  if (nb < 1) return hipErrorInvalidConfiguration;
  // its levels are small and latency-bound: one workgroup per compute unit
  // (fewer arrivals per device-wide barrier) unless asked otherwise
  nb = blocks_per_cu > 0 ? std::min(nb, blocks_per_cu) : 1;
  *grid = nb * g.num_cu;
  // A graph that few workgroups sweep gets few, for the same reason: a 4096-vertex
  // R-MAT (56,314 slices) takes 149 us a call on 256 workgroups, 141 on 64, 139 on
  // 32 and on 16; 65,536 vertices with 1.38 M slices take 190, 221 and 281 on 256,
  // 64 and 32. 2048 slices a workgroup is one pass of its waves over the queue.
  if (blocks_per_cu <= 0)
    *grid = static_cast<int>(std::min<int64_t>(*grid, std::max<int64_t>(32, (g.nslices + 2047) / 2048)));
  return hipSuccess;
}

BfsArgs bfs_args(const DevGraph& g) {
  BfsArgs a{};
  a.rp = to_global(g.rp);
  a.col = to_global(g.col);
  a.slice_ptr = to_global(g.slice_ptr);
  a.slices = to_global(g.slices);
  a.degmask = to_global(g.degmask);
  a.rp_in = to_global(g.rp_in);
  a.col_in = to_global(g.col_in);
  a.degmask_in = to_global(g.degmask_in);
  a.orig_id = to_global(g.orig_id);
  a.n = g.n;
  a.m = g.m;
  a.nsets = g.nsets;
  a.tau = g.tau;
  a.sigma = g.sigma;
  a.vis = to_global(g.vis);
  a.front = to_global(g.front);
  a.fstride = static_cast<long long>(g.fstride);
  a.mark = to_global(g.mark);
  a.queue[2] = to_global(g.queue[2]);
  for (int i = 0; i < 2; ++i) {
    a.queue[i] = to_global(g.queue[i]);
    a.flight[i] = to_global(g.flight[i]);
    a.fheavy[i] = to_global(g.fheavy[i]);
  }
  a.ctl = to_global(g.ctl);
  a.part = to_global(g.part);
  a.hstat = to_global(g.hstat);
  a.log = to_global(g.log);
  a.log_cap = g.log_cap;
  a.mlp = to_global(g.mlp);
  a.prefilter = g.prefilter;
  a.count_work = g.count_work;
  a.single_block = g.single_block;
  a.pwords = to_global(g.pwords);
  a.pbase = to_global(g.pbase);
  a.pptr = to_global(g.pptr);
  a.npanels = static_cast<int32_t>(g.npanels);
  a.panel_rb = g.panel_rb;
  a.panel_mode = g.panel_mode;
  a.panel_slots = g.nchunks * kPanelChunk;
  a.nvss = g.nvss;
  a.nslices = g.nslices;
  a.count_first = g.count_first;
  a.timeout_ticks = 1000000000ULL;  // 10 s at the 100 MHz device clock
  return a;
}

hipError_t bfs_run(const DevGraph& g, BfsArgs a, hipStream_t st) {
  if (g.sigma == 8 && !g.wide) return run_block<8, uint32_t>(g, a, st);
  if (g.sigma == 8) return run_block<8, uint64_t>(g, a, st);
  if (g.sigma == 16) return run_block<16, uint64_t>(g, a, st);
  return run_block<32, uint64_t>(g, a, st);
}

hipError_t bfs_grid_size(const DevGraph& g, int policy_learned, int blocks_per_cu, int* grid) {
  const size_t shmem = policy_learned ? kLdsMlpFloats * sizeof(float) : 0;
  int nb = 0;
  hipError_t e;
  if (g.sigma == 8 && !g.wide)
    e = occupancy_block<8, uint32_t>(g, shmem, &nb);
  else if (g.sigma == 8)
    e = occupancy_block<8, uint64_t>(g, shmem, &nb);
  else if (g.sigma == 16)
    e = occupancy_block<16, uint64_t>(g, shmem, &nb);
  else
    e = occupancy_block<32, uint64_t>(g, shmem, &nb);
  if (e != hipSuccess) return e;
  if (nb < 1) return hipErrorInvalidConfiguration;
  if (blocks_per_cu > 0 && blocks_per_cu < nb) nb = blocks_per_cu;
  *grid = nb * g.num_cu;
  return hipSuccess;
}

}  // namespace blest
