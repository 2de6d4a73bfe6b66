// Operator-sequence matcher on the GPU.
//
// (i) Similarity of two integer operator sequences and the stage machine of Algo. 1
//     (Sec. 3 of the SmartSwap paper): length within 5 %, cosine above 95 %.  The three
//     integer sums of the cosine are reduced on the GPU; the threshold is decided exactly
//     on the host in 128-bit integer arithmetic.
// (ii) Re-anchoring of policy items in the current sequence (Sec. 5.1: multi-feature
//     matching on operator name, call stack and data type with integer comparisons
//     only): an anchor's ordinal among the reference's operators with its key, at each of three
//     relaxation levels, and the operator of that ordinal in the current sequence.  Short sequences of few keys: one workgroup does
//     it all.  Few anchors or short sequences: one workgroup or wavefront per anchor counts and searches.  Many: the layers of a model
//     share their keys, so the anchors' distinct keys are collected first, both sequences are gone through once, chunk by
//     chunk, to number the occurrences of each key, and an anchor looks its ordinal up.
#include <algorithm>
#include <cstring>

#include "ss_internal.h"

namespace {

constexpr uint32_t kTokenLimit = SS_TOKEN_LIMIT;
constexpr uint32_t kLenLimit = 1u << 23;

constexpr uint32_t kMaxParts = 1024;
// Calls until short sequences are given to one workgroup again after one with too many keys.  A try for nothing costs 9 us, a context's
// first 14; so where none has been worth it yet, the last one wasn't or was of sequences half as long, some operators are looked at
// first (more_keys, 1 us).
constexpr uint32_t kTryAgain = 64;

// Everything that has to be done before anchors can be looked for, in one pass: the sequences (and anchors) are copied
// from pinned host memory to device memory if dref / dcur / danc are given, the sums of the cosine taken on the way
// (unless counted: histograms), and the words of `clear` set (tables of the kernels that follow).
struct PrepArgs {
  const ss_op_t *ref, *cur;  const ss_anchor_t *anchors;
  ss_op_t *dref, *dcur;      ss_anchor_t *danc;
  uint32_t n, m, k, cosine;
  uint4 *ones, *zeros;       uint32_t n_ones, n_zeros;       // in 16-byte words
  ss_cosine_part *part;          // one per workgroup
  ss_done done;              // if this is the call's last kernel
};

// kTogether: a thread reads four operators of each sequence together.  From device memory (500,000 of each one by one take
// 25 us, together 6) and for short sequences from pinned memory, where the link's latency is what it takes (1,154 of each
// 22.4 us a call, together 20.1; 8,000 27 to 29 and 25.5).  Long ones come over the link faster one by one (18,464 38.5 and
// 38.0, 30,000 52.0 and 52.6, 65,536 96 and 105).
constexpr uint32_t kTogetherMapped = 16384;

// Sequences of this many bytes each take two such passes: the reference comes over the link while the host copies the other
// one to pinned memory (about 30 GB/s, half the link's rate).  The cosine of 65,536 operators 105 us a call in one pass and
// 90 in two, of 50,000 68.1 and 66.6, of 24,000 39.4 and 38.9, of 9,000 20.2 and 21.8.
constexpr size_t kSplitBytes = 768 * 1024;

template <bool kTogether>
__global__ __launch_bounds__(256) void ss_prep_kernel(PrepArgs a) {
  const uint32_t stride = gridDim.x * 256, first = blockIdx.x * 256 + threadIdx.x, len = a.n > a.m ? a.n : a.m;
  uint64_t dot = 0, na = 0, nb = 0;
  uint32_t bad = 0;
  auto take = [&](uint32_t i, const ss_op_t &c, const ss_op_t &r) {
    if (a.dcur && i < a.m) a.dcur[i] = c;
    if (a.dref && i < a.n) a.dref[i] = r;
    const uint64_t x = c.op_token, y = r.op_token;
    if (x >= kTokenLimit || y >= kTokenLimit) bad = 1;
    dot += x * y;
    na += x * x;
    nb += y * y;
  };
  if constexpr (kTogether) {
    constexpr uint32_t kAhead = 4;
    for (uint32_t i0 = first; i0 < len; i0 += kAhead * stride) {
      ss_op_t c[kAhead], r[kAhead];                      // the shorter sequence is padded with token 0
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) {
        const uint32_t i = i0 + u * stride;
        c[u] = r[u] = ss_op_t{0, 0, 0, 0};
        if (i < a.m) c[u] = a.cur[i];
        if (i < a.n) r[u] = a.ref[i];
      }
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) take(i0 + u * stride, c[u], r[u]);
    }
  } else {
    for (uint32_t i = first; i < len; i += stride) {
      ss_op_t c = {0, 0, 0, 0}, r = {0, 0, 0, 0};
      if (i < a.m) c = a.cur[i];
      if (i < a.n) r = a.ref[i];
      take(i, c, r);
    }
  }
  if (a.danc)
    for (uint32_t i = first; i < a.k; i += stride) a.danc[i] = a.anchors[i];
  for (uint32_t i = first; i < a.n_ones; i += stride) a.ones[i] = uint4{~0u, ~0u, ~0u, ~0u};
  for (uint32_t i = first; i < a.n_zeros; i += stride) a.zeros[i] = uint4{0, 0, 0, 0};
  if (a.cosine) ss_put_part<256>(a.part, dot, na, nb, bad);
  ss_tell_host(a.done);
}

// occurrence counts per token of both sequences (token 0 never counts).  A model has few operator names, so most
// additions would meet at a few addresses: each workgroup counts the low tokens in LDS first.
constexpr uint32_t kLdsTokens = 1024;

__global__ __launch_bounds__(256) void ss_histogram_kernel(const ss_op_t *__restrict__ ref, uint32_t n,
                                                           const ss_op_t *__restrict__ cur, uint32_t m,
                                                           uint32_t *h_ref, uint32_t *h_cur, uint32_t *flags) {
  __shared__ uint32_t low[2][kLdsTokens];
  for (uint32_t t = threadIdx.x; t < 2 * kLdsTokens; t += 256) low[0][t] = 0;
  __syncthreads();
  const uint32_t len = n > m ? n : m;
  auto add = [&](uint32_t t, uint32_t *mine, uint32_t *all) {
    if (t >= kTokenLimit) atomicOr(flags, 1u);
    else if (t >= kLdsTokens) atomicAdd(all + t, 1u);
    else if (t) atomicAdd(mine + t, 1u);
  };
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < len; i += gridDim.x * blockDim.x) {
    if (i < m) add(cur[i].op_token, low[0], h_cur);
    if (i < n) add(ref[i].op_token, low[1], h_ref);
  }
  __syncthreads();
  for (uint32_t t = threadIdx.x; t < kLdsTokens; t += 256) {
    if (low[0][t]) atomicAdd(h_cur + t, low[0][t]);
    if (low[1][t]) atomicAdd(h_ref + t, low[1][t]);
  }
}

__global__ __launch_bounds__(256) void ss_histdot_kernel(const uint32_t *__restrict__ h_ref,
                                                         const uint32_t *__restrict__ h_cur, uint32_t vocab,
                                                         const uint32_t *__restrict__ flags, ss_cosine_part *part, ss_done done) {
  uint64_t dot = 0, na = 0, nb = 0;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < vocab; i += gridDim.x * blockDim.x) {
    const uint64_t a = h_cur[i], b = h_ref[i];
    dot += a * b; na += a * a; nb += b * b;
  }
  ss_put_part<256>(part, dot, na, nb, *flags);
  ss_tell_host(done);
}

// By shuffles: with ss_wave_sum's moves 8,001 searches for distinct keys, whose registers it takes, go from 259 to 284 us.
__device__ inline uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += (uint32_t)__shfl_xor((int)v, d, 64);
  return v;
}

// Lane index of the bit of `mask` that has exactly `need` set bits below it.
__device__ inline int nth_set_bit(uint64_t mask, uint32_t need, int lane) {
  const uint64_t below = lane ? (mask & (~0ull >> (64 - lane))) : 0ull;
  const bool mine = ((mask >> lane) & 1ull) && (uint32_t)__popcll(below) == need;
  const uint64_t sel = __ballot(mine);
  return __ffsll((long long)sel) - 1;
}

// Equality of two operators at each relaxation level: (token, stack, sig), (token, sig), (token).  Without short cuts (&&):
// behind one the compiler reads the stack only once the token is known to be equal, a second dependent load in every turn
// of a search (8,001 anchors over 18,464 operators, each searched for by a wavefront, 448 us a call against 296; 20,000 over
// 65,536 3,060 against 1,515).
__device__ __forceinline__ void same_key(const ss_op_t &x, const ss_op_t &y, bool &e0, bool &e1, bool &e2) {
  e2 = x.op_token == y.op_token;
  e1 = e2 & (x.sig == y.sig);
  e0 = e1 & (x.stack_hash == y.stack_hash);
}

// The first level whose landing place has the slot and the data type; f[L] < 0: none at level L.
__device__ __forceinline__ int32_t choose_landing(const ss_op_t *cur, const ss_op_t &R, uint32_t slot, const int32_t f[3],
                                                  uint8_t &level) {
#pragma unroll
  for (int L = 0; L < 3; ++L) {
    if (f[L] < 0) continue;
    const ss_op_t o = cur[f[L]];
    if (slot < o.n_out && (o.sig & 0xFFu) == (R.sig & 0xFFu)) { level = (uint8_t)L; return f[L]; }
  }
  level = 255;
  return -1;
}

// Among anchors landing on the same (operator, slot) only the lowest anchor index keeps it.
// Two passes over an open-addressing table of at least 2k slots keyed by (operator, slot): every
// landed anchor finds or claims its key's slot (compare-and-swap, linear probing) and lowers the
// slot's owner to its own index (integer minimum: any order, same result); then an anchor keeps its
// landing exactly if it owns its slot.  Linear in k (20,000 anchors: all earlier anchors compared one
// by one took 2 ms).
constexpr unsigned long long kEmptyKey = ~0ull;

struct ClaimTable {
  unsigned long long *keys;    // all kEmptyKey before the first claim
  uint32_t *owner;             // all ones
  uint32_t mask, shift;
};

__device__ __forceinline__ uint32_t claim(const ClaimTable &t, int32_t j, uint32_t slot, uint32_t a) {
  const unsigned long long key = ((unsigned long long)(uint32_t)j << 32) | slot;     // j < 2^31: never kEmptyKey
  uint32_t h = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> t.shift);
  // at most k distinct keys in more than 2k slots: a free or matching slot is met within mask + 1 probes
  for (uint32_t probe = 0; probe <= t.mask; ++probe) {
    const unsigned long long seen = atomicCAS(t.keys + h, kEmptyKey, key);
    if (seen == kEmptyKey || seen == key) {
      atomicMin(t.owner + h, a);
      return h;
    }
    h = (h + 1) & t.mask;
  }
  return 0;
}

struct AnchorArgs {
  const ss_op_t *ref, *cur;
  const ss_anchor_t *anchors;
  uint32_t n, m, k;
  int32_t *land;               // operator index in cur, or -1
  uint8_t *lvl;                // its level, or 255
  uint32_t *slot_of;           // its slot of the claim table
  ClaimTable table;
};

struct AnchorShared {
  uint32_t in_ref[4][3], in_cur[4][3];
  int32_t found[3];
  uint32_t lands[3];           // ss_anchor_kernel in registers: the found operator has the slot and the data type
};

// The landing of anchor a, found by the whole workgroup.  Each wavefront counts, over its quarter of the reference up to
// the anchor and its quarter of the current sequence, the operators with the anchor's key at each level; the ordinal's
// quarter is then known and its wavefront walks it 64 operators at a time (ballots and population counts find the
// operator).
__device__ __forceinline__ void search_anchor(const AnchorArgs &g, uint32_t a, AnchorShared &sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t i = g.anchors[a].ref_op, slot = g.anchors[a].out_slot;
  if (i >= g.n || g.ref[i].op_token == 0) {              // uniform
    if (threadIdx.x == 0) { g.land[a] = -1; g.lvl[a] = 255; }
    return;
  }
  const ss_op_t R = g.ref[i];
  const uint32_t rq = (i + 255) / 256 * 64, cq = (g.m + 255) / 256 * 64;       // quarters, whole strips of 64
  const uint32_t r_lo = w * rq, r_hi = min(i, r_lo + rq), c_lo = w * cq, c_hi = min(g.m, c_lo + cq);
  uint32_t r[3] = {0, 0, 0}, c[3] = {0, 0, 0};
  auto count = [&](const ss_op_t *seq, uint32_t lo, uint32_t hi, uint32_t *out) {
    constexpr uint32_t kAhead = 4;
    for (uint32_t j0 = lo + lane; j0 < hi; j0 += 64 * kAhead) {
      ss_op_t o[kAhead];
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) {
        o[u].op_token = 0;                               // padding: never the anchor's token
        if (j0 + 64 * u < hi) o[u] = seq[j0 + 64 * u];
      }
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) {
        bool e0, e1, e2;
        same_key(o[u], R, e0, e1, e2);
        out[0] += e0; out[1] += e1; out[2] += e2;
      }
    }
#pragma unroll
    for (int L = 0; L < 3; ++L) out[L] = wave_sum_u32(out[L]);
  };
  count(g.ref, r_lo, r_hi, r);
  count(g.cur, c_lo, c_hi, c);
  if (lane < 3) {
    sh.in_ref[w][lane] = lane == 0 ? r[0] : lane == 1 ? r[1] : r[2];
    sh.in_cur[w][lane] = lane == 0 ? c[0] : lane == 1 ? c[1] : c[2];
  }
  if (threadIdx.x < 3) sh.found[threadIdx.x] = -1;
  __syncthreads();
  // this wavefront's levels: the ordinal lies in its quarter
  uint32_t need[3];
  bool open[3];
#pragma unroll
  for (int L = 0; L < 3; ++L) {
    uint32_t ord = sh.in_ref[0][L] + sh.in_ref[1][L] + sh.in_ref[2][L] + sh.in_ref[3][L], before = 0;
    for (int v = 0; v < w; ++v) before += sh.in_cur[v][L];
    open[L] = ord >= before && ord < before + sh.in_cur[w][L];
    need[L] = ord - before;
  }
  for (uint32_t base = c_lo; (open[0] || open[1] || open[2]) && base < c_hi; base += 64) {
    const uint32_t j = base + lane;
    bool e[3] = {false, false, false};
    if (j < c_hi) same_key(g.cur[j], R, e[0], e[1], e[2]);
#pragma unroll
    for (int L = 0; L < 3; ++L) {
      const uint64_t b = __ballot(e[L]);
      if (!open[L]) continue;
      const uint32_t pc = __popcll(b);
      if (need[L] < pc) {
        const int at = nth_set_bit(b, need[L], lane);
        if (lane == 0) sh.found[L] = (int32_t)base + at;
        open[L] = false;
      } else {
        need[L] -= pc;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int32_t f[3] = {sh.found[0], sh.found[1], sh.found[2]};
    uint8_t level;
    const int32_t j = choose_landing(g.cur, R, slot, f, level);
    g.land[a] = j;
    g.lvl[a] = level;
    if (j >= 0) g.slot_of[a] = claim(g.table, j, slot, a);
  }
}

// The same for sequences of up to kRegOps operators, which the workgroup holds in registers: they are loaded while the anchor
// and its operator are, counted, walked and landed on without another load.
constexpr uint32_t kPerLane = 8, kRegOps = 256 * kPerLane;

__device__ __forceinline__ void search_in_registers(const AnchorArgs &g, uint32_t a, AnchorShared &sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t rq = (g.n + 255) / 256 * 64, cq = (g.m + 255) / 256 * 64;     // quarters, whole strips of 64
  const uint32_t r_lo = w * rq, c_lo = w * cq;
  ss_op_t r[kPerLane], c[kPerLane];
#pragma unroll
  for (uint32_t u = 0; u < kPerLane; ++u) {
    r[u] = c[u] = ss_op_t{0, 0, 0, 0};                   // padding: never the anchor's token
    const uint32_t i = r_lo + 64 * u + lane, j = c_lo + 64 * u + lane;
    if (64 * u < rq && i < g.n) r[u] = g.ref[i];
    if (64 * u < cq && j < g.m) c[u] = g.cur[j];
  }
  const uint32_t i = g.anchors[a].ref_op, slot = g.anchors[a].out_slot;
  ss_op_t R = {0, 0, 0, 0};
  if (i < g.n) R = g.ref[i];
  if (R.op_token == 0) {                                 // uniform
    if (threadIdx.x == 0) { g.land[a] = -1; g.lvl[a] = 255; }
    return;
  }
  uint32_t rn[3] = {0, 0, 0}, cn[3] = {0, 0, 0};
#pragma unroll
  for (uint32_t u = 0; u < kPerLane; ++u) {
    bool e[3], f[3];
    same_key(r[u], R, e[0], e[1], e[2]);
    same_key(c[u], R, f[0], f[1], f[2]);
    const bool before = r_lo + 64 * u + lane < i;
#pragma unroll
    for (int L = 0; L < 3; ++L) {
      rn[L] += __popcll(__ballot(e[L] & before));
      cn[L] += __popcll(__ballot(f[L]));
    }
  }
  if (lane < 3) {
    sh.in_ref[w][lane] = lane == 0 ? rn[0] : lane == 1 ? rn[1] : rn[2];
    sh.in_cur[w][lane] = lane == 0 ? cn[0] : lane == 1 ? cn[1] : cn[2];
  }
  if (threadIdx.x < 3) { sh.found[threadIdx.x] = -1; sh.lands[threadIdx.x] = 0; }
  __syncthreads();
#pragma unroll
  for (int L = 0; L < 3; ++L) {
    uint32_t ord = sh.in_ref[0][L] + sh.in_ref[1][L] + sh.in_ref[2][L] + sh.in_ref[3][L], before = 0;
    for (int v = 0; v < w; ++v) before += sh.in_cur[v][L];
    if (ord < before || ord >= before + cn[L]) continue; // uniform: another wavefront's, or nowhere
    uint32_t need = ord - before;
#pragma unroll
    for (uint32_t u = 0; u < kPerLane; ++u) {
      bool f[3];
      same_key(c[u], R, f[0], f[1], f[2]);
      const uint64_t b = __ballot(f[L]);
      const uint32_t pc = __popcll(b);
      if (need < pc) {
        if (lane == nth_set_bit(b, need, lane)) {
          sh.found[L] = (int32_t)(c_lo + 64 * u + lane);
          sh.lands[L] = slot < c[u].n_out && (c[u].sig & 0xFFu) == (R.sig & 0xFFu);
        }
        break;
      }
      need -= pc;
    }
  }
  __syncthreads();
  if (threadIdx.x) return;
  int32_t j = -1;
  uint8_t level = 255;
#pragma unroll
  for (int L = 2; L >= 0; --L)
    if (sh.lands[L]) { j = sh.found[L]; level = (uint8_t)L; }
  g.land[a] = j;
  g.lvl[a] = level;
  if (j >= 0) g.slot_of[a] = claim(g.table, j, slot, a);
}

// One workgroup per anchor.  Bound by the latency of the loads and walks: 480 anchors of 1,154 operators 6.1 us in registers,
// claims included, 8.3 reading them as they are counted and walked; a wavefront per anchor, all of both sequences in one walk,
// took 13.0 us and the claims 3.1 us in a launch of their own.
__global__ __launch_bounds__(256) void ss_anchor_kernel(AnchorArgs g) {
  __shared__ AnchorShared sh;
  if (g.n <= kRegOps && g.m <= kRegOps) search_in_registers(g, blockIdx.x, sh);
  else search_anchor(g, blockIdx.x, sh);
}

// The landing of anchor a, found by one wavefront: all of both sequences in one walk.
__device__ __forceinline__ int32_t search_alone(const AnchorArgs &g, const ss_op_t &R, uint32_t i, uint32_t slot, uint8_t &level) {
  const int lane = threadIdx.x & 63;
  int32_t f[3] = {-1, -1, -1};
  uint32_t r[3] = {0, 0, 0};
  for (uint32_t j = lane; j < i; j += 64) {
    bool e0, e1, e2;
    same_key(g.ref[j], R, e0, e1, e2);
    r[0] += e0; r[1] += e1; r[2] += e2;
  }
#pragma unroll
  for (int L = 0; L < 3; ++L) r[L] = wave_sum_u32(r[L]);
  for (uint32_t base = 0; base < g.m; base += 64) {
    const uint32_t j = base + lane;
    bool e[3] = {false, false, false};
    if (j < g.m) same_key(g.cur[j], R, e[0], e[1], e[2]);
#pragma unroll
    for (int L = 0; L < 3; ++L) {
      const uint64_t b = __ballot(e[L]);
      if (f[L] >= 0) continue;
      const uint32_t pc = __popcll(b);
      if (r[L] < pc) f[L] = (int32_t)base + nth_set_bit(b, r[L], lane);
      else r[L] -= pc;
    }
    if (f[0] >= 0 && f[1] >= 0 && f[2] >= 0) break;
  }
  return choose_landing(g.cur, R, slot, f, level);
}

// One wavefront per anchor, for kAloneAnchors and more that are at least twice the operators: then a workgroup's barriers
// and launch cost more than its four wavefronts gain.  20,000 anchors over 60 + 60 operators 56 us a call against 85, 2,000
// over 500 + 500 43.2 against 43.9, 8,000 over 1,000 + 1,000 62 against 72, but 2,000 over these 45.1 against 42.9.  The
// rule also keeps the other kernel's launch within 2^32 work-items (2^24 anchors may come with one operator).
constexpr uint32_t kAloneAnchors = 2048;

__global__ __launch_bounds__(256) void ss_anchor_short_kernel(AnchorArgs g) {
  const uint32_t a = (blockIdx.x * 256 + threadIdx.x) >> 6;
  if (a >= g.k) return;                                      // uniform per wavefront
  const uint32_t i = g.anchors[a].ref_op, slot = g.anchors[a].out_slot;
  int32_t result = -1;
  uint8_t level = 255;
  if (i < g.n && g.ref[i].op_token != 0) result = search_alone(g, g.ref[i], i, slot, level);
  if ((threadIdx.x & 63) == 0) {
    g.land[a] = result;
    g.lvl[a] = level;
    if (result >= 0) g.slot_of[a] = claim(g.table, result, slot, a);
  }
}

// ---- short sequences with few keys: one workgroup does it all ----------------------------------------------------------
//
// The operators of both sequences get the number of their key through a table in LDS.  Each key has a bit map of its places in
// either sequence for each level: at the second and the third that of the lowest key equal to it there, where those of all of
// them are put together.  With the places before each word counted, an anchor's thread finds its ordinal in one map and its landing by
// search in the other, level after level.  Bound by the latency of the link (7,200 of 27,400 cycles are the wait for the operators),
// of LDS and of the barriers between nine short phases: 480 anchors of 1,154 + 1,156 operators 12.3 us.  A wavefront for each
// anchor that the first level doesn't land, over the maps of its equals, took 33,600 cycles where 37 don't, and without a bound;
// every operator into all three levels' maps at once 30,800 (atomics on shared words take turns).  Fetched, searched for by a
// workgroup each and made injective in three launches they took 15.3 us and two gaps.
struct ShortArgs {
  const ss_op_t *ref, *cur;            // pinned
  const ss_anchor_t *anchors;
  uint32_t n, m, k, most_keys;         // short_keys
  int32_t *new_idx;                    // pinned
  uint8_t *level;
  uint32_t *lost, *too_many;           // pinned: anchors without a place; keys, if there are more than that (nothing else is written)
  ss_cosine_part *part;
  ss_done done;
};

constexpr uint32_t kShortOps = 2048, kShortAnchors = 2048, kShortKeys = 256, kShortThreads = 1024;
constexpr uint32_t kShortPer = 2 * kShortOps / kShortThreads, kShortMine = kShortAnchors / kShortThreads, kNoOp = ~0u;
constexpr uint32_t kShortSlots = 8192, kShortClaims = 2 * kShortAnchors, kShortMap = 2 * kShortSlots + 6 * kShortOps;
struct ShortLds {
  union {
    struct { uint32_t rep[kShortSlots], id[kShortSlots], token[2 * kShortOps], stack[2 * kShortOps], sig[2 * kShortOps]; } table;     // cur first
    uint32_t map[kShortMap];           // by level and key; then, 16 bits each, the places before each word
    struct { unsigned long long key[kShortClaims]; uint32_t owner[kShortClaims]; } claims;
  };
  uint32_t n_out[kShortOps];           // of cur
  uint32_t key_token[kShortKeys], key_sig[kShortKeys];
  unsigned long long dot, na, nb;
  uint32_t n_keys, lost, bad;
  uint16_t ref_key[kShortOps];
  uint8_t cur_type[kShortOps];
  uint8_t lowest[2][kShortKeys];       // key equal at the second level, at the third
};
static_assert(sizeof(ShortLds) <= 150 * 1024, "one workgroup's LDS");

// places before each of the words of a row of sixteen lanes, four a lane
__device__ __forceinline__ uint2 counts_before(uint4 b) {
  const uint32_t x = (uint32_t)__popc(b.x), y = x + (uint32_t)__popc(b.y), z = y + (uint32_t)__popc(b.z), all = z + (uint32_t)__popc(b.w);
  const uint32_t first = row_scan_u32(all) - all;
  return uint2{first | (first + x) << 16, (first + y) | (first + z) << 16};
}

static __host__ __device__ __forceinline__ uint32_t up_to_four(uint32_t x) { return (x + 3) / 4 * 4; }

// Words of a key's maps at a level: an odd number of 16 bytes, so that the maps' starts lie in different banks.
static __host__ __device__ __forceinline__ uint32_t map_stride(uint32_t n, uint32_t m) {
  return (up_to_four((n + 31) / 32) + up_to_four((m + 31) / 32)) | 4;
}

// How many keys one workgroup matches: as many as the maps of three levels, with 16 bits more a word, fit LDS for, and no more than are
// as fast as three launches.  Each key is compared with all and its maps are put together, which few anchors don't make up for
// (three launches | one; 100 anchors of 200 operators, 115 keys 21.0 | 20.9 us, 145 21.4 | 22.4, 200 21.0 | 25.6; 1,000 anchors, 160 keys
// 27.8 | 25.0, 200 27.7 | 27.6, of 300 operators 26.3 | 27.9; 1,500 anchors, 200 keys 33.6 | 29.7).
static uint32_t short_keys(uint32_t n, uint32_t m, uint32_t k) {
  const uint32_t fit = 2 * kShortMap / (9 * map_stride(n, m)), fast = k < 768 ? 120 : k < 1280 ? 180 : kShortKeys;
  return fit < fast ? fit : fast;
}

// the bit of `word` with `need` set bits below it
__device__ __forceinline__ uint32_t select_bit(uint32_t word, uint32_t need) {
  uint32_t at = 0;
#pragma unroll
  for (uint32_t half = 16; half; half /= 2) {
    const uint32_t below = __popc(word & ((1u << half) - 1));
    if (need >= below) { need -= below; word >>= half; at += half; }
    else word &= (1u << half) - 1;
  }
  return at;
}

// Whether operators spread over a sequence have more than that many keys.
static bool more_keys(const ss_op_t *ops, uint32_t n, uint32_t most) {
  constexpr uint32_t kLooks = 256, kSlots = 4 * kLooks;
  uint16_t slots[kSlots] = {};                               // 1 + the look that a key was met at
  uint32_t keys = 0;
  for (uint32_t x = 0; x < std::min(n, kLooks); ++x) {
    const ss_op_t &o = ops[(uint64_t)x * n / std::min(n, kLooks)];
    uint32_t h = ss_key_hash(o.op_token, o.stack_hash, o.sig, 64 - 10);
    static_assert(kSlots == 1u << 10, "hash bits");
    for (; slots[h]; h = (h + 1) % kSlots) {
      const ss_op_t &r = ops[(uint64_t)(slots[h] - 1) * n / std::min(n, kLooks)];
      if (r.op_token == o.op_token && r.stack_hash == o.stack_hash && r.sig == o.sig) break;
    }
    if (slots[h]) continue;
    slots[h] = (uint16_t)(x + 1);
    if (++keys > most) return true;
  }
  return false;
}

__global__ __launch_bounds__(kShortThreads) void ss_match_short_kernel(ShortArgs a) {
  extern __shared__ uint4 short_lds[];
  ShortLds &sh = *reinterpret_cast<ShortLds *>(short_lds);
  constexpr uint32_t kShift = 64 - 13;
  static_assert(kShortSlots == 1u << 13, "hash bits");
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  ss_op_t o[kShortPer];                                        // of cur, then of ref: the first ones of a thread stand at one place
  uint32_t at[kShortPer];                                      // in LDS cur is first
#pragma unroll
  for (uint32_t u = 0; u < kShortPer; ++u) {
    const uint32_t i = u % (kShortPer / 2) * kShortThreads + tid;
    const bool is_ref = u >= kShortPer / 2;
    at[u] = i < (is_ref ? a.n : a.m) ? (is_ref ? a.m : 0) + i : kNoOp;
    if (at[u] != kNoOp) o[u] = (is_ref ? a.ref : a.cur)[i];
  }
  ss_anchor_t anc[kShortMine];
#pragma unroll
  for (uint32_t u = 0; u < kShortMine; ++u) {
    const uint32_t x = u * kShortThreads + tid;
    if (x < a.k) anc[u] = a.anchors[x];
  }
  for (uint32_t i = tid; i < kShortSlots / 4; i += kShortThreads) short_lds[i] = uint4{0, 0, 0, 0};
  if (tid == 0) {
    sh.n_keys = sh.lost = sh.bad = 0;
    sh.dot = sh.na = sh.nb = 0;
  }
#pragma unroll
  for (uint32_t u = 0; u < kShortPer; ++u) {
    const uint32_t i = at[u];
    if (i == kNoOp) continue;
    sh.table.token[i] = o[u].op_token; sh.table.stack[i] = o[u].stack_hash; sh.table.sig[i] = o[u].sig;
    if (u < kShortPer / 2) {
      sh.n_out[i] = o[u].n_out;
      sh.cur_type[i] = (uint8_t)o[u].sig;
    }
  }
  __syncthreads();
  // at most kShortSlots / 2 keys: a free or matching slot is met
  uint32_t slot[kShortPer];
#pragma unroll
  for (uint32_t u = 0; u < kShortPer; ++u) {
    const uint32_t i = at[u];
    slot[u] = 0;
    if (i == kNoOp) continue;
    uint32_t h = ss_key_hash(o[u].op_token, o[u].stack_hash, o[u].sig, kShift);
    for (uint32_t probe = 0; probe < kShortSlots; ++probe) {
      uint32_t seen = *(volatile uint32_t *)(sh.table.rep + h);
      if (!seen) {
        seen = atomicCAS(sh.table.rep + h, 0u, i + 1);
        if (!seen) {
          const uint32_t id = atomicAdd(&sh.n_keys, 1u);
          sh.table.id[h] = id;
          if (id < kShortKeys) { sh.key_token[id] = o[u].op_token; sh.key_sig[id] = o[u].sig; }
          break;
        }
      }
      const uint32_t r = seen - 1;
      if ((sh.table.token[r] == o[u].op_token) & (sh.table.stack[r] == o[u].stack_hash) & (sh.table.sig[r] == o[u].sig)) break;
      h = (h + 1) % kShortSlots;
    }
    slot[u] = h;
  }
  __syncthreads();
  const uint32_t keys = sh.n_keys, ref_words = (a.n + 31) / 32, cur_words = (a.m + 31) / 32, cur_at = up_to_four(ref_words),
                 stride = map_stride(a.n, a.m);
  const uint32_t level_words = keys * stride;
  if (keys > a.most_keys) {
    if (tid == 0) *a.too_many = keys;
    ss_tell_host(a.done);
    return;
  }
  uint32_t id[kShortPer];
#pragma unroll
  for (uint32_t u = 0; u < kShortPer; ++u) id[u] = sh.table.id[slot[u]];
  for (uint32_t q = tid / 16; q < keys; q += kShortThreads / 16) {            // sixteen lanes look at sixteen keys for one
    const uint32_t r = lane % 16, token = sh.key_token[q], sig = sh.key_sig[q];
    uint32_t lowest[2] = {kNoOp, kNoOp};
    for (uint32_t q0 = 0; q0 < keys && lowest[0] == kNoOp; q0 += 16) {        // the third level's is no higher than the second's
      const bool key = q0 + r < keys;
      const uint32_t its = key ? sh.key_token[q0 + r] : 0, its_sig = key ? sh.key_sig[q0 + r] : 0;
      const uint64_t third = __ballot(key & (its == token)) >> (lane & 48) & 0xFFFF, second = __ballot(key & (its == token) & (its_sig == sig)) >> (lane & 48) & 0xFFFF;
      if (third && lowest[1] == kNoOp) lowest[1] = q0 + (uint32_t)__builtin_ctz((uint32_t)third);
      if (second) lowest[0] = q0 + (uint32_t)__builtin_ctz((uint32_t)second);
    }
    if (r < 2) sh.lowest[r][q] = (uint8_t)lowest[r];
  }
  __syncthreads();
  for (uint32_t i = tid; i < (3 * level_words + 3) / 4; i += kShortThreads) short_lds[i] = uint4{0, 0, 0, 0};
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kShortPer; ++u) {
    const uint32_t i = at[u], j = i - a.m;
    if (i == kNoOp) continue;
    if (u < kShortPer / 2) {
      atomicOr(&sh.map[id[u] * stride + cur_at + i / 32], 1u << (i % 32));
    } else {
      sh.ref_key[j] = (uint16_t)id[u];
      atomicOr(&sh.map[id[u] * stride + j / 32], 1u << (j % 32));
    }
  }
  __syncthreads();
  for (uint32_t q = tid / 16; q < keys; q += kShortThreads / 16) {            // the other levels' maps: sixteen lanes add a key's
    const uint32_t second = level_words + sh.lowest[0][q] * stride, third = 2 * level_words + sh.lowest[1][q] * stride;
    for (uint32_t w = lane % 16; w < cur_at + cur_words; w += 16) {
      const uint32_t v = sh.map[q * stride + w];
      if (!v) continue;
      atomicOr(&sh.map[second + w], v);
      atomicOr(&sh.map[third + w], v);
    }
  }
  __syncthreads();
  // sixteen lanes count the places of a key at a level, four words of its maps each; what isn't the lowest of its equals has none
  uint16_t *const before = reinterpret_cast<uint16_t *>(sh.map + 3 * level_words);
  for (uint32_t g = tid / 16; g < 3 * keys; g += kShortThreads / 16) {
    const uint32_t w = lane % 16 * 4, row = g * stride + w;
    const bool in_ref = w < ref_words, in_cur = w < cur_words;
    const uint4 b = in_ref ? *reinterpret_cast<const uint4 *>(sh.map + row) : uint4{}, c = in_cur ? *reinterpret_cast<const uint4 *>(sh.map + row + cur_at) : uint4{};
    const uint2 x = counts_before(b), y = counts_before(c);
    if (in_ref) *reinterpret_cast<uint2 *>(before + row) = x;
    if (in_cur) *reinterpret_cast<uint2 *>(before + row + cur_at) = y;
  }
  __syncthreads();
  {
    uint64_t dot = 0, na = 0, nb = 0;
    uint32_t bad = 0;
#pragma unroll
    for (uint32_t u = 0; u < kShortPer / 2; ++u) {             // the shorter sequence is padded with token 0
      const uint32_t x = at[u] != kNoOp ? o[u].op_token : 0, y = at[u + kShortPer / 2] != kNoOp ? o[u + kShortPer / 2].op_token : 0;
      bad |= x >= kTokenLimit || y >= kTokenLimit;
      dot += (uint64_t)x * y; na += (uint64_t)x * x; nb += (uint64_t)y * y;
    }
    const uint64_t any = __ballot(bad != 0);                   // of tokens that are too large the sums may wrap to 0
    if (any | __ballot((na | nb) != 0)) {
      dot = ss_wave_sum(dot); na = ss_wave_sum(na); nb = ss_wave_sum(nb);
      if (lane == 63) {
        atomicAdd(&sh.dot, (unsigned long long)dot);
        atomicAdd(&sh.na, (unsigned long long)na);
        atomicAdd(&sh.nb, (unsigned long long)nb);
        if (any) sh.bad = 1;
      }
    }
  }
  int32_t land[kShortMine];
  uint8_t level[kShortMine];
#pragma unroll
  for (uint32_t u = 0; u < kShortMine; ++u) {
    const uint32_t x = u * kShortThreads + tid, i = x < a.k ? anc[u].ref_op : a.n;
    land[u] = -1;
    level[u] = 255;
    if (i >= a.n) continue;
    const uint32_t key = sh.ref_key[i], type = sh.key_sig[key] & 0xFFu;
    if (sh.key_token[key] == 0) continue;
#pragma unroll 1
    for (uint32_t L = 0; L < 3; ++L) {
      const uint32_t row = (L ? L * keys + sh.lowest[L - 1][key] : key) * stride, word = row + i / 32;
      const uint32_t ordinal = before[word] + (uint32_t)__popc(sh.map[word] & ((1u << (i % 32)) - 1));
      // the last word of cur with no more than that many places before it
      const uint16_t *const upto = before + row + cur_at;
      uint32_t w = 0;
#pragma unroll
      for (uint32_t step = 16; step; step /= 4) {
        const uint32_t end = cur_words - 1, p = w + step, q = p + step, r = q + step;
        const uint32_t at_p = upto[min(p, end)], at_q = upto[min(q, end)], at_r = upto[min(r, end)];
        w += step * (((p <= end) & (at_p <= ordinal)) + ((q <= end) & (at_q <= ordinal)) + ((r <= end) & (at_r <= ordinal)));
      }
      const uint32_t bits = sh.map[row + cur_at + w], need = ordinal - upto[w];
      const uint32_t j = w * 32 + select_bit(bits, need);
      if (need < (uint32_t)__popc(bits) && anc[u].out_slot < sh.n_out[j] && sh.cur_type[j] == type) {
        land[u] = (int32_t)j;
        level[u] = (uint8_t)L;
        break;
      }
    }
  }
  __syncthreads();
  // a place that several land on goes to the lowest anchor
  uint32_t bits = 6;
  while ((1u << bits) < 2 * a.k) ++bits;
  for (uint32_t i = tid; i < 1u << bits; i += kShortThreads) {
    sh.claims.key[i] = kEmptyKey;
    sh.claims.owner[i] = ~0u;
  }
  __syncthreads();
  uint32_t mine[kShortMine];
#pragma unroll
  for (uint32_t u = 0; u < kShortMine; ++u) {
    const uint32_t x = u * kShortThreads + tid;
    if (land[u] < 0) continue;
    const unsigned long long key = (unsigned long long)(uint32_t)land[u] << 32 | anc[u].out_slot;
    uint32_t s = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> (64 - bits));
    for (uint32_t probe = 0; probe < 1u << bits; ++probe) {    // at most k places in 2k slots
      const unsigned long long seen = atomicCAS(&sh.claims.key[s], kEmptyKey, key);
      if (seen == kEmptyKey || seen == key) break;
      s = (s + 1) & ((1u << bits) - 1);
    }
    atomicMin(&sh.claims.owner[s], x);
    mine[u] = s;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kShortMine; ++u) {
    const uint32_t x = u * kShortThreads + tid;
    if (land[u] >= 0 && sh.claims.owner[mine[u]] != x) { land[u] = -1; level[u] = 255; }
    if (x < a.k) {
      a.new_idx[x] = land[u];
      a.level[x] = level[u];
    }
    const uint64_t b = __ballot(x < a.k && land[u] < 0);
    if (lane == 0 && b) atomicAdd(&sh.lost, (uint32_t)__popcll(b));
  }
  __syncthreads();
  if (tid == 0) {
    *a.part = ss_cosine_part{sh.dot, sh.na, sh.nb, sh.bad};
    *a.lost = sh.lost;
  }
  ss_tell_host(a.done);
}

// ---- many anchors: the distinct keys first ------------------------------------------------------------------------
//
// 8,001 anchors over 18,464 + 18,467 operators: comparing every anchor with every operator is bound by the issue of 300
// million compares (186 us).  With some forty distinct keys the three launches below take 3.9 us for the keys, 4.1 to number
// their occurrences and 8.8 for the anchors.  (A workgroup per key that went through both sequences and listed its places took
// 16.5 us, bound by the turns of one workgroup, and the anchors 7.8.)

// Per level: an open-addressing table of at least 2k slots, up to 2^kKeyBits, holding the anchor that stands for a key, and
// beside it the key itself with its number; and for every operator of both sequences the number of its key and how many with
// that key come before it in its chunk.
struct KeyTable {
  uint32_t *rep[3];
  uint4 *key[3];               // {1 + number, token, stack, sig}; zeros: no key
  uint32_t *n_used;            // [3]: distinct keys
  uint32_t *info[2][3];        // [0] ref, [1] cur: number << kRankBits | rank in the chunk, or kNoKey; whole chunks
  uint32_t *count[2];          // [level][chunk][number]: occurrences in the chunk, n_used of the level to a chunk
  uint32_t mask, shift, max_keys;
  uint32_t probes;             // slots that are looked at for a key at most
  uint32_t chunk_bits[2], chunks[2];         // operators of a chunk (a power of two), chunks
};
// They take the calls of that many comparisons of an anchor with an operator (10 us of comparing), and those where a single
// search goes through that many operators, whatever the number of anchors: 500 anchors over 6,100 + 6,100 operators 38.6 us a
// call with some forty keys and 47.6 with a key each, a search each 43.8 and 45.9; 300 over 18,464 53.7 and 56.6 against 94.9
// and 90.4; 20 over 65,536 105 against 279; but 500 over 5,000 38.3 and 51 against 41.7 and 40.
constexpr uint64_t kManyPairs = 1ull << 24, kLongSearch = 12000;
constexpr uint32_t kRankBits = 20, kNoKey = 0xFFFFFFFFu;
constexpr uint32_t kChunkThreads = 512, kMaxChunks = 256;
static_assert((1u << 23) / kMaxChunks < 1u << kRankBits, "a rank fits its bits");

// More distinct keys (of all levels) than this, and an anchor is searched for by itself.
constexpr uint32_t kMaxKeys = 4096;
static_assert(kMaxKeys <= 1u << (32 - kRankBits), "a key's number fits its bits");

// The tables are cleared by every call, 60 bytes a slot, and no more than kMaxKeys of their keys are made use of: 2^16 slots
// do for any number of anchors (2^24 over 2^23 operators: 1.5 GiB of scratch, with 2k slots 3.8, the call 190 ms; 2^20 over
// 2^20 0.14 and 0.28 GiB, 5.1 and 5.2 ms).  Keys may outnumber these slots.  At most one slot in sixteen is taken while the
// keys can be made use of, so a key that finds no place in kProbes of them says that there are too many.
constexpr uint32_t kKeyBits = 16, kProbes = 32, kTooMany = 1u << 30;
static_assert(3 * ((uint64_t)kTooMany + (1u << kKeyBits)) < 1ull << 32, "the levels' numbers are added");

__device__ __forceinline__ bool same_at(const ss_op_t &x, const ss_op_t &y, int L) {
  return (x.op_token == y.op_token) & ((L == 2) | (x.sig == y.sig)) & ((L != 0) | (x.stack_hash == y.stack_hash));
}

__device__ __forceinline__ unsigned long long level_hash(const ss_op_t &o, int L) {
  unsigned long long x = o.op_token;
  if (L < 2) x |= (unsigned long long)o.sig << 32;
  if (L < 1) x ^= (unsigned long long)o.stack_hash << 18;
  return x * 0x9E3779B97F4A7C15ull;
}

// workgroup (x, L): the anchors' keys of level L.  They are few, and every anchor would go for the same few slots: only the
// first of each key within the workgroup (found through a table in LDS) goes.
__global__ __launch_bounds__(256) void ss_keys_kernel(AnchorArgs g, KeyTable q) {
  constexpr uint32_t kSlots = 512, kShift = 64 - 9;
  __shared__ uint32_t first[kSlots];
  __shared__ ss_op_t ops[256];
  const uint32_t a = blockIdx.x * 256 + threadIdx.x;
  const int L = blockIdx.y;
  ss_op_t R = {0, 0, 0, 0};
  if (a < g.k) {
    const uint32_t i = g.anchors[a].ref_op;
    if (i < g.n) R = g.ref[i];
  }
  const bool live = R.op_token != 0;
  ops[threadIdx.x] = R;
  for (uint32_t i = threadIdx.x; i < kSlots; i += 256) first[i] = 0;
  __syncthreads();
  const unsigned long long x = level_hash(R, L);
  uint32_t l = (uint32_t)(x >> kShift);
  bool goes = false;
  for (uint32_t probe = 0; live && probe < kSlots; ++probe) {  // at most 256 keys in 512 slots
    uint32_t seen = *(volatile uint32_t *)(first + l);
    if (!seen) {
      seen = atomicCAS(first + l, 0u, threadIdx.x + 1);
      if (!seen) { goes = true; break; }
    }
    if (same_at(ops[seen - 1], R, L)) break;
    l = (l + 1) % kSlots;
  }
  // a slot holds 1 + the anchor and seven more bits of the hash: another key's anchor is rarely looked at (two dependent loads)
  constexpr uint32_t kTagShift = 25;
  uint32_t h = (uint32_t)(x >> q.shift);
  const uint32_t tag = (uint32_t)(x >> (q.shift - 7)) & 127u, entry = tag << kTagShift | (a + 1);
  bool won = false, placed = !goes;
  for (uint32_t probe = 0; !placed && probe < q.probes; ++probe) {
    uint32_t seen = __hip_atomic_load(q.rep[L] + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!seen) {
      seen = atomicCAS(q.rep[L] + h, 0u, entry);
      if (!seen) { won = placed = true; break; }
    }
    placed = seen >> kTagShift == tag && same_at(g.ref[g.anchors[(seen & ((1u << kTagShift) - 1)) - 1].ref_op], R, L);
    if (!placed) h = (h + 1) & q.mask;
  }
  if (!placed) atomicMax(q.n_used + L, kTooMany);
  // numbers for a wavefront's new keys at once: additions to one word are served one after the other
  const uint64_t winners = __ballot(won);
  if (!winners) return;
  const int lane = threadIdx.x & 63;
  uint32_t number = 0;
  if (lane == __builtin_ctzll(winners)) number = atomicAdd(q.n_used + L, (uint32_t)__popcll(winners));
  number = (uint32_t)__builtin_amdgcn_readlane((int)number, __builtin_ctzll(winners));
  number += (uint32_t)__popcll(winners & (lane ? (~0ull >> (64 - lane)) : 0ull));
  if (won) q.key[L][h] = uint4{number + 1, R.op_token, L < 1 ? R.stack_hash : 0, L < 2 ? R.sig : 0};
}

// Where the counts of a level's chunks are.
__device__ __forceinline__ uint32_t *counts_of(const KeyTable &q, int which, int L) {
  uint32_t before = 0;
  for (int l = 0; l < L; ++l) before += q.n_used[l];
  return q.count[which] + (size_t)before * q.chunks[which];
}

// Workgroup (x, L): the operators of a chunk of ref or cur at level L, 512 at a time.  Equal numbers within a wavefront are
// found by a ballot for each of their bits, and wavefronts tell each other their counts.
__global__ __launch_bounds__(kChunkThreads) void ss_chunks_kernel(AnchorArgs g, KeyTable q) {
  constexpr uint32_t W = kChunkThreads / 64;
  __shared__ uint8_t mine[W][kMaxKeys];
  __shared__ uint32_t seen[kMaxKeys];
  const int L = blockIdx.y;
  const uint32_t keys = q.n_used[L], tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (q.n_used[0] + q.n_used[1] + q.n_used[2] > q.max_keys) return;
  const uint32_t which = blockIdx.x >= q.chunks[0], chunk = blockIdx.x - (which ? q.chunks[0] : 0);
  const ss_op_t *const seq = which ? g.cur : g.ref;
  const uint32_t len = which ? g.m : g.n, size = 1u << q.chunk_bits[which], lo = chunk * size;
  const uint32_t bits = keys > 1 ? 32 - __builtin_clz(keys - 1) : 0;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (uint32_t u = tid; u < keys; u += kChunkThreads) seen[u] = 0;
  for (uint32_t at = 0; at < size; at += kChunkThreads) {
    const uint32_t i = lo + at + tid;
    ss_op_t o = {0, 0, 0, 0};
    if (i < len) o = seq[i];
    for (uint32_t u = tid; u < keys; u += kChunkThreads)
#pragma unroll
      for (uint32_t v = 0; v < W; ++v) mine[v][u] = 0;
    uint32_t id = kNoKey;
    if (o.op_token) {
      uint32_t h = (uint32_t)(level_hash(o, L) >> q.shift);
      for (uint32_t probe = 0; probe <= q.mask; ++probe) {     // half of the slots are free at least
        const uint4 k = q.key[L][h];
        if (!k.x) break;
        if ((k.y == o.op_token) & ((L == 2) | (k.w == o.sig)) & ((L != 0) | (k.z == o.stack_hash))) { id = k.x - 1; break; }
        h = (h + 1) & q.mask;
      }
    }
    const bool live = id != kNoKey;
    uint64_t same = __ballot(live);
    for (uint32_t b = 0; b < bits; ++b) {
      const bool set = (id >> b) & 1u;
      const uint64_t with = __ballot(set);
      same &= set ? with : ~with;
    }
    const uint32_t rank = (uint32_t)__popcll(same & below);
    __syncthreads();
    if (live && !rank) mine[w][id] = (uint8_t)__popcll(same);
    __syncthreads();
    uint32_t before = 0;
    if (live) {
      before = seen[id] + rank;
#pragma unroll
      for (uint32_t v = 0; v < W; ++v) before += v < w ? mine[v][id] : 0;
    }
    q.info[which][L][i] = live ? id << kRankBits | before : kNoKey;
    __syncthreads();
    for (uint32_t u = tid; u < keys; u += kChunkThreads) {
      uint32_t all = 0;
#pragma unroll
      for (uint32_t v = 0; v < W; ++v) all += mine[v][u];
      seen[u] += all;                                          // each thread its own keys: zeroed and read by others behind barriers
    }
  }
  uint32_t *const out = counts_of(q, which, L) + (size_t)chunk * keys;
  for (uint32_t u = tid; u < keys; u += kChunkThreads) out[u] = seen[u];
}

// The operator of cur with the number and ordinal of operator i of ref at level L, or -1; by one wavefront.
__device__ __forceinline__ int32_t look_up(const KeyTable &q, uint32_t i, int L) {
  const uint32_t lane = threadIdx.x & 63, keys = q.n_used[L], info = q.info[0][L][i], id = info >> kRankBits;
  const uint32_t *const in_ref = counts_of(q, 0, L), *const in_cur = counts_of(q, 1, L);
  const uint32_t c = i >> q.chunk_bits[0];
  uint32_t ordinal = 0;
  for (uint32_t c0 = 0; c0 < c; c0 += 64) ordinal += c0 + lane < c ? in_ref[(size_t)(c0 + lane) * keys + id] : 0;
  ordinal = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_u32(ordinal), 63) + (info & ((1u << kRankBits) - 1));
  for (uint32_t c0 = 0, before = 0; c0 < q.chunks[1]; c0 += 64) {
    const uint32_t v = c0 + lane < q.chunks[1] ? in_cur[(size_t)(c0 + lane) * keys + id] : 0, upto = before + wave_scan_u32(v);
    const uint64_t there = __ballot(upto > ordinal);
    if (there) {
      const int l = __builtin_ctzll(there);
      const uint32_t want = id << kRankBits | (ordinal - (uint32_t)__builtin_amdgcn_readlane((int)(upto - v), l));
      const uint32_t lo = (c0 + (uint32_t)l) << q.chunk_bits[1];
      const uint4 *const infos = reinterpret_cast<const uint4 *>(q.info[1][L] + lo);
      for (uint32_t o = 0; o < 1u << q.chunk_bits[1]; o += 512) {
        const uint4 a = infos[o / 4 + lane], b = infos[o / 4 + 64 + lane];
        const uint32_t at = a.x == want ? 0 : a.y == want ? 1 : a.z == want ? 2 : a.w == want ? 3 : b.x == want ? 256
                          : b.y == want ? 257 : b.z == want ? 258 : b.w == want ? 259 : kNoKey;
        const uint64_t hit = __ballot(at != kNoKey);
        if (hit) {
          const int x = __builtin_ctzll(hit);
          return (int32_t)(lo + o + 4 * (uint32_t)x + (uint32_t)__builtin_amdgcn_readlane((int)at, x));
        }
      }
      return -1;
    }
    before = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
  }
  return -1;
}

// A wavefront per anchor looks its ordinal up, four to a workgroup or, up to kOneEach anchors, one.  With too many distinct
// keys for numbers an anchor is searched for by itself: by its workgroup where that has no other, else by its wavefront.
// 1,000 anchors over 65,536 operators 302 us a call with a workgroup each, 711 with a wavefront each; 4,000 over 18,464
// operators 180 and 255, 8,001 260 and 296, 20,000 488 and 478.  Where there are numbers a workgroup each costs its launch:
// 8,001 anchors 227 us against 222, 2,048 nothing to be seen.
constexpr uint32_t kOneEach = 4096;

__global__ __launch_bounds__(256) void ss_lookup_kernel(AnchorArgs g, KeyTable q, uint32_t per) {
  __shared__ AnchorShared sh;
  const bool listed = q.n_used[0] + q.n_used[1] + q.n_used[2] <= q.max_keys;
  if (!listed && per == 1) {
    search_anchor(g, blockIdx.x, sh);
    return;
  }
  const uint32_t w = threadIdx.x >> 6, a = blockIdx.x * per + w;
  if (w >= per || a >= g.k) return;                          // uniform per wavefront
  const uint32_t i = g.anchors[a].ref_op, slot = g.anchors[a].out_slot;
  int32_t result = -1;
  uint8_t level = 255;
  if (i < g.n && g.ref[i].op_token != 0) {
    const ss_op_t R = g.ref[i];
    if (listed) {
      // a landing at the first level is the rule: the others are looked at only without one
      for (int L = 0; L < 3 && result < 0; ++L) {
        int32_t f[3] = {-1, -1, -1};
        f[0] = look_up(q, i, L);
        uint8_t unused;
        result = choose_landing(g.cur, R, slot, f, unused);
        if (result >= 0) level = (uint8_t)L;
      }
    } else {
      result = search_alone(g, R, i, slot, level);
    }
  }
  if ((threadIdx.x & 63) == 0) {
    g.land[a] = result;
    g.lvl[a] = level;
    if (result >= 0) g.slot_of[a] = claim(g.table, result, slot, a);
  }
}

__global__ __launch_bounds__(256) void ss_injective_kernel(AnchorArgs g, int32_t *new_idx, uint8_t *level,
                                                           uint32_t *lost_of_wg, ss_done done) {
  __shared__ uint32_t lost_of[4];
  const uint32_t a = blockIdx.x * 256 + threadIdx.x;
  bool lost = false;
  if (a < g.k) {
    int32_t j = g.land[a];
    uint8_t L = g.lvl[a];
    if (j >= 0 && g.table.owner[g.slot_of[a]] != a) { j = -1; L = 255; }
    new_idx[a] = j;
    level[a] = L;
    lost = j < 0;
  }
  const uint64_t b = __ballot(lost);
  if ((threadIdx.x & 63) == 0) lost_of[threadIdx.x >> 6] = (uint32_t)__popcll(b);
  __syncthreads();
  if (threadIdx.x == 0) lost_of_wg[blockIdx.x] = lost_of[0] + lost_of[1] + lost_of[2] + lost_of[3];
  ss_tell_host(done);
}

}  // namespace

// The stage machine of Algo. 1 as a table: a stage is left for `next` once more than `patience`
// consecutive similar iterations have been counted in it (the count includes the current one), and the
// count starts over if `restart` is set; a stage without a row entry to leave (Stable) only counts.
// Any dissimilar iteration sends every stage back to WarmUp with the count at zero.
struct StagePromotion { bool leaves; uint32_t next; bool restart; };

static void stage_step(ss_ctx *ctx, bool similar) {
  if (!similar) {
    ctx->stage = SS_STAGE_WARMUP;
    ctx->stable_step = 0;
    return;
  }
  const uint32_t patience[3] = {ctx->cfg.stage_m, ctx->cfg.stage_n, 0};
  static const StagePromotion promote[3] = {
      /* WarmUp    */ {true, SS_STAGE_GENPOLICY, true},
      /* GenPolicy */ {true, SS_STAGE_STABLE, false},
      /* Stable    */ {false, SS_STAGE_STABLE, false}};
  const uint32_t from = ctx->stage;
  ctx->stable_step += 1;
  if (from <= SS_STAGE_STABLE && promote[from].leaves && ctx->stable_step > patience[from]) {
    ctx->stage = promote[from].next;
    if (promote[from].restart) ctx->stable_step = 0;
  }
}

extern "C" int ss_match_sequence(ss_ctx *ctx, const ss_op_t *ref, uint32_t n, const ss_op_t *cur, uint32_t m,
                                 const ss_anchor_t *anchors, uint32_t k, uint32_t flags, int32_t *new_idx,
                                 uint8_t *level, ss_match_result_t *res) {
  return ss_guard([&]() -> int {
    if (!ctx || !res || (n && !ref) || (m && !cur)) return SS_E_INVAL;
    if (k && (!anchors || !new_idx || !level)) return SS_E_INVAL;
    if (n > kLenLimit || m > kLenLimit || k > (1u << 24)) return SS_E_INVAL;
    const bool hist = (flags & SS_MATCH_HISTOGRAM) != 0;
    const bool aligned = (flags & SS_MATCH_ALIGN) != 0;
    // verdict, stage machine and counters from the three sums: the same for both routes below
    auto finish = [&](const uint64_t sm[3], uint32_t unm) {
      res->dot = sm[0]; res->na = sm[1]; res->nb = sm[2];
      bool similar;
      if (n == 0 && m == 0) {
        similar = true;
      } else {
        const uint64_t diff = n > m ? n - m : m - n;
        const bool len_ok = 20ull * diff < (uint64_t)n;
        // cos > 0.95  <=>  dot > 0 and 400 dot^2 > 361 na nb; sums < 2^59, so both sides < 2^127
        const unsigned __int128 lhs = (unsigned __int128)400 * sm[0] * sm[0];
        const unsigned __int128 rhs = (unsigned __int128)361 * sm[1] * sm[2];
        similar = len_ok && sm[0] > 0 && lhs > rhs;
      }
      res->similar = similar ? 1u : 0u;
      if (flags & SS_MATCH_STEP_STAGE) stage_step(ctx, similar);
      res->stage = ctx->stage;
      res->stable_step = ctx->stable_step;
      res->n_unmatched = unm;
      for (uint32_t a = 0; a < k; ++a) ctx->stats.match_levels[level[a] <= SS_LEVEL_ALIGN ? level[a] : 4]++;
    };
    // The current sequence IS the reference one (the Stable stage of a fixed operator sequence, Sec. 3):
    // no search is needed.  Every operator is its own counterpart at the strictest level, the three sums
    // coincide, and what remains of the definition (a landing place needs more than out_slot outputs, the
    // lowest anchor index keeps a shared place) is evaluated here on the host in one pass, without a
    // round trip to the GPU.  Results are those of the kernels below on the same input.
    if (!hist && n == m && (n == 0 || std::memcmp(ref, cur, (size_t)n * sizeof(ss_op_t)) == 0)) {
      uint64_t sq = 0;
      for (uint32_t i = 0; i < n; ++i) {
        if (cur[i].op_token >= kTokenLimit) return SS_E_INVAL;
        sq += (uint64_t)cur[i].op_token * cur[i].op_token;
      }
      uint32_t unm = 0;
      if (k) {
        std::unordered_map<uint64_t, uint32_t> first;          // (operator, slot) -> lowest anchor index landing there
        if (!aligned) first.reserve(2 * (size_t)k);
        for (uint32_t a = 0; a < k; ++a) {
          const uint32_t i = anchors[a].ref_op, sl = anchors[a].out_slot;
          const bool lands = i < n && sl < cur[i].n_out && (aligned || cur[i].op_token != 0);
          new_idx[a] = lands ? (int32_t)i : -1;
          level[a] = lands ? (uint8_t)(aligned ? SS_LEVEL_ALIGN : 0) : (uint8_t)255;
          if (lands && !aligned) {
            auto ins = first.emplace(((uint64_t)i << 32) | sl, a);
            if (!ins.second) { new_idx[a] = -1; level[a] = 255; }   // an earlier anchor owns the place
          }
          unm += new_idx[a] < 0;
        }
      }
      const uint64_t sm[3] = {sq, sq, sq};
      finish(sm, unm);
      return SS_OK;
    }
    // Aligned: the sums are taken by the aligner's first kernel, which reads both sequences anyway (a pass of their own before it,
    // with a wait: some 560 operators each 36.1 us a call, so 28.3; 1,240 52.4 and 44.0).
    if (k && aligned && !hist && n && m && n <= SS_ALIGN_LEN_LIMIT && m <= SS_ALIGN_LEN_LIMIT) {
      std::vector<int32_t> ref_to_cur(n);
      ss_cosine_part sums;
      uint32_t lcs = 0, n_unm = 0;
      const int rc = ss_align_core(ctx, ref, n, cur, m, ref_to_cur.data(), &lcs, nullptr, &sums);
      if (rc != SS_OK) return rc;
      if (sums.bad) return SS_E_INVAL;                       // a token beyond 2^18
      ss_align_anchors(ref, n, cur, ref_to_cur.data(), anchors, k, new_idx, level, &n_unm);
      const uint64_t sm[3] = {sums.dot, sums.na, sums.nb};
      finish(sm, n_unm);
      return SS_OK;
    }
    const bool search = k && !aligned;
    const size_t op_bytes = sizeof(ss_op_t), in_bytes = ((size_t)n + m) * op_bytes + (size_t)k * sizeof(ss_anchor_t);
    // Inputs up to this size go through pinned memory that the first kernel reads (and copies on the way) and the last
    // one writes: a copy call for each array costs more than the kernels.  Beyond it the copy engine is as fast and
    // nothing that large is kept pinned.
    const bool mapped = in_bytes <= (4u << 20);
    const uint64_t pairs = (uint64_t)k * ((uint64_t)n + m);
    const bool listed = search && (pairs > kManyPairs || (uint64_t)n + m >= kLongSearch);
    const uint32_t len = n > m ? n : m, wgs = std::min(256u, std::max(1u, (len + 255) / 256));
    const uint32_t out_wgs = (k + 255) / 256;
    // table of the injectivity pass: a power of two of at least 2k slots
    uint32_t bits = 6;
    while ((1ull << bits) < 2ull * k) ++bits;
    const size_t slots = (size_t)1 << bits;
    const uint32_t key_bits = std::min(bits, kKeyBits);       // of the anchors' distinct keys
    const size_t key_slots = (size_t)1 << key_bits;
    size_t off = 0, hoff = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += ss_align_up(bytes, 256); return o; };
    auto htake = [&](size_t bytes) { size_t o = hoff; hoff += ss_align_up(bytes, 256); return o; };
    const size_t o_ref = take((size_t)n * op_bytes), o_cur = take((size_t)m * op_bytes), o_anc = take((size_t)k * sizeof(ss_anchor_t));
    const size_t o_land = take((size_t)k * 4), o_lvl = take(k), o_slot = take((size_t)k * 4);
    const size_t o_idx = take(mapped ? 0 : (size_t)k * 4), o_level = take(mapped ? 0 : k);
    const size_t o_ones = take(search ? slots * 8 : 0), o_owner = take(search ? slots * 4 : 0), ones_end = off;
    const size_t o_hist = take(hist ? 2 * (size_t)kTokenLimit * 4 + 256 : 0);
    size_t o_rep[3];
    for (size_t &o : o_rep) o = take(listed ? key_slots * 4 : 0);
    size_t o_key[3], o_info[2][3], o_count[2];
    for (size_t &o : o_key) o = take(listed ? key_slots * 16 : 0);
    const size_t o_n_used = take(listed ? 3 * 4 : 0), zeros_end = off;
    const uint32_t max_keys = (uint32_t)std::min<uint64_t>(kMaxKeys, 3ull * k), lens[2] = {n, m};
    uint32_t chunk_bits[2], chunks[2];
    for (int x = 0; x < 2; ++x) {
      chunk_bits[x] = 9;                                     // as many operators as a workgroup has threads
      while (lens[x] > (uint64_t)kMaxChunks << chunk_bits[x]) ++chunk_bits[x];
      chunks[x] = (uint32_t)(((uint64_t)lens[x] + (1u << chunk_bits[x]) - 1) >> chunk_bits[x]);
      for (int L = 0; L < 3; ++L) o_info[x][L] = take(listed ? ((size_t)chunks[x] << chunk_bits[x]) * 4 : 0);
      o_count[x] = take(listed ? (size_t)chunks[x] * max_keys * 4 : 0);
    }
    const size_t ho_ref = htake(mapped ? (size_t)n * op_bytes : 0), ho_cur = htake(mapped ? (size_t)m * op_bytes : 0);
    const size_t ho_anc = htake(mapped ? (size_t)k * sizeof(ss_anchor_t) : 0);
    const size_t ho_idx = htake(mapped ? (size_t)k * 4 : 0), ho_level = htake(mapped ? k : 0);
    const size_t ho_part = htake(kMaxParts * sizeof(ss_cosine_part)), ho_lost = htake(std::max<size_t>(2, out_wgs) * 4);
    int rc = ss_scratch_reserve(ctx, off, hoff);
    if (rc != SS_OK) return rc;
    uint8_t *d = (uint8_t *)ctx->d_scratch, *h = (uint8_t *)ctx->h_scratch, *hd = nullptr;
    SS_HIP(hipHostGetDevicePointer((void **)&hd, h, 0));
    hipStream_t s = ctx->s_aux;
    ss_cosine_part *dpart = (ss_cosine_part *)(hd + ho_part);
    // Short sequences: one workgroup if the keys' maps fit its LDS, which only it can tell, unless they didn't in one of the last
    // calls.  Three launches | one: 4 anchors of 60 operators 20.2 | 15.8 us, of 2,048 21.8 | 21.1; 1,024 of 60 27.8 | 19.0, of 2,048
    // 26.5 | 25.6; 2,048 of 2,048 33.1 | 30.8.  From there on three passes over the chip are the faster.
    if (mapped && search && !hist && n && m && n <= kShortOps && m <= kShortOps && k <= kShortAnchors) {
      const uint32_t most_keys = short_keys(n, m, k);
      if (ctx->match_many_keys) {
        ctx->match_many_keys--;
      } else if (n > 2 * ctx->match_few_ops && more_keys(ref, n, most_keys)) {
        ctx->match_many_keys = kTryAgain;
      } else {
        std::memcpy(h + ho_ref, ref, (size_t)n * op_bytes);
        std::memcpy(h + ho_cur, cur, (size_t)m * op_bytes);
        std::memcpy(h + ho_anc, anchors, (size_t)k * sizeof(ss_anchor_t));
        volatile uint32_t *const said = (volatile uint32_t *)(h + ho_lost);
        said[1] = 0;
        ss_done told = ss_next_done(ctx);
        told.wgs = 1;
        const ShortArgs a = {(const ss_op_t *)(hd + ho_ref), (const ss_op_t *)(hd + ho_cur), (const ss_anchor_t *)(hd + ho_anc), n, m, k,
                             most_keys, (int32_t *)(hd + ho_idx), hd + ho_level, (uint32_t *)(hd + ho_lost), (uint32_t *)(hd + ho_lost) + 1, dpart, told};
        hipLaunchKernelGGL(ss_match_short_kernel, dim3(1), dim3(kShortThreads), sizeof(ShortLds), s, a);
        SS_HIP(hipGetLastError());
        if ((rc = ss_wait_done(ctx, told)) != SS_OK) return rc;
        ctx->match_few_ops = said[1] ? 0 : n;
        if (!said[1]) {
          const ss_cosine_part &sums = *(const ss_cosine_part *)(h + ho_part);
          if (sums.bad) return SS_E_INVAL;                   // a token beyond 2^18
          std::memcpy(new_idx, h + ho_idx, (size_t)k * 4);
          std::memcpy(level, h + ho_level, k);
          const uint64_t sm[3] = {sums.dot, sums.na, sums.nb};
          finish(sm, said[0]);
          return SS_OK;
        }
        ctx->match_many_keys = kTryAgain;
      }
    }
    PrepArgs p = {};
    bool split = false;
    p.n = n; p.m = m; p.k = search ? k : 0;
    p.cosine = !hist;
    p.ones = (uint4 *)(d + o_ones);
    p.n_ones = (uint32_t)((ones_end - o_ones) / 16);
    p.zeros = (uint4 *)(d + o_hist);
    p.n_zeros = (uint32_t)((zeros_end - o_hist) / 16);
    p.part = dpart;
    // the call's last kernel tells the host, unless copies follow it
    ss_done done = search && !mapped ? ss_done{} : ss_next_done(ctx);
    auto launch_prep = [&](const PrepArgs &a) -> uint32_t {
      const uint32_t longest = std::max(a.n, a.m), clears = std::max(a.n_ones, a.n_zeros);
      const uint32_t for_ops = std::min(256u, std::max(1u, (longest + 255) / 256));
      const uint32_t grid = std::max(for_ops, std::min(kMaxParts, clears / 2048));
      PrepArgs x = a;
      if (x.done.flag) x.done.wgs = grid;
      if (mapped && longest > kTogetherMapped) hipLaunchKernelGGL(ss_prep_kernel<false>, dim3(grid), dim3(256), 0, s, x);
      else hipLaunchKernelGGL(ss_prep_kernel<true>, dim3(grid), dim3(256), 0, s, x);
      return grid;
    };
    if (mapped) {
      if (n) std::memcpy(h + ho_ref, ref, (size_t)n * op_bytes);
      if (k) std::memcpy(h + ho_anc, anchors, (size_t)k * sizeof(ss_anchor_t));
      if (!hist && (size_t)std::min(n, m) * op_bytes >= kSplitBytes) {
        PrepArgs q = p;                                      // the reference comes while the host copies the other sequence
        q.ref = (const ss_op_t *)(hd + ho_ref); q.dref = (ss_op_t *)(d + o_ref);
        q.anchors = (const ss_anchor_t *)(hd + ho_anc);
        if (search) q.danc = (ss_anchor_t *)(d + o_anc);
        q.m = q.cosine = 0;
        launch_prep(q);
        SS_HIP(hipGetLastError());
        p.k = p.n_ones = p.n_zeros = 0;
        split = true;
      }
      if (m) std::memcpy(h + ho_cur, cur, (size_t)m * op_bytes);
      p.ref = (const ss_op_t *)(hd + ho_ref); p.dref = (ss_op_t *)(d + o_ref);
      p.cur = (const ss_op_t *)(hd + ho_cur); p.dcur = (ss_op_t *)(d + o_cur);
      p.anchors = (const ss_anchor_t *)(hd + ho_anc);
      if (search && !split) p.danc = (ss_anchor_t *)(d + o_anc);
      if (split) { p.ref = (const ss_op_t *)(d + o_ref); p.dref = nullptr; }
    } else {
      if (n) SS_HIP(hipMemcpyAsync(d + o_ref, ref, (size_t)n * op_bytes, hipMemcpyHostToDevice, s));
      if (m) SS_HIP(hipMemcpyAsync(d + o_cur, cur, (size_t)m * op_bytes, hipMemcpyHostToDevice, s));
      if (k) SS_HIP(hipMemcpyAsync(d + o_anc, anchors, (size_t)k * sizeof(ss_anchor_t), hipMemcpyHostToDevice, s));
      p.ref = (const ss_op_t *)(d + o_ref);
      p.cur = (const ss_op_t *)(d + o_cur);
      if (hist) p.n = p.m = 0;                               // nothing to read them for
    }
    ss_told_by(done, search ? out_wgs : 256);                // launch_prep sets its own
    if (!search && !hist) p.done = done;
    const uint32_t prep_wgs = launch_prep(p), parts = hist ? 256 : prep_wgs;
    const ss_op_t *dref = (const ss_op_t *)(d + o_ref), *dcur = (const ss_op_t *)(d + o_cur);
    if (hist) {
      uint32_t *h_ref = (uint32_t *)(d + o_hist), *h_cur = h_ref + kTokenLimit, *bad = h_cur + kTokenLimit;
      hipLaunchKernelGGL(ss_histogram_kernel, dim3(wgs), dim3(256), 0, s, dref, n, dcur, m, h_ref, h_cur, bad);
      hipLaunchKernelGGL(ss_histdot_kernel, dim3(256), dim3(256), 0, s, h_ref, h_cur, kTokenLimit, bad, dpart,
                         search ? ss_done{} : done);
    }
    SS_HIP(hipGetLastError());
    if (search) {
      AnchorArgs g = {dref, dcur, (const ss_anchor_t *)(d + o_anc), n, m, k, (int32_t *)(d + o_land), d + o_lvl,
                      (uint32_t *)(d + o_slot),
                      {(unsigned long long *)(d + o_ones), (uint32_t *)(d + o_owner), (uint32_t)(slots - 1), 64u - bits}};
      if (listed) {
        KeyTable q = {};
        for (int L = 0; L < 3; ++L) {
          q.rep[L] = (uint32_t *)(d + o_rep[L]);
          q.key[L] = (uint4 *)(d + o_key[L]);
          for (int x = 0; x < 2; ++x) q.info[x][L] = (uint32_t *)(d + o_info[x][L]);
        }
        for (int x = 0; x < 2; ++x) {
          q.chunk_bits[x] = chunk_bits[x];
          q.chunks[x] = chunks[x];
          q.count[x] = (uint32_t *)(d + o_count[x]);
        }
        q.n_used = (uint32_t *)(d + o_n_used);
        q.mask = (uint32_t)(key_slots - 1);
        q.shift = 64u - key_bits;
        q.probes = key_bits < bits ? kProbes : (uint32_t)key_slots;        // else every key has a place
        q.max_keys = max_keys;
        hipLaunchKernelGGL(ss_keys_kernel, dim3((k + 255) / 256, 3), dim3(256), 0, s, g, q);
        if (chunks[0] + chunks[1])
          hipLaunchKernelGGL(ss_chunks_kernel, dim3(chunks[0] + chunks[1], 3), dim3(kChunkThreads), 0, s, g, q);
        const uint32_t per = k <= kOneEach ? 1 : 4;
        hipLaunchKernelGGL(ss_lookup_kernel, dim3((k + per - 1) / per), dim3(256), 0, s, g, q, per);
      } else {
        if (k >= kAloneAnchors && k >= 2 * (n + m)) hipLaunchKernelGGL(ss_anchor_short_kernel, dim3((k + 3) / 4), dim3(256), 0, s, g);
        else hipLaunchKernelGGL(ss_anchor_kernel, dim3(k), dim3(256), 0, s, g);
      }
      hipLaunchKernelGGL(ss_injective_kernel, dim3(out_wgs), dim3(256), 0, s, g,
                         (int32_t *)(mapped ? hd + ho_idx : d + o_idx), mapped ? hd + ho_level : d + o_level,
                         (uint32_t *)(hd + ho_lost), done);
      SS_HIP(hipGetLastError());
      if (!mapped) {
        SS_HIP(hipMemcpyAsync(new_idx, d + o_idx, (size_t)k * 4, hipMemcpyDeviceToHost, s));
        SS_HIP(hipMemcpyAsync(level, d + o_level, k, hipMemcpyDeviceToHost, s));
      }
    }
    if (!done.flag) SS_HIP(hipStreamSynchronize(s));
    else if ((rc = ss_wait_done(ctx, done)) != SS_OK) return rc;
    uint64_t sm[3] = {0, 0, 0}, too_large = 0;
    const ss_cosine_part *part = (const ss_cosine_part *)(h + ho_part);
    for (uint32_t w = 0; w < parts; ++w) {
      sm[0] += part[w].dot;
      sm[1] += part[w].na;
      sm[2] += part[w].nb;
      too_large |= part[w].bad;
    }
    if (too_large) return SS_E_INVAL;                        // a token beyond 2^18
    uint32_t n_unm = 0;
    if (search) {
      if (mapped) {
        std::memcpy(new_idx, h + ho_idx, (size_t)k * 4);
        std::memcpy(level, h + ho_level, k);
      }
      for (uint32_t w = 0; w < out_wgs; ++w) n_unm += ((const uint32_t *)(h + ho_lost))[w];
    }
    if (k && aligned) {                                      // the scratch is free again
      std::vector<int32_t> ref_to_cur(n);
      uint32_t lcs = 0;
      rc = ss_align_core(ctx, ref, n, cur, m, ref_to_cur.data(), &lcs, nullptr);
      if (rc != SS_OK) return rc;
      ss_align_anchors(ref, n, cur, ref_to_cur.data(), anchors, k, new_idx, level, &n_unm);
    }
    finish(sm, n_unm);
    return SS_OK;
  });
}
