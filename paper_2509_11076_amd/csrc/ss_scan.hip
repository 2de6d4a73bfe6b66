// Memory-timeline scan on the GPU (Sec. 3 last paragraph and Sec. 4.2 of the SmartSwap
// paper): from the alloc/free trace of an iteration, plus the releases and allocations a
// swap policy induces, compute the memory in use at every operator, its peak, and the
// memory reduction entries (excess over the budget per operator).
//
// Event lists come in operator order, so everything follows from running sums along each list: the sums of the
// positive and of the negative deltas and the count of the positive ones, taken at the first event of every
// operator (OpAt).  With P and N these sums over both lists at operator t, the memory of t is
//     base + P[t + 1] + N[t],
// and an event's place and total in the canonical order are its own list's running values plus differences of
// OpAt entries at t and t + 1.  No accumulator is cleared and nothing is added atomically.
//
// Short traces: one workgroup keeps the events in registers and the OpAt table in LDS, one launch.  Long ones: two
// launches over tiles of events (running sums and OpAt; operators and timeline).  A list that
// turns out not to be in operator order is gathered per operator with 64-bit integer atomics instead
// (order-independent, hence deterministic); it has no timeline.  So are the longer ones of a batch, one workgroup a scan,
// in any order.
//
// Bound by latency: barriers and dependent loads in a short trace (124 + 24 events, 66 operators: 4.3 us in one
// workgroup; with sums gathered by atomics, fences and running values in device memory 31 us), launches and one pass
// each over the events in a long one (100,000 + 40,000 events with a timeline: 7.6 + 4.6 us; with operators
// and timeline left to one workgroup 1,084 us; 1,048,574 + 20,014 events, 65,536 operators: 44 us, was 221).
#include <algorithm>
#include <cstring>
#include <mutex>

#include "ss_internal.h"

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

// running values of one list before the first event of an operator
struct OpAt { int64_t sp, sn; uint32_t f, cp; };       // sums of positive / negative deltas, events, positive events
struct TileSum { int64_t sp, sn; uint32_t cp, flags; };
struct Best { int64_t val; uint32_t idx, over; };

constexpr uint64_t kMaxTiles = 1024;       // per list: a workgroup reads the sums of all tiles before its own
constexpr uint32_t kMaxOpWgs = 256;

// What the workgroups of a long trace tell each other.  A tile's sums are five words and a maximum is four, each with the
// number of the scan in its upper half, so that a reader knows each word by itself for this scan's and neither side needs a
// fence.  `scan` is the last one's number (the second launch sets it); nothing is ever cleared, and what an earlier
// scan left is not taken for this one's.  Words that no scan has written hold number 0, which none has.
struct TileBoard {
  uint32_t scan;
  uint32_t done;              // workgroups of the second launch that have ended; the first sets it to 0
  uint64_t tile[5][2 * kMaxTiles + 2];
  uint64_t best[4][kMaxOpWgs];
};

struct ScanArgs {
  const ss_event_t *ev;    uint64_t n_ev;
  const ss_event_t *pev;   uint64_t n_pe;
  uint32_t n_ops;          int want_timeline;
  int64_t base, budget;
  // scratch (device memory; a short trace needs none)
  OpAt *at;           // [2][n_ops + 1]
  int64_t *pos, *net; // [n_ops] per-operator sums of a list out of order
  int64_t *sumx;      // [n_ev + n_pe] inclusive running sum of the event's own class in its list
  uint32_t *cntx;     // [n_ev + n_pe] events of its own class before it in its list
  TileBoard *board;
  uint32_t wait_ticks;
  uint32_t tile[2];   // events per tile of ev, of pev
  uint32_t tiles0, tiles1;
  // the first launch reads the events from here, if given, and copies them to ev / pev for the second (without the tensor
  // ids, which no kernel looks at)
  const ss_event_t *src_ev, *src_pev;
  // outputs
  int64_t *per_op, *mre, *timeline;
  ss_done done;             // host calls
  ss_scan_result_t *res;    // the flags go to res->reserved (bit 0: an event names an operator >= n_ops, nothing
                            // else is meaningful; bit 1: a list is not in operator order)
};

// ---- wavefront and workgroup sums -------------------------------------------------------------------------------

// v of another lane by one data-parallel move, 0 where there is none
template <int kCtrl, int kRows>
__device__ __forceinline__ int64_t dpp_i64(int64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(uint64_t)v, kCtrl, kRows, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)((uint64_t)v >> 32), kCtrl, kRows, 0xF, false);
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// inclusive prefix sum over the 64 lanes: within rows of 16, then the rows' last lanes handed on
__device__ __forceinline__ int64_t wave_scan(int64_t v) {
  v += dpp_i64<0x111, 0xF>(v);
  v += dpp_i64<0x112, 0xF>(v);
  v += dpp_i64<0x114, 0xF>(v);
  v += dpp_i64<0x118, 0xF>(v);
  v += dpp_i64<0x142, 0xA>(v);
  v += dpp_i64<0x143, 0xC>(v);
  return v;
}

__device__ __forceinline__ int64_t lane_i64(int64_t v, int lane) {
  return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)((uint64_t)v >> 32), lane) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, lane));
}

// operator of the event before lane 0's, else of the lane before
__device__ __forceinline__ uint32_t prev_lane(uint32_t v, uint32_t before) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)before, (int)v, 0x138, 0xF, 0xF, false);
}

__device__ inline void add_i64(int64_t *p, int64_t v) {
  atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}

__device__ __forceinline__ void better(Best &a, const Best &b) {
  if (b.val > a.val || (b.val == a.val && b.idx < a.idx)) { a.val = b.val; a.idx = b.idx; }
  a.over += b.over;
}

constexpr uint32_t kNoOp = 0xFFFFFFFFu;

__device__ __forceinline__ Best no_best() { return Best{INT64_MIN, kNoOp, 0}; }

template <int kCtrl, int kRows>
__device__ __forceinline__ int64_t max_step(int64_t v) {
  const uint32_t lo = dpp_u32<kCtrl, kRows>((uint32_t)(uint64_t)v, 0), hi = dpp_u32<kCtrl, kRows>((uint32_t)((uint64_t)v >> 32), 0x80000000u);
  const int64_t o = (int64_t)((uint64_t)hi << 32 | lo);
  return o > v ? o : v;
}

template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t min_step(uint32_t v) { return min(v, dpp_u32<kCtrl, kRows>(v, ~0u)); }

// over the wavefront, given in every lane: the largest value, its lowest index, the sum of `over`
__device__ __forceinline__ Best wave_best(Best b) {
  int64_t v = b.val;
  v = max_step<0x111, 0xF>(v);
  v = max_step<0x112, 0xF>(v);
  v = max_step<0x114, 0xF>(v);
  v = max_step<0x118, 0xF>(v);
  v = max_step<0x142, 0xA>(v);
  v = max_step<0x143, 0xC>(v);
  v = lane_i64(v, 63);
  uint32_t i = b.val == v ? b.idx : ~0u;
  i = min_step<0x111, 0xF>(i);
  i = min_step<0x112, 0xF>(i);
  i = min_step<0x114, 0xF>(i);
  i = min_step<0x118, 0xF>(i);
  i = min_step<0x142, 0xA>(i);
  i = min_step<0x143, 0xC>(i);
  return Best{v, (uint32_t)__builtin_amdgcn_readlane((int)i, 63), (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_u32(b.over), 63)};
}

__device__ __forceinline__ void write_result(const ScanArgs &a, const Best &b, int64_t final_total, uint32_t flags) {
  ss_scan_result_t r;
  if (flags & 1u) {
    r = ss_scan_result_t{a.base, a.base, -1, 0, 0, flags};
  } else {
    r.peak = a.n_ops ? b.val : a.base;
    r.final_total = final_total;
    r.argpeak_op = a.n_ops ? (int32_t)b.idx : -1;
    r.n_over = b.over;
    r.sorted = (flags & 2u) ? 0u : 1u;
    r.reserved = flags;
  }
  *a.res = r;
}

// memory at operator t; writes the per-operator outputs
__device__ __forceinline__ void put_op(const ScanArgs &a, uint32_t t, int64_t p, Best &b) {
  if (a.per_op) a.per_op[t] = p;
  const int64_t ex = p > a.budget ? p - a.budget : 0;
  if (a.mre) a.mre[t] = ex;
  better(b, Best{p, t, ex > 0 ? 1u : 0u});
}

// canonical place and total of an event: class 0 policy alloc, 1 trace alloc, 2 trace release, 3 policy release.
// sum: inclusive running sum of its class in its list, cnt: events of its class before it there
__device__ __forceinline__ void put_event(const ScanArgs &a, int64_t *timeline, bool policy, bool positive, int64_t sum, uint32_t cnt,
                                          const OpAt &e0, const OpAt &e1, const OpAt &p0, const OpAt &p1) {
  uint32_t q = e0.f + p0.f;                        // events of earlier operators
  int64_t v;
  const uint32_t n0 = p1.cp - p0.cp, n1 = e1.cp - e0.cp;
  if (policy && positive) {
    q += cnt - p0.cp;
    v = e0.sp + e0.sn + p0.sn + sum;
  } else if (positive) {
    q += n0 + cnt - e0.cp;
    v = e0.sn + p0.sn + p1.sp + sum;
  } else if (!policy) {
    q += n0 + n1 + cnt - (e0.f - e0.cp);
    v = p0.sn + p1.sp + e1.sp + sum;
  } else {
    q += n0 + (e1.f - e0.f) + cnt - (p0.f - p0.cp);
    v = e1.sn + e1.sp + p1.sp + sum;
  }
  timeline[q] = a.base + v;
}

// OpAt entries of operators (prev, op] take the values before the event that starts op.  A lane fills a short gap by
// itself; the wavefront fills a long one (more than kAlone operators) together, 64 entries a turn of about 0.1 us (one gap of
// 65,536 operators 0.1 ms; tiles of few events do it with the whole workgroup, fill_together).  A workgroup that
// does the whole scan has few long gaps in a wavefront: 4.  A tile may have many: 16 (the running sums of 20,014 events
// over 65,536 operators 30 us, with 4 37).
template <uint32_t kAlone>
__device__ __forceinline__ void fill_gap(OpAt *at, bool has, uint32_t from, uint32_t to, const OpAt &x) {
  const uint32_t len = has ? to - from : 0;
  if (len && len <= kAlone)
    for (uint32_t t = from; t < to; ++t) at[t] = x;
  uint64_t wide = __ballot(len > kAlone);
  const uint32_t lane = threadIdx.x & 63;
  while (wide) {
    const int src = __builtin_ctzll(wide);
    wide &= wide - 1;
    OpAt y;
    y.sp = lane_i64(x.sp, src);
    y.sn = lane_i64(x.sn, src);
    y.f = (uint32_t)__builtin_amdgcn_readlane((int)x.f, src);
    y.cp = (uint32_t)__builtin_amdgcn_readlane((int)x.cp, src);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)from, src), hi = (uint32_t)__builtin_amdgcn_readlane((int)to, src);
    for (uint32_t t = lo + lane; t < hi; t += 64) at[t] = y;
  }
}

// ---- running sums over a stretch of elements ---------------------------------------------------------------------

// Totals of the wavefronts' stretches, then what comes before each, and the totals after them.
struct SumShared {
  int64_t sp[64], sn[64], tot_sp, tot_sn;
  uint32_t cp[64], tot_cp;
};

// T * K consecutive elements, K per thread, element k * T + thread; dead ones have delta 0 and pos false.  Out: the sums
// of the positive and of the negative deltas and the count of the positive events before each element, carries
// included.  One barrier after the totals are written and one after they are summed; the caller puts one between calls.
template <int T, int K>
__device__ __forceinline__ void wg_sums(SumShared &sh, const int64_t *delta, const bool *pos, int64_t carry_sp,
                                        int64_t carry_sn, uint32_t carry_cp, int64_t *xsp, int64_t *xsn, uint32_t *xcp) {
  constexpr int W = T / 64, S = W * K;
  static_assert(S <= 64, "the stretches' totals are summed by one wavefront");
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t p = pos[k] ? delta[k] : 0, q = delta[k] - p;
    const int64_t ip = wave_scan(p), iq = wave_scan(q);
    const uint64_t b = __ballot(pos[k]);
    xsp[k] = ip - p;
    xsn[k] = iq - q;
    xcp[k] = (uint32_t)__popcll(b & below);
    if (lane == 63) {
      sh.sp[k * W + w] = ip;
      sh.sn[k * W + w] = iq;
      sh.cp[k * W + w] = (uint32_t)__popcll(b);
    }
  }
  __syncthreads();
  if (w == 0) {
    const int64_t p = lane < S ? sh.sp[lane] : 0, q = lane < S ? sh.sn[lane] : 0, c = lane < S ? sh.cp[lane] : 0;
    const int64_t ip = wave_scan(p), iq = wave_scan(q), ic = wave_scan(c);
    if (lane < S) {
      sh.sp[lane] = carry_sp + ip - p;
      sh.sn[lane] = carry_sn + iq - q;
      sh.cp[lane] = carry_cp + (uint32_t)(ic - c);
    }
    if (lane == 63) {
      sh.tot_sp = carry_sp + ip;
      sh.tot_sn = carry_sn + iq;
      sh.tot_cp = carry_cp + (uint32_t)ic;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    xsp[k] += sh.sp[k * W + w];
    xsn[k] += sh.sn[k * W + w];
    xcp[k] += sh.cp[k * W + w];
  }
}

// An event as a lane holds it: `prev` is the operator of the event before it in its list (its own for the first).
struct Elem {
  uint32_t op, prev;
  int64_t delta;
  bool live, pos, first, last;
};

// Elements first .. first + T * K of one list, or (both) of the two lists back to back, all loads in flight at once;
// returns the flags.
template <int T, int K>
__device__ __forceinline__ uint32_t load_events(const ss_event_t *L0, uint64_t n0, const ss_event_t *L1, uint64_t n1,
                                                uint64_t first, uint64_t end, uint32_t n_ops, Elem *x) {
  ss_event_t raw[K];
  uint32_t before[K], flags = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t i = first + (uint64_t)k * T + threadIdx.x;
    x[k].live = i < end;
    const bool second = i >= n0;
    const ss_event_t *L = second ? L1 : L0;
    const uint64_t e = second ? i - n0 : i;
    raw[k] = ss_event_t{kNoOp, 0, 0};
    before[k] = kNoOp;
    x[k].first = e == 0;
    x[k].last = e + 1 == (second ? n1 : n0);
    if (x[k].live) {
      raw[k] = L[e];
      if ((threadIdx.x & 63) == 0 && e) before[k] = L[e - 1].op_idx;
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    Elem &y = x[k];
    y.op = raw[k].op_idx;
    y.delta = y.live ? raw[k].delta : 0;
    y.pos = y.live && raw[k].delta >= 0;
    y.prev = prev_lane(y.op, before[k]);
    if (y.first) y.prev = y.op;
    y.last = y.last && y.live;
    if (y.live && y.op >= n_ops) flags |= 1u;
    if (y.live && y.prev > y.op) flags |= 2u;
  }
  return flags;
}

// OpAt entries that this element decides: those of the operators after the previous event's up to its own, and after
// the list's last event those up to n_ops.
template <uint32_t kAlone = 4>
__device__ __forceinline__ void fill_from(OpAt *at, const Elem &y, uint32_t e, int64_t sp, int64_t sn, uint32_t cp,
                                          uint32_t n_ops) {
  const bool ok = y.live && y.op < n_ops && y.prev <= y.op;
  fill_gap<kAlone>(at, ok && (y.first || y.prev != y.op), y.first ? 0 : y.prev + 1, y.op + 1, OpAt{sp, sn, e, cp});
  if (__ballot(ok && y.last))
    fill_gap<kAlone>(at, ok && y.last, y.op + 1, n_ops + 1,
             OpAt{sp + (y.pos ? y.delta : 0), sn + (y.pos ? 0 : y.delta), e + 1, cp + (y.pos ? 1 : 0)});
}

// A list out of order: per-operator sums by integer atomics.  Neighbouring events mostly belong to the same operator,
// and 64 lanes adding to one address are served one after the other: so each run of equal operators among a
// wavefront's events is folded first and only its first lane adds.
__device__ __forceinline__ void gather_run(int64_t *pos, int64_t *net, const Elem &y, uint32_t n_ops) {
  const int lane = threadIdx.x & 63;
  const bool live = y.live && y.op < n_ops, head = lane == 0 || y.first || y.prev != y.op;
  const int64_t p = live && y.pos ? y.delta : 0, d = live ? y.delta : 0;
  const int64_t ip = wave_scan(p), id = wave_scan(d);
  const uint64_t heads = __ballot(head);
  const uint64_t above = lane == 63 ? 0 : heads >> (lane + 1);
  const int last = above ? lane + __builtin_ctzll(above) : 63;
  const int64_t ep = (int64_t)(((uint64_t)(uint32_t)__shfl((int)((uint64_t)ip >> 32), last, 64) << 32) |
                               (uint32_t)__shfl((int)(uint32_t)(uint64_t)ip, last, 64));
  const int64_t ed = (int64_t)(((uint64_t)(uint32_t)__shfl((int)((uint64_t)id >> 32), last, 64) << 32) |
                               (uint32_t)__shfl((int)(uint32_t)(uint64_t)id, last, 64));
  if (head && live) {
    const int64_t tp = ep - (ip - p), td = ed - (id - d);
    if (tp) add_i64(pos + y.op, tp);
    if (td) add_i64(net + y.op, td);
  }
}

// Operators from the gathered sums: a chunked prefix scan of one workgroup.  Leaves the total in sh.tot_sp.
template <int T>
__device__ __forceinline__ Best ops_of_sums(const ScanArgs &a, const int64_t *pos, const int64_t *net, SumShared &sh) {
  Best b = no_best();
  int64_t carry = 0;
  for (uint32_t c0 = 0; c0 < a.n_ops; c0 += T) {
    const uint32_t t = c0 + threadIdx.x;
    const int64_t d[1] = {t < a.n_ops ? net[t] : 0};
    const bool all[1] = {true};
    int64_t x[1], none[1];
    uint32_t cnt[1];
    wg_sums<T, 1>(sh, d, all, carry, 0, 0, x, none, cnt);
    if (t < a.n_ops) put_op(a, t, a.base + x[0] + pos[t], b);
    carry = sh.tot_sp;
    __syncthreads();
  }
  if (threadIdx.x == 0) sh.tot_sp = carry;
  return b;
}

// ---- one workgroup: short traces, candidates of a batch ------------------------------------------------------------

struct WgShared {
  SumShared sums;
  int64_t ev_sp, ev_sn;                    // totals of the first list
  uint32_t ev_cp, flags;
  Best best[kWaves];
};

// over the workgroup, given in the first wavefront
template <int T>
__device__ __forceinline__ Best wg_best(Best b, Best *part) {
  b = wave_best(b);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = b;
  __syncthreads();
  if (threadIdx.x >= 64) return no_best();
  return wave_best(threadIdx.x < T / 64 ? part[threadIdx.x] : no_best());
}

// at: 2 * (n_ops + 1) entries; pos, net: n_ops entries, may lie in `at`.  No timeline.
template <int T, int K>
__device__ __forceinline__ void scan_wg(const ScanArgs &a, OpAt *at, int64_t *pos, int64_t *net, WgShared &sh) {
  const uint32_t n = a.n_ops, tid = threadIdx.x;
  OpAt *const at_ev = at, *const at_pe = at + n + 1;
  const uint64_t total = a.n_ev + a.n_pe;
  if (tid == 0) {
    sh.flags = 0;
    sh.ev_sp = sh.ev_sn = 0;
    sh.ev_cp = 0;
  }
  if (!a.n_ev)
    for (uint32_t t = tid; t <= n; t += T) at_ev[t] = OpAt{0, 0, 0, 0};
  if (!a.n_pe)
    for (uint32_t t = tid; t <= n; t += T) at_pe[t] = OpAt{0, 0, 0, 0};
  __syncthreads();
  Elem x[K];
  int64_t delta[K], sp[K], sn[K], carry_sp = 0, carry_sn = 0;
  uint32_t cp[K], carry_cp = 0;
  bool pos_of[K];
  // Running sums where the events take one pass or two.  A list out of order needs none: they end as soon as it shows, and
  // the events are gathered by operator, whatever their order; more events than that (of a batch: it has no timeline) are
  // gathered at once.  (Running sums always, and gathered after them where the order was wrong: six scans of 100,000 + 20
  // events over 400 operators 249 us in order and 343 out of order, gathered at once 212 and 213; of 10,000 + 2,000 over 700
  // 134 and 164 against 133 and 137; of 8,000 + 100, two passes, 67 and 90 against 67 and 76 to 83.)
  const bool in_sums = total <= 2 * (uint64_t)T * K;
  for (uint64_t first = 0; in_sums && first < total; first += (uint64_t)T * K) {
    const uint32_t bad = load_events<T, K>(a.ev, a.n_ev, a.pev, a.n_pe, first, total, n, x);
    if (bad) atomicOr(&sh.flags, bad);
    // A wavefront with events out of order fills nothing: in random order nearly every gap would be a long one (4,000 + 90
    // events over 700 operators 104 us, 24 without; six scans of 20,000 + 2,000 over 65,536 71 ms).  Known without a look at
    // LDS, which would cost an ordered trace 0.3 us.
    const bool tidy = !__ballot(bad != 0);
#pragma unroll
    for (int k = 0; k < K; ++k) { delta[k] = x[k].delta; pos_of[k] = x[k].pos; }
    wg_sums<T, K>(sh.sums, delta, pos_of, carry_sp, carry_sn, carry_cp, sp, sn, cp);
    if (total > (uint64_t)T * K && sh.flags) break;
    carry_sp = sh.sums.tot_sp; carry_sn = sh.sums.tot_sn; carry_cp = sh.sums.tot_cp;
    if (a.n_pe && first + (uint64_t)T * K > a.n_ev) {        // the second list starts from its own zero
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (first + (uint64_t)k * T + tid == a.n_ev) { sh.ev_sp = sp[k]; sh.ev_sn = sn[k]; sh.ev_cp = cp[k]; }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (first + (uint64_t)k * T + tid >= a.n_ev) { sp[k] -= sh.ev_sp; sn[k] -= sh.ev_sn; cp[k] -= sh.ev_cp; }
    }
    // a wavefront's elements of one k may belong to both lists: each list's are filled in turn
#pragma unroll
    for (int k = 0; tidy && k < K; ++k) {
      const uint64_t i = first + (uint64_t)k * T + tid;
      Elem y = x[k];
      y.live = x[k].live && i < a.n_ev;
      y.last = x[k].last && y.live;
      if (__ballot(y.live)) fill_from(at_ev, y, (uint32_t)i, sp[k], sn[k], cp[k], n);
      y.live = x[k].live && i >= a.n_ev;
      y.last = x[k].last && y.live;
      if (__ballot(y.live)) fill_from(at_pe, y, (uint32_t)(i - a.n_ev), sp[k], sn[k], cp[k], n);
    }
    __syncthreads();                                         // the shared totals are written again in the next pass
  }
  __syncthreads();
  uint32_t flags = sh.flags;
  Best b = no_best();
  int64_t final_total = a.base;
  const bool gathered = !in_sums || (flags & 3u) == 2u;
  if (gathered) {
    for (uint32_t t = tid; t < n; t += T) pos[t] = net[t] = 0;
    __threadfence();
    __syncthreads();
    for (uint64_t first = 0; first < total; first += (uint64_t)T * K) {
      const uint32_t bad = load_events<T, K>(a.ev, a.n_ev, a.pev, a.n_pe, first, total, n, x);
      if (bad) atomicOr(&sh.flags, bad);
#pragma unroll
      for (int k = 0; k < K; ++k) gather_run(pos, net, x[k], n);
    }
    __threadfence();
    __syncthreads();
    flags = sh.flags;
  }
  if (flags & 1u) {
    if (tid == 0) write_result(a, b, 0, flags);
    return;
  }
  if (gathered) {
    b = ops_of_sums<T>(a, pos, net, sh.sums);
    __syncthreads();
    final_total += n ? sh.sums.tot_sp : 0;
  } else {
    for (uint32_t t = tid; t < n; t += T)
      put_op(a, t, a.base + at_ev[t + 1].sp + at_pe[t + 1].sp + at_ev[t].sn + at_pe[t].sn, b);
    final_total += at_ev[n].sp + at_ev[n].sn + at_pe[n].sp + at_pe[n].sn;
  }
  b = wg_best<T>(b, sh.best);
  if (tid == 0) write_result(a, b, final_total, flags);
}

// ---- one workgroup, short traces -------------------------------------------------------------------------------------
//
// The events lie in registers, K consecutive ones to a lane, each list from a wavefront's first lane on, so that a
// wavefront adds up a list's running sums with one prefix sum of each kind (a wavefront issues an instruction in some five
// cycles, and with the events dealt out lane by lane and a prefix sum for every 64 the sums took 1.3 us for 148 events
// and 3 for 1,734).  An operator's OpAt entry is written by the event that starts it; those of operators without events
// are copied from the next operator that has some, found in a bit map (each gap filled by the wavefront that met it: 1.6
// and 2.5 us, 7 with 90 events over 700 operators).  The timeline is put together in LDS, so that it leaves in whole lines.
// 124 + 24 events over 66 operators: 3.9 us, before 6.0; 1,398 + 336 over 700 from and to pinned memory 9.4, before 12.1.

constexpr uint32_t kLdsOps = 2900;                       // OpAt tables of more don't fit LDS
constexpr uint32_t kHeadWords = (kLdsOps + 1 + 31) / 32;
constexpr uint64_t kSmallEvents = 4096;
constexpr size_t kShortLds = 150 * 1024;

template <int T>
struct ShortShared {
  int64_t sp[T / 64], sn[T / 64];
  uint32_t cp[T / 64], flags;
  uint32_t head[2][kHeadWords];                          // operators whose entry an event has written
  Best best[T / 64];
  SumShared sums;                                        // lists out of order
};

static __host__ __device__ constexpr uint32_t round_up(uint32_t x, uint32_t to) { return (x + to - 1) / to * to; }

// LDS beyond ShortShared: the events on their way to their lanes, then the OpAt tables (or the sums of lists out of order);
// the timeline
static size_t short_tables(int T, int K, uint32_t n_ops) {
  return ss_align_up(std::max((size_t)T * K * 12, 2 * ((size_t)n_ops + 1) * sizeof(OpAt)), 16);
}

static size_t short_lds(int T, int K, uint32_t n_ops, uint64_t events, bool timeline) {
  return short_tables(T, K, n_ops) + (timeline ? events * 8 : 0);
}

template <int T, int K>
__device__ __forceinline__ void scan_short(const ScanArgs &a, uint8_t *lds, uint32_t tl_at, ShortShared<T> &sh) {
  constexpr uint32_t W = T / 64, kChunk = 64 * K;
  const uint32_t n = a.n_ops, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t w1 = round_up((uint32_t)a.n_ev, kChunk) / kChunk;     // the second list's first wavefront
  const bool policy = w >= w1;
  const ss_event_t *const L = policy ? a.pev : a.ev;
  const uint32_t cnt = (uint32_t)(policy ? a.n_pe : a.n_ev), c0 = (policy ? w - w1 : w) * kChunk;
  OpAt *const tables = reinterpret_cast<OpAt *>(lds), *const at = tables + (policy ? n + 1 : 0);
  const OpAt *const at_ev = tables, *const at_pe = tables + n + 1;
  int64_t *const tl = reinterpret_cast<int64_t *>(lds + tl_at);
  uint32_t op[K];
  int64_t delta[K];
  uint32_t before = kNoOp;                               // operator of the event before the wavefront's first
  {
    ss_event_t raw[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t e = c0 + k * 64 + lane;
      raw[k] = ss_event_t{kNoOp, 0, 0};
      if (e < cnt) raw[k] = L[e];
    }
    if (lane == 0 && c0 && c0 < cnt) before = L[c0 - 1].op_idx;
    for (uint32_t i = tid; i < 2 * kHeadWords; i += T) sh.head[0][i] = 0;
    if (tid == 0) sh.flags = 0;
    if constexpr (K == 1) {
      op[0] = raw[0].op_idx;
      delta[0] = raw[0].delta;
    } else {
      int64_t *const mine = reinterpret_cast<int64_t *>(lds) + w * kChunk;
      uint32_t *const mine_op = reinterpret_cast<uint32_t *>(lds + (size_t)T * K * 8) + w * kChunk;
#pragma unroll
      for (int k = 0; k < K; ++k) { mine[k * 64 + lane] = raw[k].delta; mine_op[k * 64 + lane] = raw[k].op_idx; }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");           // LDS accesses of a wavefront are in order
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int k = 0; k < K; ++k) { delta[k] = mine[lane * K + k]; op[k] = mine_op[lane * K + k]; }
    }
  }
  const uint32_t e0 = c0 + lane * K;
  int64_t sp[K], sn[K], tsp = 0, tsn = 0;                // before the event; of the lane
  uint32_t cp[K], tcp = 0, flags = 0;
  bool pos[K], starts[K];
  uint32_t prev = prev_lane(op[K - 1], before);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const bool live = e0 + k < cnt;
    pos[k] = live && delta[k] >= 0;
    starts[k] = live && (e0 + k == 0 || prev != op[k]);
    if (live && op[k] >= n) flags |= 1u;
    if (live && e0 + k && prev > op[k]) flags |= 2u;
    prev = op[k];
    sp[k] = tsp; sn[k] = tsn; cp[k] = tcp;
    tsp += pos[k] ? delta[k] : 0;
    tsn += pos[k] ? 0 : delta[k];
    tcp += pos[k];
  }
  const int64_t isp = wave_scan(tsp), isn = wave_scan(tsn);
  const uint32_t icp = wave_scan_u32(tcp);
  if (lane == 63) { sh.sp[w] = isp; sh.sn[w] = isn; sh.cp[w] = icp; }
  __syncthreads();
  const uint64_t wrong = __ballot(flags != 0);
  if (wrong) {
    flags = (__ballot(flags & 1u) ? 1u : 0u) | (__ballot(flags & 2u) ? 2u : 0u);
    if (lane == 0) atomicOr(&sh.flags, flags);
  }
  {
    // what the wavefronts of the same list before this one add up to
    const bool counts = lane < w && lane >= (policy ? w1 : 0);
    const int64_t x = wave_scan(counts ? sh.sp[lane % W] : 0), y = wave_scan(counts ? sh.sn[lane % W] : 0);
    const uint32_t z = wave_scan_u32(counts ? sh.cp[lane % W] : 0);
    const int64_t bsp = lane_i64(x, 63) + isp - tsp, bsn = lane_i64(y, 63) + isn - tsn;
    const uint32_t bcp = (uint32_t)__builtin_amdgcn_readlane((int)z, 63) + icp - tcp;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      sp[k] += bsp; sn[k] += bsn; cp[k] += bcp;
      if (starts[k] && op[k] < n) {
        at[op[k]] = OpAt{sp[k], sn[k], e0 + k, cp[k]};
        atomicOr(&sh.head[policy][op[k] / 32], 1u << (op[k] % 32));
      }
      if (e0 + k + 1 == cnt) {
        at[n] = OpAt{sp[k] + (pos[k] ? delta[k] : 0), sn[k] + (pos[k] ? 0 : delta[k]), cnt, cp[k] + (pos[k] ? 1 : 0)};
        atomicOr(&sh.head[policy][n / 32], 1u << (n % 32));
      }
    }
  }
  if (tid < 2 && !(tid ? a.n_pe : a.n_ev)) {             // an empty list
    tables[tid * (n + 1) + n] = OpAt{0, 0, 0, 0};
    atomicOr(&sh.head[tid][n / 32], 1u << (n % 32));
  }
  __syncthreads();
  flags = sh.flags;
  Best b = no_best();
  int64_t final_total = a.base;
  if (flags & 1u) {
    if (tid == 0) write_result(a, b, 0, flags);
    return;
  }
  if (flags) {
    int64_t *const gpos = reinterpret_cast<int64_t *>(lds), *const gnet = gpos + n;
    const uint64_t total = a.n_ev + a.n_pe;
    for (uint32_t t = tid; t < n; t += T) gpos[t] = gnet[t] = 0;
    __syncthreads();
    for (uint64_t first = 0; first < total; first += (uint64_t)T * K) {
      Elem x[K];
      load_events<T, K>(a.ev, a.n_ev, a.pev, a.n_pe, first, total, n, x);
#pragma unroll
      for (int k = 0; k < K; ++k) gather_run(gpos, gnet, x[k], n);
    }
    __syncthreads();
    b = ops_of_sums<T>(a, gpos, gnet, sh.sums);
    __syncthreads();
    final_total += n ? sh.sums.tot_sp : 0;
  } else {
    // the words of a map that hold a bit, for where a search leaves its word (words looked through one by one: 1,000 events
    // of the trace and none of the policy over 2,900 operators 37 us, so 9.7)
    static_assert(kHeadWords <= 128, "two masks a map");
    uint64_t some[2][2];
#pragma unroll
    for (int l = 0; l < 2; ++l)
#pragma unroll
      for (uint32_t h = 0; h < 2; ++h) some[l][h] = __ballot(h * 64 + lane < kHeadWords && sh.head[l][min(h * 64 + lane, kHeadWords - 1)]);
    for (uint32_t i = tid; i < 2 * n; i += T) {
      const uint32_t l = i >= n, t = i - (l ? n : 0);
      uint32_t word = t / 32, bits = sh.head[l][word] >> (t % 32);
      if (bits & 1u) continue;
      uint32_t next = t;
      if (!bits) {                                       // the entry of n is always there
        const uint64_t lo = l ? some[1][0] : some[0][0], hi = l ? some[1][1] : some[0][1];
        ++word;
        const uint64_t here = word < 64 ? lo >> word : 0;
        if (here) {
          word += (uint32_t)__builtin_ctzll(here);
        } else {
          word = max(word, 64u);
          word += (uint32_t)__builtin_ctzll(hi >> (word - 64));
        }
        bits = sh.head[l][word];
        next = word * 32;
      }
      next += (uint32_t)__builtin_ctz(bits);
      tables[l * (n + 1) + t] = tables[l * (n + 1) + next];
    }
    __syncthreads();
    for (uint32_t t = tid; t < n; t += T)
      put_op(a, t, a.base + at_ev[t + 1].sp + at_pe[t + 1].sp + at_ev[t].sn + at_pe[t].sn, b);
    final_total += at_ev[n].sp + at_ev[n].sn + at_pe[n].sp + at_pe[n].sn;
    if (a.want_timeline) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (e0 + k < cnt)
          put_event(a, tl, policy, pos[k], (pos[k] ? sp[k] : sn[k]) + delta[k], pos[k] ? cp[k] : e0 + k - cp[k], at_ev[op[k]],
                    at_ev[op[k] + 1], at_pe[op[k]], at_pe[op[k] + 1]);
    }
  }
  b = wg_best<T>(b, sh.best);                            // its barrier is the timeline's too
  if (a.want_timeline && !flags)
    for (uint32_t i = tid; i < (uint32_t)(a.n_ev + a.n_pe); i += T) a.timeline[i] = tl[i];
  if (tid == 0) write_result(a, b, final_total, flags);
}

template <int T, int K>
__global__ __launch_bounds__(T) void ss_scan_short_kernel(ScanArgs a, uint32_t tl_at) {
  __shared__ ShortShared<T> sh;
  extern __shared__ __align__(16) uint8_t short_mem[];
  scan_short<T, K>(a, short_mem, tl_at, sh);
  ss_tell_host(a.done);
}

// candidate policies against the same trace
template <int T, int K>
__global__ __launch_bounds__(T) void ss_scan_short_batch_kernel(const ScanArgs *__restrict__ args) {
  __shared__ ShortShared<T> sh;
  extern __shared__ __align__(16) uint8_t short_mem[];
  const ScanArgs a = args[blockIdx.x];
  scan_short<T, K>(a, short_mem, 0, sh);
  ss_tell_host(a.done);
}

// lanes and events to a lane for two lists of that many
struct ShortForm { int T, K; };

// Where operators outnumber the lanes that the events need by much, filling the gaps is the work, and more lanes do it sooner: 4
// events over 2,900 operators 9.3 us with 1,024 lanes (with 256, which looked through the map word by word, 40).
static ShortForm short_form(uint64_t n_ev, uint64_t n_pe, uint32_t n_ops) {
  auto fits = [&](uint64_t T, uint64_t K) {
    return n_ops <= 4 * T && ss_align_up(n_ev, 64 * K) + ss_align_up(n_pe, 64 * K) <= T * K;
  };
  if (fits(256, 1)) return {256, 1};
  if (fits(256, 4)) return {256, 4};
  if (fits(512, 4)) return {512, 4};
  if (fits(1024, 4)) return {1024, 4};
  return {0, 0};
}

#define SS_SHORT_FORM(f, LAUNCH)                                    \
  do {                                                              \
    if ((f).T == 256 && (f).K == 1) LAUNCH(256, 1);                 \
    else if ((f).T == 256) LAUNCH(256, 4);                          \
    else if ((f).T == 512) LAUNCH(512, 4);                          \
    else LAUNCH(1024, 4);                                           \
  } while (0)

// The OpAt tables of a batch's scans lie in LDS up to this many operators (24 bytes an entry).
static size_t lds_at(uint32_t n_ops) { return 2 * ((size_t)n_ops + 1) * sizeof(OpAt); }

// one workgroup per scan: candidate policies against the same trace in a single launch
template <bool LDS>
__global__ __launch_bounds__(kThreads) void ss_scan_batch_kernel(const ScanArgs *__restrict__ args) {
  __shared__ WgShared sh;
  extern __shared__ OpAt lds[];
  const ScanArgs a = args[blockIdx.x];
  if (LDS) {
    int64_t *const sums = reinterpret_cast<int64_t *>(lds);
    scan_wg<kThreads, 4>(a, lds, sums, sums + a.n_ops, sh);
  } else {
    scan_wg<kThreads, 4>(a, a.at, a.pos, a.net, sh);
  }
  ss_tell_host(a.done);
}

// ---- long traces: two launches over tiles of events -----------------------------------------------------------------

constexpr int kTileThreads = 256;

// the tile of a workgroup: first the tiles of ev, then those of pev (at least one each)
struct Tile {
  bool policy;
  const ss_event_t *L, *src;
  uint64_t cnt, lo, hi, out0;        // events of its list; its events [lo, hi) there; where its list starts in sumx
  uint32_t first, index;             // its list's first tile; its own
  __device__ explicit Tile(const ScanArgs &a) {
    index = blockIdx.x;
    policy = index >= a.tiles0;
    first = policy ? a.tiles0 : 0;
    L = policy ? a.pev : a.ev;
    src = policy ? a.src_pev : a.src_ev;
    cnt = policy ? a.n_pe : a.n_ev;
    out0 = policy ? a.n_ev : 0;
    lo = (uint64_t)(index - first) * a.tile[policy];
    hi = lo + a.tile[policy] < cnt ? lo + a.tile[policy] : cnt;
  }
};

// N words of entry `at`, 32 bits of content each
template <int N, size_t L>
__device__ __forceinline__ void tell(uint64_t (*words)[L], uint32_t at, uint32_t scan, const uint32_t (&x)[N]) {
#pragma unroll
  for (int w = 0; w < N; ++w)
    __hip_atomic_store(&words[w][at], (uint64_t)scan << 32 | x[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// false: not all there yet
template <int N, size_t L>
__device__ __forceinline__ bool hear(const uint64_t (*words)[L], uint32_t at, uint32_t scan, uint32_t (&x)[N]) {
  uint64_t y[N];
#pragma unroll
  for (int w = 0; w < N; ++w) y[w] = __hip_atomic_load(&words[w][at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  bool all = true;
#pragma unroll
  for (int w = 0; w < N; ++w) {
    x[w] = (uint32_t)y[w];
    all &= (uint32_t)(y[w] >> 32) == scan;
  }
  return all;
}

__device__ __forceinline__ int64_t both_halves(uint32_t lo, uint32_t hi) { return (int64_t)((uint64_t)hi << 32 | lo); }
__device__ __forceinline__ uint32_t low_half(int64_t v) { return (uint32_t)(uint64_t)v; }
__device__ __forceinline__ uint32_t high_half(int64_t v) { return (uint32_t)((uint64_t)v >> 32); }

__device__ __forceinline__ void put_tile(TileBoard *b, uint32_t tile, uint32_t scan, const TileSum &s) {
  const uint32_t x[5] = {low_half(s.sp), high_half(s.sp), low_half(s.sn), high_half(s.sn), s.flags << 30 | s.cp};   // cp < 2^22
  tell(b->tile, tile, scan, x);
}

__device__ __forceinline__ bool get_tile(const TileBoard *b, uint32_t tile, uint32_t scan, TileSum &s) {
  uint32_t x[5];
  const bool there = hear(b->tile, tile, scan, x);
  s = TileSum{both_halves(x[0], x[1]), both_halves(x[2], x[3]), x[4] & 0x3FFFFFFFu, x[4] >> 30};
  return there;
}

// sums over the workgroup, given in every thread
__device__ __forceinline__ TileSum wg_total(int64_t sp, int64_t sn, uint32_t cp, uint32_t flags, TileSum *part) {
  sp = lane_i64(wave_scan(sp), 63);
  sn = lane_i64(wave_scan(sn), 63);
  const int64_t c = lane_i64(wave_scan((int64_t)cp), 63);
  flags = (__ballot(flags & 1u) ? 1u : 0u) | (__ballot(flags & 2u) ? 2u : 0u);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = TileSum{sp, sn, (uint32_t)c, flags};
  __syncthreads();
  TileSum s = part[0];
  for (int i = 1; i < kTileThreads / 64; ++i) {
    s.sp += part[i].sp; s.sn += part[i].sn; s.cp += part[i].cp; s.flags |= part[i].flags;
  }
  __syncthreads();                                           // part may be written again
  return s;
}

// Sums over events [lo, hi) of the workgroup's list.
template <int K>
__device__ __forceinline__ TileSum sum_events(const ScanArgs &a, const Tile &tl, uint64_t lo, uint64_t hi, TileSum *part) {
  int64_t sp = 0, sn = 0;
  uint32_t cp = 0, flags = 0;
  for (; lo < hi; lo += (uint64_t)kTileThreads * K) {
    Elem x[K];
    flags |= load_events<kTileThreads, K>(tl.src ? tl.src : tl.L, tl.cnt, nullptr, 0, lo, hi, a.n_ops, x);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      sp += x[k].pos ? x[k].delta : 0;
      sn += x[k].pos ? 0 : x[k].delta;
      cp += x[k].pos;
    }
  }
  return wg_total(sp, sn, cp, flags, part);
}

// Gaps of a tile of few events, each filled by the whole workgroup, 8 bytes a lane side by side: bound by how many stores a workgroup
// has under way.  Both launches of 460 + 28 events over 58,299 operators 21 us, of 2,000 + 4 over 65,536 23; one by one by the first
// wavefront, 64 entries of 24 bytes in 0.1 us (fill_gap), 29 and 56.  Where an event stands for few
// operators on average, but not everywhere, a tile of short gaps loses 0.3 and one with a long gap gains 2 us (both launches, filled each
// by its own and together; evenly spread 1,000 over 9,000: 13.9 and 14.3, 400 over 30,000: 14.5 and 14.8; the policy of 939 tensors that
// live from one half of 29,449 operators into the other, 1,878 events: 21.1 and 18.8).  Up to kLongGaps operators to an event it is as
// fast (7 to one: 16.4 and 14.7; 5 to one: 14.9 and 15.3).
constexpr uint32_t kFewInTile = 8, kLongGaps = 8;

__host__ __device__ inline bool few_in_tile(uint32_t tile, uint64_t events, uint32_t n_ops) {
  return events && tile <= kFewInTile && n_ops > kLongGaps * events;
}

struct FewGaps {
  uint32_t lo[kFewInTile + 1], hi[kFewInTile + 1];           // the last one's: after the list's last event
  OpAt x[kFewInTile + 1];
};

// `e`: the event of this thread, in its tile's order, from thread 0 on
__device__ __forceinline__ void fill_together(OpAt *at, FewGaps &gaps, const Elem &y, uint32_t e, int64_t sp, int64_t sn, uint32_t cp,
                                              uint32_t n_ops) {
  static_assert(sizeof(OpAt) == 24 && kTileThreads % 3 == 1, "whose word a thread's next one is");
  const uint32_t tid = threadIdx.x;
  if (tid <= kFewInTile) gaps.lo[tid] = gaps.hi[tid] = 0;
  __syncthreads();
  if (y.live && y.op < n_ops && y.prev <= y.op) {
    if (y.first || y.prev != y.op) {
      gaps.lo[tid] = y.first ? 0 : y.prev + 1;
      gaps.hi[tid] = y.op + 1;
      gaps.x[tid] = OpAt{sp, sn, e, cp};
    }
    if (y.last) {
      gaps.lo[kFewInTile] = y.op + 1;
      gaps.hi[kFewInTile] = n_ops + 1;
      gaps.x[kFewInTile] = OpAt{sp + (y.pos ? y.delta : 0), sn + (y.pos ? 0 : y.delta), e + 1, cp + (y.pos ? 1 : 0)};
    }
  }
  __syncthreads();
  uint64_t *const words = reinterpret_cast<uint64_t *>(at);
  for (uint32_t g = 0; g <= kFewInTile; ++g) {
    const uint64_t *const x = reinterpret_cast<const uint64_t *>(gaps.x + g);
    const uint32_t end = gaps.hi[g] * 3;
    const uint64_t v[3] = {x[tid % 3], x[(tid + 1) % 3], x[(tid + 2) % 3]};
    uint32_t w = gaps.lo[g] * 3 + tid;
    for (; w + 2 * kTileThreads < end; w += 3 * kTileThreads)
#pragma unroll
      for (uint32_t u = 0; u < 3; ++u) words[w + u * kTileThreads] = v[u];
    if (w < end) words[w] = v[0];
    if (w + kTileThreads < end) words[w + kTileThreads] = v[1];
  }
}

// How long a workgroup waits for the sums of the tiles before its own (10 ns each).  They belong to workgroups that are
// started before it and wait for no later one, so it sees them within a few us; should one of them not run all the same,
// it adds up their events itself, and no wait depends on another workgroup's progress.
constexpr uint32_t kTileWaitTicks = 10000;

// Running sums along each list: OpAt, and for a timeline each event's own.  Also clears what a list out of order is
// gathered into.  A workgroup works out its tile, tells its sums, and takes up those of the tiles before it: one launch and
// one pass over the events where the sums had a launch of their own (100,000 + 40,000 events with a timeline 7.6 us in
// place of 4.1 + 9.1, a launch of about 2.5 and the second loading of the events; 1,048,574 + 20,014 events 30.4 in place of
// 7.4 + 25.5, the filling of gaps being the most of it).
// kFew: a list has few events to a tile and long gaps (its code in the others' kernel cost 100,000 + 40,000 events 0.2 us of 10.9).
template <int K, bool kOnce, bool kFew>
__global__ __launch_bounds__(kTileThreads) void ss_scan_running_kernel(ScanArgs a) {
  __shared__ SumShared sh;
  __shared__ TileSum part[kTileThreads / 64];
  const Tile tl(a);
  const uint32_t scan = max(a.board->scan + 1, 1u), tid = threadIdx.x;
  OpAt *const at = a.at + (tl.policy ? (size_t)a.n_ops + 1 : 0);
  Elem x[K];
  int64_t delta[K], xsp[K], xsn[K];
  uint32_t xcp[K];
  bool pos[K];
  TileSum mine;
  auto sums = [&](int64_t sp, int64_t sn, uint32_t cp) {
#pragma unroll
    for (int k = 0; k < K; ++k) { delta[k] = x[k].delta; pos[k] = x[k].pos; }
    wg_sums<kTileThreads, K>(sh, delta, pos, sp, sn, cp, xsp, xsn, xcp);
  };
  if constexpr (kOnce) {
    const uint32_t f = load_events<kTileThreads, K>(tl.src ? tl.src : tl.L, tl.cnt, nullptr, 0, tl.lo, tl.hi, a.n_ops, x);
    const uint32_t flags = (__ballot(f & 1u) ? 1u : 0u) | (__ballot(f & 2u) ? 2u : 0u);
    if ((tid & 63) == 0) part[tid >> 6].flags = flags;
    sums(0, 0, 0);
    mine = TileSum{sh.tot_sp, sh.tot_sn, sh.tot_cp, 0};
    for (int i = 0; i < kTileThreads / 64; ++i) mine.flags |= part[i].flags;
  } else {
    mine = sum_events<K>(a, tl, tl.lo, tl.hi, part);
  }
  if (tid == 0) put_tile(a.board, tl.index, scan, mine);
  if (blockIdx.x == 0 && tid == 0) a.board->done = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * kTileThreads + tid; i < a.n_ops; i += (uint64_t)gridDim.x * kTileThreads)
    a.pos[i] = a.net[i] = 0;
  if (!tl.cnt)
    for (uint32_t t = tid; t <= a.n_ops; t += kTileThreads) at[t] = OpAt{0, 0, 0, 0};
  if (kOnce && tl.src) {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (x[k].live) const_cast<ss_event_t *>(tl.L)[tl.lo + (uint64_t)k * kTileThreads + tid] = ss_event_t{x[k].op, 0, x[k].delta};
  }
  if (mine.flags) return;                                    // an operator out of range, or to be gathered
  TileSum before = {0, 0, 0, 0};
  if (tl.index != tl.first) {
    bool there = true;
    const uint64_t since = wall_clock64();
    for (uint32_t i = tl.first + tid; there && i < tl.index; i += kTileThreads) {
      TileSum s;
      while (!get_tile(a.board, i, scan, s))
        if (wall_clock64() - since > a.wait_ticks) { there = false; break; }
      before.sp += s.sp; before.sn += s.sn; before.cp += s.cp; before.flags |= s.flags;
    }
    __syncthreads();                                         // everyone has read its part
    before = wg_total(before.sp, before.sn, before.cp, before.flags, part);
    if (__syncthreads_or(!there)) before = sum_events<K>(a, tl, 0, tl.lo, part);
  }
  if (before.flags) return;
  // Where filling gaps is the work it is not done for nothing if the other list is out of order: the policy's tiles wait for
  // those of the events, which were started before them (a reversed trace of 1,000 events over 65,536 operators beside 8 of
  // the policy: the call 269 us without and 217 with it), the events' own only look.  Of few events to a tile the tiles before
  // the one where the order breaks look at a line of words of their list's next ones as well (10 events in random order, a tile each,
  // beside 12 of the policy over 65,536 operators 151 us without and 127 with it; 100 events 144 and 126).
  if (a.n_ops > 2 * tl.cnt) {
    bool over = false;
    const uint32_t own_end = tl.policy ? a.tiles0 + a.tiles1 : a.tiles0;
    constexpr uint32_t kLooks = 16;
    uint64_t later = 0;
    if (kFew && tid < kLooks && tl.index + 1 + tid < own_end)
      later = __hip_atomic_load(&a.board->tile[4][tl.index + 1 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t since = wall_clock64();
    const uint32_t first = tl.policy ? 0 : a.tiles0, end = tl.policy ? a.tiles0 : a.tiles0 + a.tiles1;
    for (uint32_t i = first + tid; i < end; i += kTileThreads) {
      uint64_t last;                                         // of a tile's words; it has the flags
      do last = __hip_atomic_load(&a.board->tile[4][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      while ((uint32_t)(last >> 32) != scan && tl.policy && wall_clock64() - since <= a.wait_ticks);
      over |= (uint32_t)(last >> 32) == scan && ((uint32_t)last >> 30);
    }
    over |= (uint32_t)(later >> 32) == scan && ((uint32_t)later >> 30);
    if (__syncthreads_or(over)) return;
  }
  const bool few = kFew && few_in_tile(a.tile[tl.policy], tl.cnt, a.n_ops);
  for (uint64_t lo = tl.lo; lo < tl.hi; lo += (uint64_t)kTileThreads * K) {
    if constexpr (kOnce) {
#pragma unroll
      for (int k = 0; k < K; ++k) { xsp[k] += before.sp; xsn[k] += before.sn; xcp[k] += before.cp; }
    } else {
      load_events<kTileThreads, K>(tl.L, tl.cnt, nullptr, 0, lo, tl.hi, a.n_ops, x);
      sums(before.sp, before.sn, before.cp);
      before.sp = sh.tot_sp; before.sn = sh.tot_sn; before.cp = sh.tot_cp;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint64_t e = lo + (uint64_t)k * kTileThreads + tid;
      if (a.want_timeline && x[k].live) {
        a.sumx[tl.out0 + e] = (pos[k] ? xsp[k] : xsn[k]) + delta[k];
        a.cntx[tl.out0 + e] = pos[k] ? xcp[k] : (uint32_t)e - xcp[k];
      }
      if (!few) fill_from<16>(at, x[k], (uint32_t)e, xsp[k], xsn[k], xcp[k], a.n_ops);
    }
    if constexpr (kFew) {
      __shared__ FewGaps gaps;
      if (few) fill_together(at, gaps, x[0], (uint32_t)(lo + tid), xsp[0], xsn[0], xcp[0], a.n_ops);
    }
    __syncthreads();                                         // sh is written again in the next pass
  }
}

constexpr int kGatherK = 1;

// Up to this many events one workgroup gathers them all and goes on with the operators: 290 events out of order over 8,045
// operators 26.9 us, gathered by all workgroups 29.5; 1,000 + 500 over 4,000 19.6 and 21.4; but 2,000 in random order over
// 8,000 31.2 and 29.6, and 4,000 over 3,000 26.0 and 19.4.
constexpr uint64_t kGatherAlone = 1536;

// true in the workgroup that ends last of `wgs` that call this; what the others wrote before is visible to it.  One release a
// workgroup, and an acquire in the last one (fences both ways in all its wavefronts: 8,000 + 100 events out of order over 5,000
// operators 23.3 us, so 21.7).
__device__ __forceinline__ bool ends_last(TileBoard *b, uint32_t wgs, uint32_t *s_last) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // this wavefront's stores and atomics are complete
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");       // for the workgroup (one fence each: 64 workgroups' 1,024 took 14 us)
    *s_last = __hip_atomic_fetch_add(&b->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == wgs;
  }
  __syncthreads();
  if (!*s_last) return false;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return true;
}

// Operators (workgroups [0, op_wgs)) and, for a timeline, events (those from op_wgs on).  The first operator workgroup folds
// all their maxima; it waits for each as the tiles do, and goes through the operators of one that doesn't come itself.
// (With a fence and a counter, the last one folding: two operator workgroups 6 us more than one.)  Lists out of order are
// gathered by all workgroups, and the last one to end does the operators.
struct FinishShared {
  Best part[kWaves];
  SumShared sums;
  uint32_t last, flags[kWaves];
};

__device__ __forceinline__ void scan_finish(const ScanArgs &a, uint32_t op_wgs, FinishShared &sh) {
  const uint32_t n = a.n_ops, tid = threadIdx.x;
  const uint32_t scan = (uint32_t)(a.board->tile[4][0] >> 32);      // this scan's number, as the first launch used it
  if (blockIdx.x == 0 && tid == 0) a.board->scan = scan;
  const uint64_t total = a.n_ev + a.n_pe;
  const OpAt *const at_ev = a.at, *const at_pe = a.at + n + 1;
  uint32_t flags = 0;
  for (uint32_t i = tid; i < a.tiles0 + a.tiles1; i += kThreads) flags |= (uint32_t)a.board->tile[4][i] >> 30;
  flags = (__ballot(flags & 1u) ? 1u : 0u) | (__ballot(flags & 2u) ? 2u : 0u);
  if ((tid & 63) == 0) sh.flags[tid >> 6] = flags;
  __syncthreads();
  flags = 0;
  for (int i = 0; i < kWaves; ++i) flags |= sh.flags[i];
  if (flags & 1u) {
    if (blockIdx.x == 0 && tid == 0) write_result(a, no_best(), a.base, flags);
    return;
  }
  if (flags) {
    const bool alone = total <= kGatherAlone;
    if (alone && blockIdx.x) return;
    const uint32_t wgs = alone ? 1 : gridDim.x;
    for (uint64_t first = (uint64_t)blockIdx.x * kThreads * kGatherK; first < total; first += (uint64_t)wgs * kThreads * kGatherK) {
      Elem x[kGatherK];
      load_events<kThreads, kGatherK>(a.ev, a.n_ev, a.pev, a.n_pe, first, total, n, x);
#pragma unroll
      for (int k = 0; k < kGatherK; ++k) gather_run(a.pos, a.net, x[k], n);
    }
    if (alone) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __syncthreads();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    } else if (!ends_last(a.board, wgs, &sh.last)) {
      return;
    }
    Best b = ops_of_sums<kThreads>(a, a.pos, a.net, sh.sums);
    b = wg_best<kThreads>(b, sh.part);
    if (tid == 0) write_result(a, b, a.base + (n ? sh.sums.tot_sp : 0), flags);
    return;
  }
  if (blockIdx.x >= op_wgs) {
    if (!a.want_timeline) return;
    for (uint64_t i = (uint64_t)(blockIdx.x - op_wgs) * kThreads + tid; i < total; i += (uint64_t)(gridDim.x - op_wgs) * kThreads) {
      const bool policy = i >= a.n_ev;
      const ss_event_t x = policy ? a.pev[i - a.n_ev] : a.ev[i];
      put_event(a, a.timeline, policy, x.delta >= 0, a.sumx[i], a.cntx[i], at_ev[x.op_idx], at_ev[x.op_idx + 1], at_pe[x.op_idx],
                at_pe[x.op_idx + 1]);
    }
    return;
  }
  auto operators = [&](uint32_t first, uint32_t step) {
    Best b = no_best();
    for (uint32_t t = first; t < n; t += step)
      put_op(a, t, a.base + at_ev[t + 1].sp + at_pe[t + 1].sp + at_ev[t].sn + at_pe[t].sn, b);
    return b;
  };
  Best b = wg_best<kThreads>(operators(blockIdx.x * kThreads + tid, op_wgs * kThreads), sh.part);
  if (blockIdx.x) {
    const uint32_t x[4] = {low_half(b.val), high_half(b.val), b.idx, b.over};
    if (tid == 0) tell(a.board->best, blockIdx.x, scan, x);
    return;
  }
  if (op_wgs > 1) {
    Best other = tid == 0 ? b : no_best();
    bool there = true;
    if (tid && tid < op_wgs) {
      const uint64_t since = wall_clock64();
      uint32_t x[4];
      while (!hear(a.board->best, tid, scan, x))
        if (wall_clock64() - since > a.wait_ticks) { there = false; break; }
      other = Best{both_halves(x[0], x[1]), x[2], x[3]};
    }
    if (__syncthreads_or(!there)) other = operators(tid, kThreads);
    b = wg_best<kThreads>(other, sh.part);
  }
  if (tid == 0) write_result(a, b, a.base + at_ev[n].sp + at_ev[n].sn + at_pe[n].sp + at_pe[n].sn, 0);
}

__global__ __launch_bounds__(kThreads) void ss_scan_finish_kernel(ScanArgs a, uint32_t op_wgs) {
  __shared__ FinishShared sh;
  scan_finish(a, op_wgs, sh);
  ss_tell_host(a.done);
}

// Events of a tile.  Few to a lane is the faster form as long as there are no more tiles than a workgroup may read (the
// two launches of 140,000 events: two to a lane 12.2 us, four 13.1, eight 15.8; the first of 1,068,588 events: two, in two
// passes, 30.4 us, four 32.1, eight 42.9), so a lane gets two, or four, and beyond that a tile takes several passes of eight.
// Where operators outnumber the events, filling the gaps between them is the work (a wavefront fills gaps above kAlone one
// after the other), and few events to a tile spread it: 60,000 operators with 40,000 events and 2,000 of the policy
// 82 -> 40 us, with 6,000 and 200 66 -> 41.  Of at most 2,048 events a tile takes as many as fill about 1,024 operators, but no more
// than 8 and no fewer than make 256 tiles (one each always: 3,500 operators with 124 events, which take 8, 15.6 us, so 13.7).
// A lane that gets two or four loads them once, so there a tile is at most one pass.
int events_per_lane(uint64_t n) {
  return n <= kMaxTiles * kTileThreads * 2 ? 2 : n <= kMaxTiles * kTileThreads * 4 ? 4 : 8;
}

uint32_t tile_events(uint64_t n, uint32_t n_ops, int per_lane) {
  const uint64_t pass = (uint64_t)kTileThreads * per_lane;
  if (n_ops > 2 * n) {
    const uint64_t some = std::min<uint64_t>(kFewInTile, std::max<uint64_t>({1, (n + 255) / 256, n * 1024 / n_ops}));
    const uint64_t spread = n <= 2048 ? some : ss_align_up((n + 255) / 256, 8);
    return (uint32_t)(per_lane == 8 ? spread : std::min(spread, pass));
  }
  return (uint32_t)std::max(pass, ss_align_up((n + kMaxTiles - 1) / kMaxTiles, pass));
}

struct Tiling {
  int per_lane;
  uint32_t tile[2], tiles[2];        // events of a tile, tiles: of the trace's events, of the policy's
};

Tiling tiling_of(uint64_t n_ev, uint64_t n_pe, uint32_t n_ops) {
  Tiling t;
  t.per_lane = events_per_lane(std::max(n_ev, n_pe));
  for (int l = 0; l < 2; ++l) {
    const uint64_t n = l ? n_pe : n_ev;
    t.tile[l] = tile_events(n, n_ops, t.per_lane);
    t.tiles[l] = (uint32_t)std::max<uint64_t>(1, (n + t.tile[l] - 1) / t.tile[l]);
  }
  return t;
}

// The kernel of the running sums is the one that fills gaps together.  A list without events fills none: 100,000 events and none of the
// policy over 400 operators 9.0 us, by that kernel 9.8.
bool few_events(const Tiling &t, uint64_t n_ev, uint64_t n_pe, uint32_t n_ops) {
  return few_in_tile(t.tile[0], n_ev, n_ops) || few_in_tile(t.tile[1], n_pe, n_ops);
}

// One workgroup takes a trace whose events fit its registers and whose tables fit LDS.  Up to there it is the faster form: a
// call for 3,500 + 500 events over 2,500 operators 9.3 us, with a timeline 11.0, the two launches of the other 11 at least.
bool is_short(uint64_t n_ev, uint64_t n_pe, uint32_t n_ops, bool timeline) {
  if (n_ev + n_pe > kSmallEvents || n_ops > kLdsOps) return false;
  const ShortForm f = short_form(n_ev, n_pe, n_ops);
  return f.T && short_lds(f.T, f.K, n_ops, n_ev + n_pe, timeline) <= kShortLds;
}

// Host calls: up to this much goes through the context's pinned scratch (which starts at 1 MiB), read and written by the
// kernels themselves; a copy call for pageable memory costs 19 to 33 us at 16 to 64 KiB and a copy from pinned memory a
// launch, the link's time is the same.  Beyond it the copy engine keeps up with the link and the call's cost is small.
constexpr size_t kMappedBytes = 768 * 1024;
static_assert(kMappedBytes / sizeof(ss_event_t) <= kMaxTiles * kTileThreads * 2, "only tiles of one pass copy their events");

// Scratch of a long trace from `d` on; returns its size (nothing is assigned where `a` is null).
size_t scan_scratch(ScanArgs *a, uint8_t *d, uint64_t n_ev, uint64_t n_pe, uint64_t n_ops, bool timeline) {
  size_t off = 0;
  auto take = [&](size_t bytes) { uint8_t *p = d + off; off += ss_align_up(bytes, 256); return p; };
  const uint64_t E = timeline ? n_ev + n_pe : 0;
  uint8_t *at = take(2 * (n_ops + 1) * sizeof(OpAt)), *pos = take(n_ops * 8), *net = take(n_ops * 8);
  uint8_t *sumx = take(E * 8), *cntx = take(E * 4);
  if (a) {
    a->at = (OpAt *)at;
    a->pos = (int64_t *)pos;
    a->net = (int64_t *)net;
    a->sumx = (int64_t *)sumx;
    a->cntx = (uint32_t *)cntx;
  }
  return off;
}

void launch_scan(hipStream_t s, ScanArgs &a) {
  if (is_short(a.n_ev, a.n_pe, a.n_ops, a.want_timeline)) {
    const ShortForm f = short_form(a.n_ev, a.n_pe, a.n_ops);
    const size_t bytes = short_lds(f.T, f.K, a.n_ops, a.n_ev + a.n_pe, a.want_timeline);
    const uint32_t tl_at = (uint32_t)short_tables(f.T, f.K, a.n_ops);
#define SS_LAUNCH(T, K) hipLaunchKernelGGL((ss_scan_short_kernel<T, K>), dim3(1), dim3(T), bytes, s, a, tl_at)
    SS_SHORT_FORM(f, SS_LAUNCH);
#undef SS_LAUNCH
    return;
  }
  const Tiling t = tiling_of(a.n_ev, a.n_pe, a.n_ops);
  const int per_lane = t.per_lane;
  a.tile[0] = t.tile[0];
  a.tile[1] = t.tile[1];
  if (!a.wait_ticks) a.wait_ticks = kTileWaitTicks;
  a.tiles0 = t.tiles[0];
  a.tiles1 = t.tiles[1];
  const uint32_t tiles = a.tiles0 + a.tiles1;
  const uint32_t op_wgs = (uint32_t)std::min<uint64_t>(kMaxOpWgs, std::max<uint64_t>(1, ((uint64_t)a.n_ops + kThreads - 1) / kThreads));
  // without a timeline these are there for lists out of order only, and end at once where there are none
  const uint64_t per_wg = a.want_timeline ? kThreads : kGatherK * kThreads;
  const uint32_t ev_wgs = (uint32_t)std::min<uint64_t>(2048, (a.n_ev + a.n_pe + per_wg - 1) / per_wg);
  const bool few = few_events(t, a.n_ev, a.n_pe, a.n_ops);
#define SS_LAUNCH(K, ONCE)                                                                                                     \
  if (few) hipLaunchKernelGGL((ss_scan_running_kernel<K, ONCE, true>), dim3(tiles), dim3(kTileThreads), 0, s, a);              \
  else hipLaunchKernelGGL((ss_scan_running_kernel<K, ONCE, false>), dim3(tiles), dim3(kTileThreads), 0, s, a)
  if (per_lane == 2) { SS_LAUNCH(2, true); }
  else if (per_lane == 4) { SS_LAUNCH(4, true); }
  else { SS_LAUNCH(8, false); }
#undef SS_LAUNCH
  ss_told_by(a.done, op_wgs + ev_wgs);
  hipLaunchKernelGGL(ss_scan_finish_kernel, dim3(op_wgs + ev_wgs), dim3(kThreads), 0, s, a, op_wgs);
}

}  // namespace

// ---- the scan for callers that cannot allocate ------------------------------------------------
//
// Same kernels, but their scratch lies in a static device array instead of memory the library allocates, and inputs
// and outputs are the caller's device arrays: the call only enqueues the scan's kernels (one, or two for a long
// trace) on the caller's stream.

constexpr uint32_t kStaticMaxOps = 65536;
constexpr uint64_t kStaticMaxEvents = 262144;
constexpr size_t kBoardBytes = (sizeof(TileBoard) + 255) / 256 * 256;
constexpr size_t kStaticBytes = kBoardBytes + 2 * (kStaticMaxOps + 1) * sizeof(OpAt) + 2 * kStaticMaxOps * 8 +
                                kStaticMaxEvents * 12 + 8 * 256;
// Contexts take their boards from a pool behind it (one more than it holds allocates its own): an allocation and a clear for
// each made preparing a 7B alignment 853 -> 977 us.
constexpr int kPoolBoards = 32;
constexpr size_t kToldBytes = 256, kOwnBoard = kToldBytes + kBoardBytes, kPoolAt = (kStaticBytes + 255) / 256 * 256;
static __device__ __align__(256) uint8_t scratch[kPoolAt + kPoolBoards * kOwnBoard];          // starts as zeros: so do the boards

// Address of `scratch` on each device (the name itself is only a host-side handle): resolved once
// per device, with that device current.
constexpr int kMaxDevices = 64;
static uint8_t *g_scratch_ptr[kMaxDevices];

static int static_scratch_ptr(int device, uint8_t **out, hipError_t *err) {
  *err = hipSuccess;
  if (device < 0 || device >= kMaxDevices) return SS_E_INVAL;
  if (!g_scratch_ptr[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      *err = e;
      return SS_E_HIP;
    }
    g_scratch_ptr[device] = (uint8_t *)p;
  }
  *out = g_scratch_ptr[device];
  return SS_OK;
}

int ss_scan_static_init(ss_ctx *ctx) {
  uint8_t *p;
  hipError_t e;
  const int rc = static_scratch_ptr(ctx->device, &p, &e);
  if (rc == SS_E_HIP) SS_HIP(e);
  return rc;
}

static std::mutex g_boards_mu;
static uint32_t g_boards_taken[kMaxDevices];
static_assert(kPoolBoards <= 32, "a bit for each");

int ss_scan_board_take(ss_ctx *ctx) {
  uint8_t *base = nullptr;
  hipError_t e;
  const int rc = static_scratch_ptr(ctx->device, &base, &e);
  if (rc == SS_E_HIP) SS_HIP(e);
  if (rc != SS_OK) return rc;
  {
    std::lock_guard<std::mutex> lock(g_boards_mu);
    uint32_t &taken = g_boards_taken[ctx->device];
    for (int i = 0; i < kPoolBoards && ctx->pool_board < 0; ++i)
      if (!(taken >> i & 1u)) {
        taken |= 1u << i;
        ctx->pool_board = i;
      }
  }
  if (ctx->pool_board >= 0) {
    ctx->d_told = (uint32_t *)(base + kPoolAt + (size_t)ctx->pool_board * kOwnBoard);
  } else {
    SS_HIP(hipMalloc((void **)&ctx->d_told, kOwnBoard));
    ss_launch_fill(ctx->s_aux, (uint8_t *)ctx->d_told, kOwnBoard, 0);       // their kernels run there too
    SS_HIP(hipGetLastError());
  }
  ctx->d_board = (uint8_t *)ctx->d_told + kToldBytes;
  return SS_OK;
}

// Once nothing of the context runs any more.  The next one takes the board as it is (see TileBoard).
void ss_scan_board_give(ss_ctx *ctx) {
  if (ctx->pool_board >= 0) {
    std::lock_guard<std::mutex> lock(g_boards_mu);
    g_boards_taken[ctx->device] &= ~(1u << ctx->pool_board);
  } else if (ctx->d_told) {
    (void)hipFree(ctx->d_told);
  }
  ctx->pool_board = -1;
  ctx->d_told = nullptr;
}

extern "C" int ss_timeline_scan_static(ss_ctx *ctx, void *stream, const ss_event_t *d_ev, uint64_t n_ev,
                                       const ss_event_t *d_pev, uint64_t n_pe, uint32_t n_ops, int64_t base,
                                       int64_t budget, int64_t *d_timeline, int64_t *d_per_op, int64_t *d_mre,
                                       ss_scan_result_t *d_res) {
  if (!ctx || !d_res || (n_ev && !d_ev) || (n_pe && !d_pev)) return SS_E_INVAL;
  if (n_ops > kStaticMaxOps || n_ev > kStaticMaxEvents || n_pe > kStaticMaxEvents || n_ev + n_pe > kStaticMaxEvents)
    return SS_E_CAPACITY;
  int dev = -1;
  SS_HIP(hipGetDevice(&dev));
  if (dev != ctx->device) return SS_E_STATE;          // the context's copy of the array is on its own device
  uint8_t *d = nullptr;
  hipError_t e;
  const int rc = static_scratch_ptr(dev, &d, &e);
  if (rc == SS_E_HIP) SS_HIP(e);
  if (rc != SS_OK) return rc;
  ScanArgs a = {};
  a.ev = d_ev; a.n_ev = n_ev;
  a.pev = d_pev; a.n_pe = n_pe;
  a.n_ops = n_ops; a.want_timeline = d_timeline != nullptr;
  a.base = base; a.budget = budget;
  a.board = (TileBoard *)d;
  scan_scratch(&a, d + kBoardBytes, n_ev, n_pe, n_ops, true);          // at most kStaticBytes
  a.per_op = d_per_op; a.mre = d_mre; a.timeline = d_timeline;
  a.res = d_res;
  launch_scan((hipStream_t)stream, a);
  SS_HIP(hipGetLastError());
  return SS_OK;
}

extern "C" int ss_timeline_scan_batch(ss_ctx *ctx, const ss_event_t *ev, uint64_t n_ev, const ss_event_t *pev,
                                      const uint64_t *pe_start, uint32_t k, uint32_t n_ops, int64_t base,
                                      int64_t budget, int64_t *per_op, ss_scan_result_t *res) {
  return ss_guard([&]() -> int {
    if (!ctx || (k && (!res || !pe_start)) || (n_ev && !ev)) return SS_E_INVAL;
    if (k == 0) return SS_OK;
    if (k > 4096 || n_ops > (1u << 23)) return SS_E_INVAL;
    const uint64_t n_pe = pe_start[k];
    for (uint32_t c = 0; c < k; ++c)
      if (pe_start[c] > pe_start[c + 1]) return SS_E_INVAL;
    if (pe_start[0] != 0 || (n_pe && !pev) || n_ev + n_pe >= (1ull << 31)) return SS_E_INVAL;
    const uint64_t n = n_ops;
    const bool lds = n_ops <= kLdsOps;                 // the OpAt tables fit LDS
    const size_t ev_bytes = n_ev * sizeof(ss_event_t), pe_bytes = n_pe * sizeof(ss_event_t);
    // every scan reads the trace once: over the link while that takes no longer than the two copies' calls (about 40 us)
    const bool mapped = ev_bytes + pe_bytes <= kMappedBytes / 2 && k * (uint64_t)ev_bytes <= (1u << 20);
    size_t off = 0, hoff = 0;
    auto take = [](size_t &o, size_t bytes) { size_t at = o; o += ss_align_up(bytes, 256); return at; };
    const size_t args_bytes = ss_align_up((size_t)k * sizeof(ScanArgs), 256);
    take(hoff, args_bytes + (size_t)k * sizeof(ss_scan_result_t));
    const size_t o_ev = take(mapped ? hoff : off, ev_bytes), o_pev = take(mapped ? hoff : off, pe_bytes);
    const size_t per_scan = lds ? 0 : ss_align_up(2 * (n + 1) * sizeof(OpAt), 256) + 2 * ss_align_up(n * 8, 256);
    const size_t o_work = take(off, (size_t)k * per_scan), o_per_op = take(off, per_op ? (size_t)k * n * 8 : 0);
    int rc = ss_scratch_reserve(ctx, off, hoff);
    if (rc != SS_OK) return rc;
    uint8_t *d = (uint8_t *)ctx->d_scratch, *h = (uint8_t *)ctx->h_scratch, *hd = nullptr;
    SS_HIP(hipHostGetDevicePointer((void **)&hd, h, 0));
    hipStream_t s = ctx->s_aux;
    if (mapped) {
      if (n_ev) std::memcpy(h + o_ev, ev, ev_bytes);
      if (n_pe) std::memcpy(h + o_pev, pev, pe_bytes);
    } else {
      if (n_ev) SS_HIP(hipMemcpyAsync(d + o_ev, ev, ev_bytes, hipMemcpyHostToDevice, s));
      if (n_pe) SS_HIP(hipMemcpyAsync(d + o_pev, pev, pe_bytes, hipMemcpyHostToDevice, s));
    }
    const uint8_t *const in = mapped ? hd : d;
    ss_done done = {};
    if (!per_op || (size_t)k * n * 8 <= kToldCopyBytes) {
      done = ss_next_done(ctx);
      ss_told_by(done, k);
    }
    ScanArgs *ha = (ScanArgs *)h;                       // pinned, read and written by the kernel: arguments, results
    for (uint32_t c = 0; c < k; ++c) {
      uint8_t *w = d + o_work + (size_t)c * per_scan;
      ScanArgs a = {};
      a.ev = (const ss_event_t *)(in + o_ev); a.n_ev = n_ev;
      a.pev = (const ss_event_t *)(in + o_pev) + pe_start[c]; a.n_pe = pe_start[c + 1] - pe_start[c];
      a.n_ops = n_ops;
      a.base = base; a.budget = budget;
      if (!lds) {
        a.at = (OpAt *)w;
        a.pos = (int64_t *)(w + ss_align_up(2 * (n + 1) * sizeof(OpAt), 256));
        a.net = a.pos + ss_align_up(n * 8, 256) / 8;
      }
      a.done = done;
      if (per_op) a.per_op = (int64_t *)(d + o_per_op) + (size_t)c * n;
      a.res = (ss_scan_result_t *)(hd + args_bytes) + c;
      ha[c] = a;
    }
    const ScanArgs *dargs = (const ScanArgs *)hd;
    ShortForm f = {0, 0};                               // one for all
    bool all_short = lds;
    for (uint32_t c = 0; c < k && all_short; ++c) {
      const ShortForm g = short_form(n_ev, ha[c].n_pe, n_ops);
      all_short = g.T && n_ev + ha[c].n_pe <= kSmallEvents && short_lds(g.T, g.K, n_ops, 0, false) <= kShortLds;
      if (g.T * g.K > f.T * f.K) f = g;
    }
    if (all_short) {
#define SS_LAUNCH(T, K) \
  hipLaunchKernelGGL((ss_scan_short_batch_kernel<T, K>), dim3(k), dim3(T), short_lds(T, K, n_ops, 0, false), s, dargs)
      SS_SHORT_FORM(f, SS_LAUNCH);
#undef SS_LAUNCH
    } else if (lds) hipLaunchKernelGGL(ss_scan_batch_kernel<true>, dim3(k), dim3(kThreads), lds_at(n_ops), s, dargs);
    else hipLaunchKernelGGL(ss_scan_batch_kernel<false>, dim3(k), dim3(kThreads), 0, s, dargs);
    SS_HIP(hipGetLastError());
    if ((rc = ss_wait_done(ctx, done)) != SS_OK) return rc;
    const ss_scan_result_t *hres = (const ss_scan_result_t *)(h + args_bytes);
    for (uint32_t c = 0; c < k; ++c)
      if (hres[c].reserved & 1u) return SS_E_INVAL;
    for (uint32_t c = 0; c < k; ++c) {
      res[c] = hres[c];
      res[c].reserved = 0;
    }
    if (per_op && n) {
      SS_HIP(hipMemcpyAsync(per_op, d + o_per_op, (size_t)k * n * 8, hipMemcpyDeviceToHost, s));
      SS_HIP(hipStreamSynchronize(s));
    }
    return SS_OK;
  });
}

extern "C" int ss_timeline_scan(ss_ctx *ctx, const ss_event_t *ev, uint64_t n_ev, const ss_event_t *pev,
                                uint64_t n_pe, uint32_t n_ops, int64_t base, int64_t budget,
                                int64_t *timeline, int64_t *per_op, int64_t *mre, ss_scan_result_t *res) {
  return ss_guard([&]() -> int {
    if (!ctx || !res || (n_ev && !ev) || (n_pe && !pev)) return SS_E_INVAL;
    if (n_ops > (1u << 23) || n_ev + n_pe >= (1ull << 31)) return SS_E_INVAL;
    const uint64_t E = n_ev + n_pe, n = n_ops;
    hipStream_t s = ctx->s_aux;
    ScanArgs a = {};
    a.n_ev = n_ev; a.n_pe = n_pe;
    a.n_ops = n_ops; a.want_timeline = timeline != nullptr;
    a.base = base; a.budget = budget;
    const size_t ev_bytes = n_ev * sizeof(ss_event_t), pe_bytes = n_pe * sizeof(ss_event_t);
    const size_t out_bytes = (per_op ? n * 8 : 0) + (mre ? n * 8 : 0) + (timeline ? E * 8 : 0);
    // Short traces: the one kernel reads the events out of pinned memory.  Longer ones: the first kernel does, and copies
    // them on the way for the second.  Results are written to pinned memory in both cases.
    const bool is_small = is_short(n_ev, n_pe, n_ops, timeline != nullptr);
    const bool in_mapped = is_small || ev_bytes + pe_bytes <= kMappedBytes;
    const bool out_mapped = is_small || (in_mapped ? ev_bytes + pe_bytes : 0) + out_bytes <= kMappedBytes;
    size_t off = 0, hoff = 0;
    auto take = [](size_t &o, size_t bytes) { size_t at = o; o += ss_align_up(bytes, 256); return at; };
    const size_t ho_ev = take(hoff, in_mapped ? ev_bytes : 0), ho_pev = take(hoff, in_mapped ? pe_bytes : 0);
    const size_t o_ev = take(off, is_small ? 0 : ev_bytes), o_pev = take(off, is_small ? 0 : pe_bytes);
    size_t &oo = out_mapped ? hoff : off;
    const size_t o_perop = take(oo, per_op ? n * 8 : 0), o_mre = take(oo, mre ? n * 8 : 0);
    const size_t o_tl = take(oo, timeline ? E * 8 : 0), o_res = take(hoff, sizeof(ss_scan_result_t));
    const size_t o_scratch = take(off, is_small ? 0 : scan_scratch(nullptr, nullptr, n_ev, n_pe, n, timeline != nullptr));
    int rc = ss_scratch_reserve(ctx, off, hoff);
    if (rc != SS_OK) return rc;
    uint8_t *d = (uint8_t *)ctx->d_scratch, *h = (uint8_t *)ctx->h_scratch, *hd = nullptr;
    SS_HIP(hipHostGetDevicePointer((void **)&hd, h, 0));
    uint8_t *const out = out_mapped ? hd : d;
    a.ev = (const ss_event_t *)(is_small ? hd + ho_ev : d + o_ev);
    a.pev = (const ss_event_t *)(is_small ? hd + ho_pev : d + o_pev);
    if (in_mapped) {
      if (n_ev) std::memcpy(h + ho_ev, ev, ev_bytes);
      if (n_pe) std::memcpy(h + ho_pev, pev, pe_bytes);
      if (!is_small) {
        a.src_ev = (const ss_event_t *)(hd + ho_ev);
        a.src_pev = (const ss_event_t *)(hd + ho_pev);
      }
    } else {
      if (n_ev) SS_HIP(hipMemcpyAsync(d + o_ev, ev, ev_bytes, hipMemcpyHostToDevice, s));
      if (n_pe) SS_HIP(hipMemcpyAsync(d + o_pev, pev, pe_bytes, hipMemcpyHostToDevice, s));
    }
    if (!is_small) {
      scan_scratch(&a, d + o_scratch, n_ev, n_pe, n, timeline != nullptr);
      a.board = (TileBoard *)ctx->d_board;
      a.wait_ticks = ctx->scan_wait_ticks;
    }
    a.per_op = per_op ? (int64_t *)(out + o_perop) : nullptr;
    a.mre = mre ? (int64_t *)(out + o_mre) : nullptr;
    a.timeline = timeline ? (int64_t *)(out + o_tl) : nullptr;
    a.res = (ss_scan_result_t *)(hd + o_res);
    if (out_mapped || (per_op || mre ? n : E) * 8 <= kToldCopyBytes) a.done = ss_next_done(ctx);
    launch_scan(s, a);
    SS_HIP(hipGetLastError());
    if ((rc = ss_wait_done(ctx, a.done)) != SS_OK) return rc;
    ss_scan_result_t r;
    std::memcpy(&r, h + o_res, sizeof(r));
    const uint32_t flags = r.reserved;
    if (flags & 1u) return SS_E_INVAL;
    r.reserved = 0;
    *res = r;
    const bool tl_ok = timeline && !(flags & 2u);
    if (out_mapped) {
      if (per_op && n) std::memcpy(per_op, h + o_perop, n * 8);
      if (mre && n) std::memcpy(mre, h + o_mre, n * 8);
      if (tl_ok && E) std::memcpy(timeline, h + o_tl, E * 8);
    } else {
      if (per_op && n) SS_HIP(hipMemcpyAsync(per_op, d + o_perop, n * 8, hipMemcpyDeviceToHost, s));
      if (mre && n) SS_HIP(hipMemcpyAsync(mre, d + o_mre, n * 8, hipMemcpyDeviceToHost, s));
      if (tl_ok && E) SS_HIP(hipMemcpyAsync(timeline, d + o_tl, E * 8, hipMemcpyDeviceToHost, s));
      SS_HIP(hipStreamSynchronize(s));
    }
    if (timeline && !tl_ok) return SS_E_ORDER;
    return SS_OK;
  });
}

// For tests: how long a workgroup of the context's long scans waits for a tile's sums (10 ns each; 0 = the usual time).
extern "C" void ss_scan_wait_limit(ss_ctx *ctx, uint32_t ticks) {
  if (ctx) ctx->scan_wait_ticks = ticks;
}

// For tests: how a long trace is cut. out: events to a lane, then for each list the events of a tile and the tiles.
extern "C" void ss_scan_tiling(uint64_t n_ev, uint64_t n_pe, uint32_t n_ops, uint32_t *out) {
  const Tiling t = tiling_of(n_ev, n_pe, n_ops);
  out[0] = (uint32_t)t.per_lane;
  for (int l = 0; l < 2; ++l) {
    out[1 + 2 * l] = t.tile[l];
    out[2 + 2 * l] = t.tiles[l];
  }
}

// For tests: whether its gaps are filled by whole workgroups.
extern "C" int ss_scan_few_events(uint64_t n_ev, uint64_t n_pe, uint32_t n_ops) {
  return few_events(tiling_of(n_ev, n_pe, n_ops), n_ev, n_pe, n_ops);
}

// For tests: the number of the scan that the context's last long one had.
extern "C" int ss_scan_number(ss_ctx *ctx, uint32_t number) {
  if (!ctx) return SS_E_INVAL;
  SS_HIP(hipStreamSynchronize(ctx->s_aux));
  SS_HIP(hipMemcpy(&((TileBoard *)ctx->d_board)->scan, &number, sizeof(number), hipMemcpyHostToDevice));
  return SS_OK;
}
