// Policy generator (Sec. 4 of the SmartSwap paper): logical layers with the time estimate of
// Eq. 1, the memory reduction list, the candidate list ranked by Eq. 2, the swap simulator
// (pre-triggered swap-in, Eq. 3; swap-out completion) and the loop of Algo. 2.  The memory curve
// without swaps and the check of the finished policy are timeline scans on the GPU; the
// simulator itself is sequential integer work on the host.  Time is counted in link bytes, so a
// transfer costs its size and a layer owns link_bytes_per_op times its operator count.
#include <algorithm>
#include <cstring>

#include "ss_internal.h"

namespace {

struct Layer {
  uint32_t first, end;     // operators [first, end)
  uint32_t type;           // 0 forward, 1 backward, 2 optimizer
  uint32_t lo, hi;         // its operators among its phase's: [lo, hi)
  int64_t remaining;       // link bytes still free in this layer
  uint64_t bpo;            // link bytes one operator of this layer is worth (Eq. 1)
};

struct Chosen {
  uint32_t row, layer_in, t_in, t_free;
  bool late;
};

typedef unsigned __int128 u128;

// What the parameter sets of a call share.  Entries are the operators over the limit (the memory reduction list of Sec. 4.2);
// there are far fewer of them than operators (67 of 700 at 90 % of the peak), and all that is asked of the list is asked for
// a stretch of it.
struct Shared {
  std::vector<uint32_t> ops_of[3];     // operators of each phase, in execution order
  std::vector<uint32_t> entry_op;      // operators of the entries
  std::vector<uint32_t> before;        // [n_ops + 1]: entries before the operator
  std::vector<int64_t> excess;         // of the entries
  // tensors that can be away from some entry: operators t with last_fwd_use + 1 < t < first_bwd_use
  struct Away { uint32_t row, lo, hi, id, last_fwd, first_bwd; uint64_t size; };
  std::vector<Away> away;
};

void share(const ss_op_t *ops, uint32_t n_ops, const ss_tensor_t *tensors, uint32_t n_tensors, const std::vector<int64_t> &per_op,
           int64_t limit, Shared &s) {
  s.before.resize(n_ops + 1);
  s.ops_of[0].reserve(n_ops);
  s.away.reserve(n_tensors);
  for (uint32_t i = 0; i < n_ops; ++i) {
    s.ops_of[std::min<uint32_t>(ops[i].sig >> 16, 2u)].push_back(i);
    s.before[i] = (uint32_t)s.entry_op.size();
    if (per_op[i] > limit) {
      s.entry_op.push_back(i);
      s.excess.push_back(per_op[i] - limit);
    }
  }
  s.before[n_ops] = (uint32_t)s.entry_op.size();
  for (uint32_t r = 0; r < n_tensors; ++r) {
    const ss_tensor_t &t = tensors[r];
    if (t.last_fwd_use == SS_NONE_OP || t.first_bwd_use == SS_NONE_OP || t.last_fwd_use >= t.first_bwd_use || t.first_bwd_use >= n_ops ||
        t.last_fwd_use + 2 >= t.first_bwd_use)
      continue;
    const uint32_t lo = s.before[t.last_fwd_use + 2], hi = s.before[t.first_bwd_use];
    if (lo < hi) s.away.push_back({r, lo, hi, t.tensor_id, t.last_fwd_use, t.first_bwd_use, t.nbytes});
  }
}

// The entries that are left, as a bit map with a second one over its words.
struct Entries {
  std::vector<uint64_t> word, some;
  std::vector<uint32_t> upto;          // entries left before each (before each word, if there are many), as of the last count()
  uint32_t left = 0, shift = 0;
  void all(uint32_t n, bool many) {
    left = n;
    shift = many ? 6 : 0;
    word.assign(n / 64 + 1, ~0ull);
    word[n / 64] = (1ull << n % 64) - 1;
    some.assign(word.size() / 64 + 1, 0);
    for (size_t w = 0; w < word.size(); ++w) some[w / 64] |= (uint64_t)(word[w] != 0) << w % 64;
    upto.resize((n >> shift) + 1);
  }
  bool has(uint32_t e) const { return word[e / 64] >> e % 64 & 1u; }
  void take(uint32_t w, uint64_t gone) {
    left -= (uint32_t)__builtin_popcountll(gone);
    if (!(word[w] &= ~gone)) some[w / 64] &= ~(1ull << w % 64);
  }
  void count() {
    uint32_t c = 0;
    for (size_t i = 0; i < upto.size(); ++i) {
      upto[i] = c;
      c += shift ? (uint32_t)__builtin_popcountll(word[i]) : has((uint32_t)i);
    }
  }
  uint32_t rank(uint32_t e) const {
    return shift ? upto[e / 64] + (uint32_t)__builtin_popcountll(word[e / 64] & ((1ull << e % 64) - 1)) : upto[e];
  }
  // the last one in [lo, hi), or -1
  int64_t last(uint32_t lo, uint32_t hi) const {
    uint64_t x = word[hi / 64] & ((1ull << hi % 64) - 1);
    uint32_t w = hi / 64;
    if (!x) {
      uint64_t y = some[w / 64] & ((1ull << w % 64) - 1);
      uint32_t v = w / 64;
      while (!y && v) y = some[--v];
      if (!y) return -1;
      w = v * 64 + 63 - (uint32_t)__builtin_clzll(y);
      x = word[w];
    }
    const uint32_t e = w * 64 + 63 - (uint32_t)__builtin_clzll(x);
    return e >= lo ? (int64_t)e : -1;
  }
};

// Cut the operators of each phase, in execution order, into groups of (almost) equal count.
void build_layers(const Shared &s, uint32_t n_ops, uint32_t g_fwd, uint32_t g_bwd, const uint64_t bpo[3], std::vector<Layer> &layers,
                  std::vector<uint32_t> &layer_of) {
  const uint32_t groups[3] = {g_fwd, g_bwd, 1};
  layers.clear();
  for (uint32_t ph = 0; ph < 3; ++ph) {
    const std::vector<uint32_t> &idx = s.ops_of[ph];
    const uint64_t G = std::min<uint64_t>(groups[ph], idx.size());
    for (uint64_t g = 0; g < G; ++g) {
      const uint32_t lo = (uint32_t)(g * idx.size() / G), hi = (uint32_t)((g + 1) * idx.size() / G);
      layers.push_back(Layer{idx[lo], idx[hi - 1] + 1, ph, lo, hi, (int64_t)(bpo[ph] * (hi - lo)), bpo[ph]});
    }
  }
  std::sort(layers.begin(), layers.end(), [](const Layer &a, const Layer &b) { return a.first < b.first; });
  layer_of.resize(n_ops);
  for (uint32_t li = 0; li < layers.size(); ++li)
    for (uint32_t i = layers[li].lo; i < layers[li].hi; ++i) layer_of[s.ops_of[layers[li].type][i]] = li;
}

// What generate_core works with; kept from one set to the next.
struct Work {
  std::vector<Layer> layers;
  std::vector<uint32_t> layer_of, order;
  std::vector<int64_t> excess;
  Entries entries;
  std::vector<uint8_t> taken;
  std::vector<Chosen> chosen;
  struct Cand { uint32_t at, n_mre; u128 key; };
  std::vector<Cand> list;
};

}  // namespace

// The generator proper.  Fills `items` in commit order and the counters of `res` that do not need a scan.
// Bound by the host's work on lists of some hundred elements.  Entries over the limit are kept as a bit map, so that how many a
// tensor can be away from, the last of them and their reduction cost what is left of the list and not the length of the trace; the
// tensors' stretches of it are found once for all sets.  A round ranks little more than the candidates that it commits, and in one
// that can commit none (it then accepts a late tensor) only the best is looked for.  Six sets, on one core: 700 operators, 67
// entries, 60 items 30 us (spans counted over all operators, candidates sorted whole: 105); 265 operators, 24 entries, with sets
// that run out of candidates 198 (647); one of 65,536 operators with 4,000 long spans 7.4 ms (12.6).  The call of the first with
// its scans 56 us (98).
static int generate_core(uint64_t bpo, const Shared &s, Work &k, uint32_t n_ops, const ss_tensor_t *tensors, const ss_gen_params_t *params,
                         std::vector<ss_policy_item_t> &items, std::vector<ss_event_t> &pe, ss_gen_result_t *res) {
  uint64_t bpo3[3];
  for (int ph = 0; ph < 3; ++ph) bpo3[ph] = params->phase_bytes_per_op[ph] ? params->phase_bytes_per_op[ph] : bpo;
  std::vector<Layer> &layers = k.layers;
  std::vector<uint32_t> &layer_of = k.layer_of;
  build_layers(s, n_ops, params->g_fwd, params->g_bwd, bpo3, layers, layer_of);
  k.excess = s.excess;
  const uint32_t n_entries = (uint32_t)s.entry_op.size();
  k.entries.all(n_entries, n_entries > 4 * s.away.size());
  k.taken.assign(s.away.size(), 0);
  std::vector<Chosen> &chosen = k.chosen;
  chosen.clear();

  auto commit = [&](uint32_t at, uint32_t L_in, bool late) {
    const Shared::Away &a = s.away[at];
    const uint32_t t_in = layers[L_in].first, hi = s.before[t_in];
    layers[L_in].remaining -= (int64_t)a.size;
    for (uint32_t w = a.lo / 64; w * 64 < hi; ++w) {
      uint64_t here = k.entries.word[w], gone = 0;
      if (w == a.lo / 64) here &= ~0ull << a.lo % 64;
      if (hi - w * 64 < 64) here &= (1ull << hi % 64) - 1;
      int64_t *const excess = k.excess.data() + (size_t)w * 64;
      if (here == ~0ull)
        for (uint32_t b = 0; b < 64; ++b) gone |= (uint64_t)((excess[b] -= (int64_t)a.size) <= 0) << b;
      else
        for (uint64_t x = here; x; x &= x - 1) {
          const uint32_t b = (uint32_t)__builtin_ctzll(x);
          gone |= (uint64_t)((excess[b] -= (int64_t)a.size) <= 0) << b;
        }
      if (gone) k.entries.take(w, gone);
    }
    k.taken[at] = 1;
    chosen.push_back(Chosen{a.row, L_in, t_in, 0, late});
  };
  // pre-trigger swap-in (Sec. 4.3.1): the latest layer between the last entry and the use that has the time, or -1
  auto layer_in = [&](uint32_t at) -> int64_t {
    const Shared::Away &a = s.away[at];
    const int64_t last = k.entries.last(a.lo, a.hi);
    if (last < 0) return -1;
    const uint32_t L_use = layer_of[a.first_bwd], L_peak = layer_of[s.entry_op[(size_t)last]];
    for (int64_t L = (int64_t)L_use - 1; L > (int64_t)L_peak; --L)
      if (layers[(size_t)L].remaining > (int64_t)a.size) return L;
    return -1;
  };
  using Cand = Work::Cand;
  std::vector<Cand> &cl = k.list;
  auto above = [&](const Cand &x, const Cand &y) {
    if (x.key != y.key) return x.key > y.key;
    const Shared::Away &a = s.away[x.at], &b = s.away[y.at];
    if (a.size != b.size) return a.size > b.size;
    return a.id != b.id ? a.id < b.id : x.at < y.at;
  };
  while (k.entries.left) {                              // Algo. 2
    cl.clear();
    const bool whole = k.entries.left == n_entries;
    if (!whole) k.entries.count();
    uint32_t max_n = 0;
    uint64_t max_s = 0;
    for (uint32_t at = 0; at < s.away.size(); ++at) {
      const Shared::Away &a = s.away[at];
      if (k.taken[at] || a.size < params->min_bytes) continue;
      const uint32_t c = whole ? a.hi - a.lo : k.entries.rank(a.hi) - k.entries.rank(a.lo);
      if (!c) continue;
      cl.push_back(Cand{at, c, 0});
      max_n = std::max(max_n, c);
      max_s = std::max(max_s, a.size);
    }
    if (cl.empty()) return SS_E_INFEASIBLE;             // "Raise Error"
    for (Cand &c : cl)                                  // Eq. 2, scaled to integers
      c.key = (u128)c.n_mre * max_s * params->c_den + (u128)params->c_num * s.away[c.at].size * max_n;
    res->n_rounds++;

    size_t some = 0;                                    // until something is committed nothing changes: can anything be?
    while (some < cl.size() && layer_in(cl[some].at) < 0) ++some;
    if (some < cl.size()) {
      size_t ranked = 0;
      for (size_t i = 0; i < cl.size() && k.entries.left; ++i) {
        if (i == ranked) {                              // the next ones in order, as many again
          const size_t end = std::min(cl.size(), std::max<size_t>(16, 2 * ranked));
          if (end < cl.size()) std::nth_element(cl.begin() + ranked, cl.begin() + end, cl.end(), above);
          std::sort(cl.begin() + ranked, cl.begin() + end, above);
          ranked = end;
        }
        const int64_t L = layer_in(cl[i].at);
        if (L >= 0) commit(cl[i].at, (uint32_t)L, false);
      }
      continue;
    }
    const Cand *best = nullptr;                         // accept latency rather than stop
    uint32_t best_in = 0;
    for (const Cand &c : cl) {
      const Shared::Away &a = s.away[c.at];
      const uint32_t L_use = layer_of[a.first_bwd];
      const uint32_t L_in = std::max<uint32_t>(L_use ? L_use - 1 : 0, layer_of[a.last_fwd] + 1);
      if (L_in > L_use || (best && !above(c, *best))) continue;
      best = &c;
      best_in = L_in;
    }
    if (!best) return SS_E_INFEASIBLE;
    commit(best->at, best_in, true);
  }

  // SetFreeTime: swap-out completion in swap-out order (Sec. 4.3.2)
  std::vector<uint32_t> &order = k.order;
  order.resize(chosen.size());
  for (uint32_t i = 0; i < order.size(); ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
    const ss_tensor_t &a = tensors[chosen[x].row], &b = tensors[chosen[y].row];
    return a.last_fwd_use != b.last_fwd_use ? a.last_fwd_use < b.last_fwd_use : a.tensor_id < b.tensor_id;
  });
  for (uint32_t i : order) {
    Chosen &c = chosen[i];
    const ss_tensor_t &t = tensors[c.row];
    const uint32_t L0 = layer_of[t.last_fwd_use];
    const int64_t last = (int64_t)c.layer_in - 1;
    int64_t found = -1;
    for (int64_t L = L0; L <= last; ++L) {
      int64_t avail = layers[(size_t)L].remaining;
      if (L == (int64_t)L0) {
        // the swap-out starts right after the last forward use: of that use's own layer only the operators
        // that follow it can carry the transfer
        uint64_t after = 0;
        for (uint64_t op = (uint64_t)t.last_fwd_use + 1; op < layers[(size_t)L].end; ++op)
          after += layer_of[op] == (uint32_t)L;
        avail = std::min<int64_t>(avail, (int64_t)(layers[(size_t)L].bpo * after));
      }
      if (avail > (int64_t)t.nbytes) { found = L; break; }
    }
    if (found < 0) {
      found = std::max<int64_t>(L0, last);
      c.late = true;
    }
    layers[(size_t)found].remaining -= (int64_t)t.nbytes;
    const uint32_t end_op = layers[(size_t)found].end - 1;
    c.t_free = std::min<uint32_t>(std::max<uint32_t>(end_op, t.last_fwd_use + 1), c.t_in - 1);
  }

  items.clear();
  pe.clear();
  pe.reserve(2 * chosen.size());
  for (size_t i = 0; i < chosen.size(); ++i) {
    const Chosen &c = chosen[i];
    const ss_tensor_t &t = tensors[c.row];
    ss_policy_item_t p;
    std::memset(&p, 0, sizeof(p));
    p.ref_op = t.producer_op; p.out_slot = t.out_slot; p.tensor_id = t.tensor_id;
    p.flags = c.late ? SS_F_LATE : 0;
    p.t_out = t.last_fwd_use; p.t_free = c.t_free; p.t_in = c.t_in; p.t_use = t.first_bwd_use;
    p.nbytes = t.nbytes;
    items.push_back(p);
    res->bytes += t.nbytes;
    res->n_late += c.late;
    pe.push_back(ss_event_t{c.t_free, t.tensor_id, -(int64_t)t.nbytes});
    pe.push_back(ss_event_t{c.t_in, t.tensor_id, (int64_t)t.nbytes});
  }
  res->n_items = (uint32_t)chosen.size();
  std::stable_sort(pe.begin(), pe.end(), [](const ss_event_t &a, const ss_event_t &b) { return a.op_idx < b.op_idx; });
  return SS_OK;
}

extern "C" int ss_generate_policy(ss_ctx *ctx, const ss_op_t *ops, uint32_t n_ops, const ss_tensor_t *tensors,
                                  uint32_t n_tensors, const ss_event_t *ev, uint64_t n_ev, int64_t base,
                                  int64_t limit, const ss_gen_params_t *params, ss_policy_item_t *policy_out,
                                  uint32_t *n_policy, ss_gen_result_t *res) {
  return ss_guard([&]() -> int {
    uint32_t chosen = 0;
    return ss_generate_policy_best(ctx, ops, n_ops, tensors, n_tensors, ev, n_ev, base, limit, params, 1, policy_out,
                                   n_policy, &chosen, res);
  });
}

extern "C" int ss_generate_policy_best(ss_ctx *ctx, const ss_op_t *ops, uint32_t n_ops, const ss_tensor_t *tensors,
                                       uint32_t n_tensors, const ss_event_t *ev, uint64_t n_ev, int64_t base,
                                       int64_t limit, const ss_gen_params_t *params, uint32_t n_params,
                                       ss_policy_item_t *policy_out, uint32_t *n_policy, uint32_t *chosen,
                                       ss_gen_result_t *res) {
  return ss_guard([&]() -> int {
    if (!ctx || !params || !n_params || !n_policy || !chosen || !res || (n_ops && !ops) || (n_tensors && !tensors))
      return SS_E_INVAL;
    if (*n_policy && !policy_out) return SS_E_INVAL;
    const uint64_t bpo = ctx->cfg.link_bytes_per_op;
    if ((u128)bpo * (n_ops + 1ull) >= ((u128)1 << 62)) return SS_E_INVAL;
    for (uint32_t c = 0; c < n_params; ++c) {
      if (params[c].c_den == 0 || params[c].g_fwd == 0 || params[c].g_bwd == 0) return SS_E_INVAL;
      for (int ph = 0; ph < 3; ++ph)
        if ((u128)params[c].phase_bytes_per_op[ph] * (n_ops + 1ull) >= ((u128)1 << 62)) return SS_E_INVAL;
    }
    std::memset(res, 0, sizeof(*res));

    // memory without swaps -> memory reduction list (Sec. 4.2)
    std::vector<int64_t> per_op(n_ops);
    ss_scan_result_t sr;
    int rc = ss_timeline_scan(ctx, ev, n_ev, nullptr, 0, n_ops, base, limit, nullptr, per_op.data(), nullptr, &sr);
    if (rc != SS_OK) return rc;
    const int64_t peak_no_swap = sr.peak;

    struct Cand { std::vector<ss_policy_item_t> items; std::vector<ss_event_t> pe; ss_gen_result_t r; int rc; };
    std::vector<Cand> cands(n_params);
    std::vector<ss_event_t> all_pe;
    std::vector<uint64_t> pe_start(n_params + 1, 0);
    bool any = false;
    Shared shared;
    Work work;
    share(ops, n_ops, tensors, n_tensors, per_op, limit, shared);
    for (uint32_t c = 0; c < n_params; ++c) {
      std::memset(&cands[c].r, 0, sizeof(ss_gen_result_t));
      cands[c].rc = generate_core(bpo, shared, work, n_ops, tensors, &params[c], cands[c].items, cands[c].pe, &cands[c].r);
      if (cands[c].rc != SS_OK && cands[c].rc != SS_E_INFEASIBLE) return cands[c].rc;
      if (cands[c].rc != SS_OK) cands[c].pe.clear();
      any = any || cands[c].rc == SS_OK;
      all_pe.insert(all_pe.end(), cands[c].pe.begin(), cands[c].pe.end());
      pe_start[c + 1] = all_pe.size();
    }
    if (!any) return SS_E_INFEASIBLE;
    // what the release points really give: every candidate scanned with its own events, one launch
    std::vector<ss_scan_result_t> scans(n_params);
    rc = ss_timeline_scan_batch(ctx, ev, n_ev, all_pe.data(), pe_start.data(), n_params, n_ops, base, limit, nullptr,
                                scans.data());
    if (rc != SS_OK) return rc;
    int best = -1;
    for (uint32_t c = 0; c < n_params; ++c) {
      if (cands[c].rc != SS_OK) continue;
      cands[c].r.peak_no_swap = peak_no_swap;
      cands[c].r.peak_with_policy = scans[c].peak;
      cands[c].r.n_over_with_policy = scans[c].n_over;
      if (best < 0) { best = (int)c; continue; }
      const ss_gen_result_t &x = cands[c].r, &y = cands[best].r;
      // within the limit first, then fewer items that cost latency, then fewer bytes over the link
      const bool xf = x.n_over_with_policy == 0, yf = y.n_over_with_policy == 0;
      if (xf != yf) { if (xf) best = (int)c; continue; }
      if (!xf && x.n_over_with_policy != y.n_over_with_policy) {
        if (x.n_over_with_policy < y.n_over_with_policy) best = (int)c;
        continue;
      }
      if (x.n_late != y.n_late) { if (x.n_late < y.n_late) best = (int)c; continue; }
      if (x.bytes < y.bytes) best = (int)c;
    }
    const Cand &w = cands[(size_t)best];
    if (w.items.size() > *n_policy) return SS_E_CAPACITY;
    if (!w.items.empty()) std::memcpy(policy_out, w.items.data(), w.items.size() * sizeof(ss_policy_item_t));
    *n_policy = (uint32_t)w.items.size();
    *chosen = (uint32_t)best;
    *res = w.r;
    return SS_OK;
  });
}
