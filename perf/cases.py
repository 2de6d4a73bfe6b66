"""The work that a training program has this framework do, as cases that can be timed.

Every iteration of a swapped training run records its operator sequence, matches it against the sequence the
policy was made for (`ss_match_sequence`; `ss_align_sequence` where operators come and go), checks the memory
curve (`ss_timeline_scan`, `ss_timeline_scan_static` for callers that cannot allocate) and moves the policy's
tensors to pinned host memory and back (`ss_dispatch`).  Once per policy the generator runs
(`ss_generate_policy_best`).  The cases go through those entry points as a user's program calls them; all results
are whole numbers or bytes, so every comparison is exact.

Sizes: configuration 1 is a toy decoder (2 layers), 2 a 1.3B shape (hidden 2048, 24 layers), 3 / 4 a 7B shape
(hidden 4096, 32 layers; in 4 the sequence varies from iteration to iteration), 5 the small-tensor stress
(20,000 tensors, 100,000 memory events).  The long cases are what the default trace capacity takes (65,536
operators, 1,048,576 events) and iterations of many gradient-accumulation steps.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2509_11076_amd.binding as B
from paper_2509_11076_amd.executor import dispatch_points, run_iteration_dispatch
import workloads as W

ALIGN = 256                     # staging slots and arena blocks
MIB = 1 << 20


# ---- the cases -------------------------------------------------------------------------------------------------

def listed():
    return [
        # A scan enqueued on the program's own stream with everything on the device already (a serving loop, code
        # under graph capture), for the smallest trace: the toy decoder's 66 operators.
        dict(name="scan_device_toy", kind="scan", where="device", n_ops=66, n_tensors=62, n_swapped=12,
             timeline=True),
        # The scan of every iteration of a 1.3B training run: host arrays in and out, with the policy's events.
        dict(name="scan_host_1p3b", kind="scan", where="host", n_ops=700, n_tensors=699, n_swapped=168,
             timeline=True),
        # The small-tensor trace (100,000 events) with the 40,000 events of its whole swap set.
        dict(name="scan_device_small_tensors", kind="scan", where="device", n_ops=400, n_tensors=50000,
             n_swapped=20000, timeline=True),
        # The longest trace the default capacity holds, as the policy generator scans it (no timeline).
        dict(name="scan_host_longest", kind="scan", where="host", n_ops=65536, n_tensors=524287, n_swapped=10007,
             timeline=False),
        # Policy generation for the 1.3B shape at 90 % of its peak: six parameter sets, the best one kept.
        dict(name="generate_1p3b", kind="generate", family="flash", hidden=2048, layers=24, heads=16, seq=2048,
             limit_pct=90),
        # Re-anchoring in a varying 7B iteration: operators dropped and inserted, branch counts moving.
        dict(name="match_7b_varying", kind="match", layers=32, steps=1, branches=4, anchors=480, flags=0),
        # The same for an iteration of 16 accumulation steps, most of its forward operators anchored.
        dict(name="match_accumulated", kind="match", layers=32, steps=16, branches=4, anchors=8001, flags=0),
        # Aligning a varying 7B iteration with the reference one (the matcher's fourth level).
        dict(name="align_7b_varying", kind="align", layers=32, steps=1, branches=4, anchors=480),
        # The same for an iteration of 28 accumulation steps.
        dict(name="align_accumulated", kind="align", layers=32, steps=28, branches=4, anchors=8001),
        # One iteration's swaps of the toy decoder: 12 tensors of 64..256 KiB, one batch an operator.
        dict(name="swap_toy", kind="swap", route="auto", n_tensors=12, lo=64 << 10, hi=256 << 10, unit=64 << 10,
             group=1),
        # Swaps of many small ragged tensors, 100 to a batch: the copy kernel's case.
        dict(name="swap_small_tensors", kind="swap", route="auto", n_tensors=1000, lo=4096, hi=4 * MIB, unit=2,
             group=100),
        # Three layers of the 1.3B shape's tensors through the HBM rings.
        dict(name="swap_staged_1p3b", kind="swap", route="staged", n_tensors=42, lo=8 * MIB, hi=64 * MIB,
             unit=8 * MIB, group=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan", "scan", "match", "match", "align", "align", "swap", "swap", "generate"])
    if kind == "scan":
        where = rng.choice(["host", "device"])
        n_tensors = _log(rng, 40, 450000 if where == "host" else 90000)
        return dict(kind="scan", where=where, n_ops=_log(rng, 60, 60000), n_tensors=n_tensors,
                    n_swapped=_log(rng, 1, max(2, min(40000, n_tensors // 3))),
                    timeline=n_tensors < 100000 and rng.random() < 0.6)
    if kind == "match":
        layers, steps = rng.randint(2, 40), _log(rng, 1, 12)
        return dict(kind="match", layers=layers, steps=steps, branches=rng.randint(0, 6),
                    anchors=_log(rng, 5, 10 * layers * steps),
                    flags=rng.choice([0, 0, B.SS_MATCH_HISTOGRAM, B.SS_MATCH_ALIGN]))
    if kind == "align":
        layers, steps = rng.randint(2, 40), _log(rng, 1, 18)
        return dict(kind="align", layers=layers, steps=steps, branches=rng.randint(0, 6),
                    anchors=_log(rng, 5, 10 * layers * steps))
    if kind == "swap":
        route = rng.choice(["auto", "kernel", "engine", "staged"])
        if route == "staged":
            return dict(kind="swap", route=route, n_tensors=rng.randint(5, 40), lo=256 * rng.randint(1, 4000),
                        hi=rng.randint(4, 48) * MIB, unit=256, group=rng.randint(1, 5))
        return dict(kind="swap", route=route, n_tensors=_log(rng, 5, 250 if route == "engine" else 900),
                    lo=_log(rng, 64, 65536), hi=_log(rng, 1 << 18, 4 * MIB), unit=rng.choice([1, 2, 4]),
                    group=_log(rng, 1, 100))
    fam = rng.choice(["flash", "naive"])
    return dict(kind="generate", family=fam, hidden=1024 * rng.randint(1, 4), layers=rng.randint(4, 32), heads=16,
                seq=128 * rng.randint(4, 32), limit_pct=rng.randint(85, 95))


# ---- inputs ----------------------------------------------------------------------------------------------------

class _Ctx:
    """a library context that goes when its state does"""

    def __init__(self, **kw):
        cfg = B.ss_config_default()
        cfg.staging_bytes = 4096
        for k, v in kw.items():
            setattr(cfg, k, v)
        self.h = B.ss_create(cfg)

    def __del__(self):
        h, self.h = getattr(self, "h", None), None
        if h is not None:
            B.ss_destroy(h)


class _Staging:
    """the staging area as an array that keeps its context alive"""

    def __init__(self, ctx, nbytes):
        self.ctx = ctx
        at = B.ss_host_peek(ctx.h, 0, nbytes).ctypes.data
        self.__array_interface__ = dict(shape=(nbytes // 8,), typestr="<i8", data=(at, False), version=3)


def _events(op, tid, delta):
    ev = np.zeros(len(op), dtype=B.EVENT_DT)
    ev["op_idx"], ev["tensor_id"], ev["delta"] = op, tid, delta
    return ev


def _memory_trace(case, seed):
    """(events, policy events, base, budget): tensor lifetimes over an iteration, forward half then backward half.
    The first n_swapped tensors live from the forward into the backward half; most others are short-lived."""
    rng = np.random.default_rng(seed)
    n, t, k = case["n_ops"], case["n_tensors"], case["n_swapped"]
    half = n // 2
    nbytes = np.exp(rng.uniform(math.log(4096), math.log(4 * MIB), t)).astype(np.int64) // 4 * 4
    alloc = rng.integers(0, n, t)
    free = np.minimum(n - 1, alloc + rng.integers(0, 16, t))
    alloc[:k] = rng.integers(0, half, k)
    free[:k] = np.minimum(n - 1, n - 1 - alloc[:k] + rng.integers(0, 8, k))
    ids = np.arange(t)
    op = np.concatenate([alloc, free])
    delta = np.concatenate([nbytes, -nbytes])
    tid = np.concatenate([ids, ids])
    order = np.lexsort((tid, delta < 0, op))
    ev = _events(op[order], tid[order], delta[order])
    # released some operators after the last forward use, back some operators before the first backward one
    t_free = np.minimum(free[:k] - 1, alloc[:k] + rng.integers(0, max(1, half // 8), k))
    t_free = np.maximum(t_free, 0)
    t_in = np.minimum(free[:k], np.maximum(t_free + 1, half + rng.integers(0, max(1, half // 2), k)))
    op = np.concatenate([t_in, t_free])
    delta = np.concatenate([nbytes[:k], -nbytes[:k]])
    tid = np.concatenate([ids[:k], ids[:k]])
    order = np.lexsort((tid, delta < 0, op))
    pe = _events(op[order], tid[order], delta[order])
    base = int(rng.integers(1 << 20, 1 << 33))
    return ev, pe, base, base + int(nbytes[:k].sum()) // 4


def _operators(case, seed):
    """(ref, cur, anchors): the operator sequence of `steps` accumulation steps over a stack of decoder layers, and
    the same iteration with each operator dropped or preceded by a foreign one with probability 0.1 each and branch
    operators coming and going.  Layers share their keys, as call stacks without layer numbers do."""
    rng = np.random.default_rng(seed)
    layers, steps, br = case["layers"], case["steps"], case["branches"]
    # forward operators of a layer: (token, call stack, outputs); one has two outputs
    tok = np.array([1, 2, 2, 2, 3, 4, 3, 2, 5, 1, 2, 6, 2, 5])
    n_out = np.array([1, 1, 1, 1, 1, 2, 1, 1, 1, 1, 1, 1, 1, 1])
    stk = rng.integers(1, 1 << 32, len(tok) + 3, dtype=np.uint64)

    def sequence(branches):
        cols = [[], [], [], []]                            # token, stack, phase, outputs
        for s in range(steps):
            fwd = [(np.array([7]), stk[-1:], np.array([1]))]
            for layer in range(layers):
                b = branches[s * layers + layer]
                fwd.append((np.concatenate([tok[:10], np.full(b, 2), tok[10:]]),
                            np.concatenate([stk[:10], np.repeat(stk[-2:-1], b), stk[10:-3]]),
                            np.concatenate([n_out[:10], np.ones(b, dtype=np.int64), n_out[10:]])))
            fwd = [np.concatenate([f[i] for f in fwd]) for i in range(3)]
            for phase in (0, 1):
                d = 1 if phase == 0 else -1
                cols[0].append(fwd[0][::d] + 10 * phase)
                cols[1].append(fwd[1][::d])
                cols[2].append(np.full(len(fwd[0]), phase))
                cols[3].append(fwd[2] if phase == 0 else np.ones(len(fwd[0]), dtype=np.int64))
        t, s, p, o = (np.concatenate(c) for c in cols)
        ops = np.zeros(len(t), dtype=B.OP_DT)
        ops["op_token"], ops["stack_hash"], ops["n_out"] = t, s.astype(np.uint32), o
        ops["sig"] = 1 | (o.astype(np.uint32) << 8) | (p.astype(np.uint32) << 16)
        return ops

    ref = sequence(np.full(layers * steps, br))
    cur = sequence(np.minimum(2 * br, rng.integers(0, 2 * br + 1, layers * steps)))
    keep = rng.random(len(cur)) >= 0.1
    before = rng.random(len(cur)) < 0.1
    noise = np.zeros(len(cur), dtype=B.OP_DT)
    noise["op_token"] = 40 + rng.integers(0, 8, len(cur))
    noise["stack_hash"] = np.uint32(stk[-3] & 0xFFFFFFFF)
    noise["n_out"] = 1
    noise["sig"] = 2 | (1 << 8)
    both = np.stack([noise, cur], axis=1).reshape(-1)
    cur = np.ascontiguousarray(both[np.stack([before, keep], axis=1).reshape(-1)])
    fwd = np.nonzero(ref["sig"] >> 16 == 0)[0]
    anchors = np.zeros(min(case["anchors"], len(fwd)), dtype=B.ANCHOR_DT)
    anchors["ref_op"] = np.sort(rng.choice(fwd, len(anchors), replace=False))
    two = ref["n_out"][anchors["ref_op"]] == 2
    anchors["out_slot"] = np.where(two, rng.integers(0, 2, len(anchors)), 0)
    return ref, cur, anchors


def _tensor_sizes(case, seed):
    n, unit = case["n_tensors"], case["unit"]
    # the sizes are the model's; where the blocks lie and what they hold differ from run to run
    sizes = np.random.default_rng([n, case["lo"], case["hi"]])
    rng = np.random.default_rng(seed)
    raw = np.exp(sizes.uniform(math.log(case["lo"]), math.log(case["hi"]), n))
    nbytes = np.maximum(unit, np.rint(raw / unit).astype(np.int64) * unit)
    slot = (nbytes + ALIGN - 1) // ALIGN * ALIGN
    # blocks lie in the arena in random order; they come back to other blocks, needed in the reverse groups' order
    def place():
        order = rng.permutation(n)
        off = np.zeros(n, dtype=np.int64)
        off[order] = np.cumsum(slot[order]) - slot[order]
        return off
    return nbytes, slot, place(), place()


def _swap_arena(case, seed):
    nbytes, slot, off_out, off_in = _tensor_sizes(case, seed)
    span = int(slot.sum())
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    arena = torch.zeros(2 * span // 8, dtype=torch.int64, device="cuda")
    arena[:span // 8].random_(-2 ** 62, 2 ** 62, generator=g)
    return nbytes, slot, off_out, off_in + span, span, arena


def _prepare_swap(case, seed):
    nbytes, slot, off_out, off_in, span, arena = _swap_arena(case, seed)
    n, group = case["n_tensors"], case["group"]
    nb = (n + group - 1) // group
    tab = np.zeros(n, dtype=B.TENSOR_DT)
    i = np.arange(n)
    tab["tensor_id"], tab["dtype"], tab["nbytes"] = i, 1, nbytes
    tab["producer_op"] = tab["alloc_op"] = tab["last_fwd_use"] = i // group
    tab["out_slot"] = i % group
    tab["first_bwd_use"] = tab["free_op"] = 2 * nb - i // group          # last produced, first needed
    tab["dev_off"], tab["dev_off_in"] = off_out, off_in
    pol = np.zeros(n, dtype=B.POLICY_DT)
    pol["ref_op"], pol["out_slot"], pol["tensor_id"], pol["nbytes"] = i // group, i % group, i, nbytes
    path = dict(auto=B.SS_PATH_AUTO, kernel=B.SS_PATH_KERNEL, engine=B.SS_PATH_ENGINE,
                staged=B.SS_PATH_STAGED)[case["route"]]
    ctx = _Ctx(staging_bytes=span, link_bytes_per_op=1 << 40, copy_path=path, copy_path_in=path, max_ops=4096,
               max_events=4096)
    B.ss_bind(ctx.h, arena.data_ptr(), 2 * span, torch.cuda.current_stream().cuda_stream)
    B.ss_staging_fill(ctx.h, 0)
    ap = B.ss_apply_policy(ctx.h, pol, pol["ref_op"].astype(np.int32), tab)
    assert ap["n_kept"] == n and ap["staging_bytes"] == span
    return dict(kind="swap", ctx=ctx, arena=arena, n_ops=2 * nb + 1, points=dispatch_points(ap["actions"]),
                staging=np.asarray(_Staging(ctx, span)), back=arena[span // 8:])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "swap":
        return _prepare_swap(case, seed)
    if kind == "scan":
        ev, pe, base, budget = _memory_trace(case, seed)
        st = dict(kind="scan_" + case["where"], ctx=_Ctx(), ev=ev, pe=pe, n_ops=case["n_ops"], base=base,
                  budget=budget, timeline=case["timeline"])
        if case["where"] == "device":
            n, e = case["n_ops"], len(ev) + len(pe)
            st["d_ev"] = torch.from_numpy(ev.view(np.int64).copy()).cuda()
            st["d_pe"] = torch.from_numpy(pe.view(np.int64).copy()).cuda()
            st["d_tl"] = torch.zeros(e, dtype=torch.int64, device="cuda") if case["timeline"] else None
            st["d_per"] = torch.zeros(n, dtype=torch.int64, device="cuda")
            st["d_mre"] = torch.zeros(n, dtype=torch.int64, device="cuda")
            st["d_res"] = torch.zeros(ctypes.sizeof(B.ss_scan_result_t) // 4, dtype=torch.int32, device="cuda")
        return st
    if kind in ("match", "align"):
        ref, cur, anchors = _operators(case, seed)
        return dict(kind=kind, ctx=_Ctx(), ref=ref, cur=cur, anchors=anchors, flags=case.get("flags", 0))
    shape = W.ModelShape(case["family"], case["hidden"], case["layers"], case["heads"], case["seq"], 1, 4)
    tr = W.build_trace(shape, seed=seed, iteration=1, perturb=dict(seq_jitter=0.15))
    ops = np.zeros(tr.n_ops, dtype=B.OP_DT)
    ctx = _Ctx(link_bytes_per_op=8 * MIB)
    for i in range(tr.n_ops):
        ops[i] = B.ss_intern_op(ctx.h, tr.op_name[i], tr.op_stack[i], tr.op_dtype[i], len(tr.op_outputs[i]),
                                tr.op_phase[i])
    peak = B.ss_timeline_scan(ctx.h, tr.events, None, tr.n_ops, 0, 1 << 62, want_per_op=False)["peak"]
    sets = [dict(g_fwd=max(1, case["layers"] // div), g_bwd=max(1, case["layers"] // div), c_num=c, min_bytes=1 << 16)
            for div in (1, 2, 4) for c in (1, 4)]
    return dict(kind="generate", ctx=ctx, ops=ops, tensors=tr.tensors, events=tr.events,
                limit=peak * case["limit_pct"] // 100, sets=sets)


# ---- one pass --------------------------------------------------------------------------------------------------

def run(st):
    kind, ctx = st["kind"], st["ctx"].h
    if kind == "swap":
        run_iteration_dispatch(ctx, st["n_ops"], None, st["points"])
        return {"back": st["back"], "staging": st["staging"]}
    if kind == "scan_host":
        r = B.ss_timeline_scan(ctx, st["ev"], st["pe"], st["n_ops"], st["base"], st["budget"],
                               want_timeline=st["timeline"])
        return r
    if kind == "scan_device":
        tl = st["d_tl"]
        B.ss_timeline_scan_static(ctx, torch.cuda.current_stream().cuda_stream, st["d_ev"].data_ptr(), len(st["ev"]),
                                  st["d_pe"].data_ptr(), len(st["pe"]), st["n_ops"], st["base"], st["budget"],
                                  tl.data_ptr() if tl is not None else 0, st["d_per"].data_ptr(),
                                  st["d_mre"].data_ptr(), st["d_res"].data_ptr())
        return {"timeline": tl, "per_op": st["d_per"], "mre": st["d_mre"], "result": st["d_res"]}
    if kind == "match":
        return B.ss_match_sequence(ctx, st["ref"], st["cur"], st["anchors"], flags=st["flags"])
    if kind == "align":
        return B.ss_align_sequence(ctx, st["ref"], st["cur"], st["anchors"])
    pol, info, chosen = B.ss_generate_policy_best(ctx, st["ops"], st["tensors"], st["events"], 0, st["limit"],
                                                  st["sets"])
    rows = np.zeros((len(st["tensors"]), B.POLICY_DT.itemsize // 4), dtype=np.uint32)      # as many rows for any policy
    rows[:len(pol)] = pol.view(np.uint32).reshape(len(pol), -1)
    return {"policy": rows, "info": info, "chosen": chosen}


# ---- what a pass cannot do without -----------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "scan":
        e = 2 * (case["n_tensors"] + case["n_swapped"])
        return {"bytes": 16 * e + 16 * case["n_ops"] + (8 * e if case["timeline"] else 0), "flops": e + case["n_ops"]}
    if kind in ("match", "align"):
        n = 2 * case["steps"] * (case["layers"] * (14 + case["branches"]) + 1)
        k = case["anchors"]
        if kind == "match" and case["flags"] != B.SS_MATCH_ALIGN:
            return {"bytes": 32 * n + 13 * k, "flops": 6 * n}
        # the bit-vector recurrence: a word of 64 columns takes five operations a row
        return {"bytes": 32 * n + 4 * n + 13 * k, "flops": 5 * n * ((n + 63) // 64)}
    if kind == "swap":
        lo, hi, n = case["lo"], case["hi"], case["n_tensors"]
        mean = (hi - lo) / math.log(hi / lo) if hi > lo else lo
        return {"bytes": int(4 * n * mean), "flops": 0}    # read and written once in each direction
    n = case["layers"] * 28 + case["layers"] + 4
    t = case["layers"] * 30
    return {"bytes": 16 * n + 56 * t + 32 * t + 40 * t // 4, "flops": 6 * n * t // 4}


def tolerance(case):
    return "exact"


# ---- the same results from plain numpy -------------------------------------------------------------------------

def _exact_scan(case, seed):
    ev, pe, base, budget = _memory_trace(case, seed)
    n = case["n_ops"]
    op = np.concatenate([ev["op_idx"], pe["op_idx"]]).astype(np.int64)
    delta = np.concatenate([ev["delta"], pe["delta"]])
    cls = np.concatenate([np.where(ev["delta"] >= 0, 1, 2), np.where(pe["delta"] >= 0, 0, 3)])
    pos, net = np.zeros(n, dtype=np.int64), np.zeros(n, dtype=np.int64)
    np.add.at(net, op, delta)
    np.add.at(pos, op[delta >= 0], delta[delta >= 0])
    per = base + np.cumsum(net) - net + pos
    mre = np.maximum(0, per - budget)
    order = np.lexsort((np.arange(len(op)), cls, op))
    tl = base + np.cumsum(delta[order]) if case["timeline"] else None
    peak, final = int(per.max()), base + int(net.sum())
    arg, over = int(per.argmax()), int((mre > 0).sum())
    if case["where"] == "device":
        words = np.array([peak, final], dtype=np.int64).view(np.int32)
        return {"timeline": tl, "per_op": per, "mre": mre,
                "result": np.concatenate([words, np.array([arg, over, 1, 0], dtype=np.int32)])}
    return dict(timeline=tl, per_op=per, mre=mre, peak=peak, argpeak_op=arg, n_over=over, final=final, sorted=1)


def _align(ref, cur):
    """pairing of the longest common subsequence, read from the end: pair equal operators, else step back in cur if
    that loses nothing, else in ref; bit j of row i is 0 where the length grows from column j to j + 1"""
    rk = list(zip(ref["op_token"].tolist(), ref["stack_hash"].tolist(), ref["sig"].tolist()))
    ck = list(zip(cur["op_token"].tolist(), cur["stack_hash"].tolist(), cur["sig"].tolist()))
    n, m = len(rk), len(ck)
    full = (1 << m) - 1
    where = {}
    for j, key in enumerate(ck):
        where.setdefault(key, bytearray(m // 8 + 1))[j >> 3] |= 1 << (j & 7)
    mask = {key: int.from_bytes(b, "little") for key, b in where.items()}
    rows, v = [], full
    for key in rk:
        u = v & mask.get(key, 0)
        v = ((v + u) | (v - u)) & full
        rows.append(v.to_bytes(m // 8 + 1, "little"))
    pair = np.full(n, -1, dtype=np.int32)
    i, j = n, m
    while i and j:
        if rk[i - 1] == ck[j - 1]:
            i, j = i - 1, j - 1
            pair[i] = j
        elif rows[i - 1][(j - 1) >> 3] >> ((j - 1) & 7) & 1:
            j -= 1
        else:
            i -= 1
    return pair, len(where)


def _land_aligned(pair, cur, anchors):
    j = pair[anchors["ref_op"]]
    ok = (j >= 0) & (anchors["out_slot"] < cur["n_out"][j])
    return np.where(ok, j, -1).astype(np.int32), np.where(ok, B.SS_LEVEL_ALIGN, 255).astype(np.uint8)


def _land_keyed(ref, cur, anchors):
    """the operator of the same ordinal among those with the anchor's key, the key relaxed from (token, stack, sig)
    to (token, sig) to (token); the lowest anchor keeps a shared place"""
    keys = [lambda o: (o[0], o[1], o[2]), lambda o: (o[0], o[2]), lambda o: o[0]]
    rl, cl = [o.tolist() for o in ref], [o.tolist() for o in cur]
    ordinal, places = [], []
    for key in keys:
        seen, out = {}, []
        for o in rl:
            x = key(o)
            out.append(seen.get(x, 0))
            seen[x] = out[-1] + 1
        ordinal.append(out)
        at = {}
        for j, o in enumerate(cl):
            at.setdefault(key(o), []).append(j)
        places.append(at)
    idx, lvl, taken = [], [], set()
    for i, s in anchors.tolist():
        land, level = -1, 255
        for q, key in enumerate(keys):
            p = places[q].get(key(rl[i]), ())
            if ordinal[q][i] < len(p):
                j = p[ordinal[q][i]]
                if s < cl[j][3] and cl[j][2] & 0xFF == rl[i][2] & 0xFF:
                    land, level = j, q
                    break
        if land >= 0 and (land, s) in taken:
            land, level = -1, 255
        taken.add((land, s))
        idx.append(land)
        lvl.append(level)
    return np.array(idx, dtype=np.int32), np.array(lvl, dtype=np.uint8)


def _exact_match(case, seed):
    ref, cur, anchors = _operators(case, seed)
    a, b = cur["op_token"].astype(np.int64), ref["op_token"].astype(np.int64)
    if case["flags"] & B.SS_MATCH_HISTOGRAM:
        a, b = np.bincount(a, minlength=64), np.bincount(b, minlength=64)
    else:
        n = max(len(a), len(b))
        a, b = np.pad(a, (0, n - len(a))), np.pad(b, (0, n - len(b)))
    dot, na, nb = int((a * b).sum()), int((a * a).sum()), int((b * b).sum())
    similar = 20 * abs(len(ref) - len(cur)) < len(ref) and dot > 0 and 400 * dot * dot > 361 * na * nb
    if case["flags"] & B.SS_MATCH_ALIGN:
        idx, lvl = _land_aligned(_align(ref, cur)[0], cur, anchors)
    else:
        idx, lvl = _land_keyed(ref, cur, anchors)
    return dict(similar=similar, dot=dot, na=na, nb=nb, stage=0, stable_step=0, new_idx=idx, level=lvl,
                n_unmatched=int((idx < 0).sum()))


def exact(case, seed):
    kind = case["kind"]
    if kind == "scan":
        return _exact_scan(case, seed)
    if kind == "match":
        return _exact_match(case, seed)
    if kind == "align":
        ref, cur, anchors = _operators(case, seed)
        pair, n_keys = _align(ref, cur)
        idx, lvl = _land_aligned(pair, cur, anchors)
        lcs = int((pair >= 0).sum())
        return dict(ref_to_cur=pair, new_idx=idx, level=lvl, lcs=lcs, distance=len(ref) + len(cur) - 2 * lcs,
                    n_keys=n_keys, n_unmatched=int((idx < 0).sum()))
    if kind == "swap":
        nbytes, slot, off_out, off_in, span, arena = _swap_arena(case, seed)
        src = arena[:span // 8].cpu().numpy().view(np.uint8)
        staging, back = np.zeros(span, dtype=np.uint8), np.zeros(span, dtype=np.uint8)
        at = np.cumsum(slot) - slot                        # staging slots in swap-out order
        for i in range(len(nbytes)):
            piece = src[off_out[i]:off_out[i] + nbytes[i]]
            staging[at[i]:at[i] + nbytes[i]] = piece
            back[off_in[i] - span:off_in[i] - span + nbytes[i]] = piece
        return {"back": back.view(np.int64), "staging": staging.view(np.int64)}
    return None
