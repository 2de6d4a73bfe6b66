"""Small copy-kernel batches (64 KiB, or 256 KiB where the schedule releases them soon) are copied on the compute stream while
no other batch is outstanding: batches at and beyond these sizes mixed, released at once or late, swap-outs in either order,
one or several swap streams a direction, several iterations that end with and without a host wait, the compute stream lagging
behind the calls; bytes exact in staging and arena."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
K = 1 << 10


@pytest.fixture(scope="module")
def P():
    import paper_2509_11076_amd.binding as B
    return B


@pytest.mark.parametrize("flags_name", [None, "SS_CFG_TIMING", "SS_CFG_STALL_TIMING", "SS_CFG_MEMORY_MARKERS"])
@pytest.mark.parametrize("release", ["at once", "late", "reversed"])
@pytest.mark.parametrize("end", ["drain", "no wait"])
def test_small_and_large_batches_mixed(P, flags_name, release, end):
    import torch
    groups = [[1], [256 * K], [256 * K + 1], [16], [64 * K, 100 * K + 3], [1024 * K], [], [255 * K, K], [128 * K, 128 * K + 1],
              [300 * K], [5] * 9, [64 * K], [64 * K + 1], [32 * K, 32 * K], [3]]
    sizes = [n for g in groups for n in g]
    start = np.cumsum([0] + [len(g) for g in groups]).astype(np.uint32)
    slot = [(n + 255) // 256 * 256 for n in sizes]
    span, n = sum(slot), len(sizes)
    d_out, d_in = np.zeros(n, dtype=W.DESC_DT), np.zeros(n, dtype=W.DESC_DT)
    rng = np.random.default_rng(8)
    src, dst = np.zeros(n, dtype=np.int64), np.zeros(n, dtype=np.int64)
    for off in (src, dst):
        order = rng.permutation(n)
        off[order] = np.cumsum(np.array(slot)[order]) - np.array(slot)[order]
    h = np.cumsum(slot) - slot
    for i in range(n):
        d_out[i] = (src[i], h[i], sizes[i], i, 0)
        d_in[i] = (span + dst[i], h[i], sizes[i], i, 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    srcs = [torch.randint(0, 256, (span,), dtype=torch.uint8, device="cuda", generator=g) for _ in range(4)]
    arena = torch.zeros(2 * span, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    cfg = P.ss_config_default()
    cfg.staging_bytes = span
    cfg.copy_path = cfg.copy_path_in = P.SS_PATH_KERNEL
    cfg.flags = getattr(P, flags_name) if flags_name else 0
    ctx = P.ss_create(cfg)
    stream = torch.cuda.Stream()
    try:
        with torch.cuda.stream(stream):
            P.ss_bind(ctx, arena.data_ptr(), 2 * span, stream.cuda_stream)
            P.ss_staging_fill(ctx, 0)
            P.ss_load_schedule(ctx, d_out, start, d_in, start)
            got = []
            for it, s in enumerate(srcs):
                torch.cuda._sleep(2000000)                   # a millisecond or so behind the calls
                arena[:span].copy_(s)
                batches = list(range(len(groups)))
                for b in batches[::-1] if release == "reversed" else batches:
                    P.ss_swap_out(ctx, b)
                    if release == "at once":
                        for t in range(start[b], start[b + 1]):
                            P.ss_sync(ctx, P.SS_SYNC_FREE, t)
                for t in range(n):
                    P.ss_sync(ctx, P.SS_SYNC_FREE, t)
                arena.fill_(0x3C)
                for b in batches[::-1]:
                    P.ss_swap_in(ctx, b)
                    if b % 2:
                        for t in range(start[b], start[b + 1]):
                            P.ss_sync(ctx, P.SS_SYNC_WAIT_IN, t)
                for t in range(n):
                    P.ss_sync(ctx, P.SS_SYNC_WAIT_IN, t)
                got.append(arena.clone())
                last = it + 1 == len(srcs)
                torch.cuda._sleep(200000)                    # what follows the last batch there
                P.ss_sync(ctx, P.SS_SYNC_DRAIN if last or end == "drain" else P.SS_SYNC_ITERATION_END)
                if last or end == "drain":
                    want = np.zeros(span, dtype=np.uint8)
                    oracle.swap_out(s.cpu().numpy(), want, [tuple(int(x) for x in r) for r in d_out.tolist()])
                    assert np.array_equal(P.ss_host_peek(ctx, 0, span), want)
            torch.cuda.synchronize()
        for s, a in zip(srcs, got):
            staging, want = np.zeros(span, dtype=np.uint8), np.full(2 * span, 0x3C, dtype=np.uint8)
            oracle.swap_out(s.cpu().numpy(), staging, [tuple(int(x) for x in r) for r in d_out.tolist()])
            oracle.swap_in(want, staging, [tuple(int(x) for x in r) for r in d_in.tolist()])
            assert np.array_equal(a.cpu().numpy(), want)
        st = P.ss_get_stats(ctx)
        waits = 4 * sum(1 for x in groups if x)
        assert st["free_waits"] == waits and st["in_waits"] == waits and st["bytes_out"] == 4 * sum(sizes)
        if flags_name == "SS_CFG_TIMING":
            for dr in (0, 1):
                assert all(P.ss_batch_ms(ctx, dr, b)[0] >= 0 for b in range(len(groups)))
    finally:
        P.ss_destroy(ctx)


def test_a_batch_is_done_before_what_follows_it_on_the_compute_stream(P):
    import time
    import torch
    n = 64 * K
    arena = torch.randint(0, 256, (2 * n,), dtype=torch.uint8, device="cuda")
    want = arena[:n].cpu().numpy()
    d_out, d_in = np.zeros(1, dtype=W.DESC_DT), np.zeros(1, dtype=W.DESC_DT)
    d_out[0], d_in[0] = (0, 0, n, 0, 0), (n, 0, n, 0, 0)
    start = np.array([0, 1], dtype=np.uint32)
    cfg = P.ss_config_default()
    cfg.staging_bytes = n
    ctx = P.ss_create(cfg)
    try:
        P.ss_bind(ctx, arena.data_ptr(), 2 * n, torch.cuda.current_stream().cuda_stream)
        P.ss_load_schedule(ctx, d_out, start, d_in, start)
        torch.cuda.synchronize()
        P.ss_swap_out(ctx, 0)
        torch.cuda._sleep(1 << 30)                           # half a second
        t = time.time()
        while not P.ss_batch_done(ctx, 0, 0):
            assert time.time() - t < 0.2
        assert np.array_equal(P.ss_host_peek(ctx, 0, n), want)
        P.ss_sync(ctx, P.SS_SYNC_DRAIN)                      # waits for the batch alone
        assert time.time() - t < 0.2
        torch.cuda.synchronize()
    finally:
        P.ss_destroy(ctx)


def two_copies(P, torch, groups):
    """context, arena (random bytes, then as many zeros), start, sizes: `groups` of tensors leave from the first half and come
    back to the second"""
    sizes = [n for g in groups for n in g]
    start = np.cumsum([0] + [len(g) for g in groups]).astype(np.uint32)
    slot = [(n + 255) // 256 * 256 for n in sizes]
    span, at = sum(slot), np.cumsum([0] + slot)
    arena = torch.zeros(2 * span, dtype=torch.uint8, device="cuda")
    arena[:span] = torch.randint(0, 256, (span,), dtype=torch.uint8, device="cuda")
    cfg = P.ss_config_default()
    cfg.staging_bytes = span
    cfg.copy_path = cfg.copy_path_in = P.SS_PATH_KERNEL
    ctx = P.ss_create(cfg)
    P.ss_bind(ctx, arena.data_ptr(), 2 * span, torch.cuda.current_stream().cuda_stream)
    d_out, d_in = np.zeros(len(sizes), dtype=W.DESC_DT), np.zeros(len(sizes), dtype=W.DESC_DT)
    for i, n in enumerate(sizes):
        d_out[i], d_in[i] = (at[i], at[i], n, i, 0), (span + at[i], at[i], n, i, 0)
    torch.cuda.synchronize()
    return ctx, arena, d_out, d_in, start, at


def unsettled(P, ctx):
    import ctypes
    f = P._lib.ss_swap_unsettled
    f.argtypes, f.restype = [ctypes.c_void_p], ctypes.c_uint32
    return f(ctx)


def test_a_late_release_counts_for_its_own_batch(P):
    """the streams are joined between a batch and its release; a larger batch issued in between is still on its way then, and a
    small swap-in of one of its tensors must not be copied ahead of it"""
    import torch
    ctx, arena, d_out, d_in, start, at = two_copies(P, torch, [[1024 * K], [96 << 20, 64 * K], [64 * K]])
    try:
        ins = np.array([0, 1], dtype=np.uint32)              # the second tensor of the large batch, by itself
        P.ss_load_schedule(ctx, d_out, start, d_in[2:3], ins, in_dep=[1])
        for late in (False, True):
            P.ss_swap_out(ctx, 0)
            assert unsettled(P, ctx) == 1
            P.ss_staging_fill(ctx, 0x77)                     # joins the swap streams
            assert unsettled(P, ctx) == 0
            P.ss_swap_out(ctx, 1)
            if late:
                P.ss_swap_out(ctx, 2)
            P.ss_sync(ctx, P.SS_SYNC_FREE, 0)
            assert unsettled(P, ctx) == 1 + late
            P.ss_swap_in(ctx, 0)
            P.ss_sync(ctx, P.SS_SYNC_WAIT_IN, 2)
            back = arena.clone()
            assert unsettled(P, ctx) == 1 + late
            P.ss_sync(ctx, P.SS_SYNC_FREE, 1)
            P.ss_sync(ctx, P.SS_SYNC_FREE, 2)                # the same batch again
            assert unsettled(P, ctx) == late
            P.ss_sync(ctx, P.SS_SYNC_DRAIN)
            assert unsettled(P, ctx) == 0
            half = len(back) // 2
            assert torch.equal(back[half + at[2]:half + at[3]], back[at[2]:at[3]])
            arena[half:].zero_()
    finally:
        P.ss_destroy(ctx)


def test_batches_that_are_never_released_or_empty(P):
    """an empty batch holds nothing up; one that is never released does until the host has waited for its iteration"""
    import torch
    ctx, arena, d_out, d_in, start, at = two_copies(P, torch, [[1024 * K], [], [64 * K], [512 * K]])
    try:
        P.ss_load_schedule(ctx, d_out, start, d_in, start)
        left_over = 0
        for it in range(6):
            leave = it in (1, 2)
            P.ss_swap_out(ctx, 0)
            P.ss_swap_out(ctx, 1)
            assert unsettled(P, ctx) == 1 + left_over
            P.ss_sync(ctx, P.SS_SYNC_FREE, 0)
            P.ss_swap_out(ctx, 2)                            # on the compute stream where nothing is left over
            assert unsettled(P, ctx) == (2 if left_over else 0)
            P.ss_sync(ctx, P.SS_SYNC_FREE, 1)
            P.ss_swap_out(ctx, 3)
            if not leave:
                P.ss_sync(ctx, P.SS_SYNC_FREE, 2)
            for b in range(4):
                P.ss_swap_in(ctx, b)
            for t in range(3):
                P.ss_sync(ctx, P.SS_SYNC_WAIT_IN, t)
            back = arena.clone()
            P.ss_sync(ctx, P.SS_SYNC_ITERATION_END)
            left_over = int(leave)
            assert unsettled(P, ctx) == left_over
            torch.cuda.synchronize()
            half = len(back) // 2
            assert torch.equal(back[half:], back[:half])
            arena[half:].zero_()
    finally:
        P.ss_destroy(ctx)


def scheduled(P, torch, sizes_of_op, bpo, streams=1, flags=0):
    """context with a schedule of ss_apply_policy: the tensors of each operator leave after it and come back before its mirror
    image, from the first half of the arena to the second; the link moves bpo bytes during an operator"""
    flat = [(op, n) for op, sizes in enumerate(sizes_of_op) for n in sizes]
    n_ops, n = 3 * len(sizes_of_op) + 40, len(flat)
    slot = [(x + 255) // 256 * 256 for _, x in flat]
    span = sum(slot)
    tab, pol = np.zeros(n, dtype=P.TENSOR_DT), np.zeros(n, dtype=P.POLICY_DT)
    order = np.random.default_rng(4).permutation(n)
    at = np.zeros(n, dtype=np.int64)
    at[order] = np.cumsum(np.array(slot)[order]) - np.array(slot)[order]
    for i, (op, size) in enumerate(flat):
        tab["tensor_id"][i], tab["dtype"][i], tab["nbytes"][i] = i, 1, size
        tab["producer_op"][i] = tab["alloc_op"][i] = tab["last_fwd_use"][i] = op
        tab["out_slot"][i] = pol["out_slot"][i] = sum(1 for o, _ in flat[:i] if o == op)
        tab["first_bwd_use"][i] = tab["free_op"][i] = n_ops - 1 - op
        pol["ref_op"][i], pol["tensor_id"][i], pol["nbytes"][i] = op, i, size
    tab["dev_off"], tab["dev_off_in"] = at, span + at
    cfg = P.ss_config_default()
    cfg.staging_bytes, cfg.link_bytes_per_op, cfg.flags = span, bpo, flags
    cfg.copy_path = cfg.copy_path_in = P.SS_PATH_KERNEL
    cfg.out_streams = cfg.in_streams = streams
    arena = torch.zeros(2 * span, dtype=torch.uint8, device="cuda")
    ctx = P.ss_create(cfg)
    P.ss_bind(ctx, arena.data_ptr(), 2 * span, torch.cuda.current_stream().cuda_stream)
    ap = P.ss_apply_policy(ctx, pol, pol["ref_op"].astype(np.int32), tab)
    assert ap["n_kept"] == n
    return ctx, arena, ap["actions"], n_ops, at, [x for _, x in flat]


@pytest.mark.parametrize("size,bpo,soon", [
    (64 * K, 1 << 40, True), (64 * K, 8 * K, False), (64 * K + 1, 1 << 40, True), (64 * K + 1, 16 * K, False),
    (256 * K, 256 * K, True), (256 * K, 255 * K, False), (256 * K + 1, 1 << 40, True)])
def test_which_batches_are_copied_on_the_compute_stream(P, size, bpo, soon):
    """at most 64 KiB, or 256 KiB where at most one operator runs between the batch and its release or wait"""
    import torch
    ctx, arena, actions, n_ops, at, sizes = scheduled(P, torch, [[size]], bpo)
    try:
        op = {k: int(actions["op_idx"][actions["kind"] == k][0]) for k in range(4)}
        gaps = (op[P.SS_ACT_FREE] - op[P.SS_ACT_OUT], op[P.SS_ACT_WAIT_IN] - op[P.SS_ACT_IN])
        assert all((g <= 1) == soon for g in gaps)
        inline = size <= (256 * K if soon else 64 * K)
        for loaded in (False, True):                         # the same schedule without its actions: when it ends isn't known
            if loaded:
                start = np.array([0, 1], dtype=np.uint32)
                d_out, d_in = np.zeros(1, dtype=W.DESC_DT), np.zeros(1, dtype=W.DESC_DT)
                d_out[0], d_in[0] = (at[0], 0, size, 0, 0), (len(arena) // 2 + at[0], 0, size, 0, 0)
                P.ss_load_schedule(ctx, d_out, start, d_in, start)
                inline = size <= 64 * K
            P.ss_swap_out(ctx, 0)
            assert unsettled(P, ctx) == (0 if inline else 1)
            P.ss_sync(ctx, P.SS_SYNC_FREE, 0)
            P.ss_swap_in(ctx, 0)
            assert unsettled(P, ctx) == (0 if inline else 1)
            P.ss_sync(ctx, P.SS_SYNC_WAIT_IN, 0)
            P.ss_sync(ctx, P.SS_SYNC_DRAIN)
    finally:
        P.ss_destroy(ctx)


@pytest.mark.parametrize("flags_name", [None, "SS_CFG_TIMING", "SS_CFG_STALL_TIMING"])
@pytest.mark.parametrize("streams", [1, 3])
@pytest.mark.parametrize("bpo", [1 << 40, 200 * K])
def test_scheduled_batches(P, flags_name, streams, bpo):
    """whole iterations by their actions, most batches released soon or none of the larger ones"""
    import torch
    from paper_2509_11076_amd.executor import dispatch_points, run_iteration_dispatch
    groups = [[1], [256 * K], [16], [256 * K + 1], [200 * K], [64 * K, 100 * K + 3], [255 * K, K], [1024 * K], [128 * K, 128 * K],
              [300 * K], [5] * 9, [64 * K], [64 * K + 1], [130 * K], [3]]
    ctx, arena, actions, n_ops, at, sizes = scheduled(P, torch, groups, bpo, streams, getattr(P, flags_name) if flags_name else 0)
    try:
        points, half = dispatch_points(actions), len(arena) // 2
        last_out = int(actions["op_idx"][actions["kind"] >= P.SS_ACT_OUT].max())
        gen = torch.Generator(device="cuda")
        gen.manual_seed(5)
        for it in range(5):
            src = torch.randint(0, 256, (half,), dtype=torch.uint8, device="cuda", generator=gen)
            arena[:half].copy_(src)
            arena[half:].zero_()
            torch.cuda.synchronize()

            def run_op(i):
                torch.cuda._sleep(60000 if i % 3 else 3000)
                if i == last_out + 1:
                    arena[:half].fill_(0x3C)                 # every block has been released
            run_iteration_dispatch(ctx, n_ops, run_op, points,
                                   end=P.SS_SYNC_ITERATION_END if it % 2 else P.SS_SYNC_DRAIN)
            back, want = arena[half:].clone().cpu().numpy(), src.cpu().numpy()
            for a, n in zip(at, sizes):
                assert np.array_equal(back[a:a + n], want[a:a + n])
        P.ss_sync(ctx, P.SS_SYNC_DRAIN)
    finally:
        P.ss_destroy(ctx)


@pytest.mark.parametrize("sizes", [[64 * K, 16, 1000], [1024 * K, 300 * K], [64 * K, 1024 * K, 16, 300 * K]])
def test_an_iteration_captured_into_a_graph(P, sizes):
    """batches on the compute stream and on streams of their own, captured with the step; what the capture recorded is no event
    that a drain could wait for.  Replays with new bytes, eager iterations and drains in between"""
    import torch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx, arena, d_out, d_in, start, at = two_copies(P, torch, [[n] for n in sizes])
        half = len(arena) // 2
        try:
            P.ss_load_schedule(ctx, d_out, start, d_in, start)

            def iteration():
                for b in range(len(sizes)):
                    P.ss_swap_out(ctx, b)
                for t in range(len(sizes)):
                    P.ss_sync(ctx, P.SS_SYNC_FREE, t)
                arena[:half].fill_(0x3C)
                for b in range(len(sizes)):
                    P.ss_swap_in(ctx, b)
                for t in range(len(sizes)):
                    P.ss_sync(ctx, P.SS_SYNC_WAIT_IN, t)

            def check(step):
                src = torch.randint(0, 256, (half,), dtype=torch.uint8, device="cuda")
                arena[:half].copy_(src)
                arena[half:].zero_()
                step()
                torch.cuda.synchronize()
                for a, n in zip(at, sizes):
                    assert torch.equal(arena[half + a:half + a + n], src[a:a + n])
                    assert np.array_equal(P.ss_host_peek(ctx, int(a), n), src[a:a + n].cpu().numpy())
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                iteration()
            P.ss_sync(ctx, P.SS_SYNC_DRAIN)
            for _ in range(3):
                check(graph.replay)
                check(iteration)
                P.ss_sync(ctx, P.SS_SYNC_DRAIN)
                check(graph.replay)
        finally:
            P.ss_destroy(ctx)
