"""Working memory on a device without room: which tier a call runs on, what is
given back for what, and what captured plans and the caller see of it.  Host
code on a stand-in for the HIP runtime (tests/fake_hip)."""
import ctypes

import numpy as np
import pytest

from paper_2206_13574_amd import gwfa
from tests import fake_hip

PRUNED = dict(prune=gwfa.PRUNE_HEURISTIC, a_diff=50)
MIB = 1 << 20


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    return fake_hip.Host(fake_hip.compile_host(str(tmp_path_factory.mktemp("host"))))


@pytest.fixture
def H(host):
    """(host, context, graph) on an empty device of 288 GiB; tiers of 2^14,
    2^18, 2^20 and 2^22 pages."""
    host.reset()
    ctx = host.context(lanes=64, dir_log2_max=18, list_cap=1 << 17, dir_factor=256)
    g = host.graph(ctx)
    yield host, ctx, g
    host.lib.gwfa_graph_destroy(g)
    host.lib.gwfa_ctx_destroy(ctx)
    assert host.lib.fake_used() == 0


def test_tiers_in_order(H):
    """With room: exact calls on the configured tier, pruned ones on the small
    arenas, overflows on the next."""
    h, ctx, g = H
    assert h.align(ctx, g) == 0 and h.dirs() == [18]
    assert h.align(ctx, g, **PRUNED) == 0 and h.dirs() == [14]
    h.lib.fake_overflow(14, 7)
    h.lib.fake_overflow(18, 3)
    assert h.align(ctx, g, **PRUNED) == 0 and h.dirs() == [14, 18, 20]


@pytest.mark.parametrize("prune", [PRUNED, dict(prune=gwfa.PRUNE_LEARNED)])
def test_pruned_calls_run_where_the_small_arenas_do_not_fit(H, prune):
    """The rest of the device is the caller's: a pruned call, and a plan of
    one, take the configured tier, as exact calls do."""
    h, ctx, g = H
    assert h.align(ctx, g) == 0
    h.lib.fake_memory(h.lib.fake_used() + 64 * MIB)
    h.launches()
    assert h.align(ctx, g, **prune) == 0 and h.dirs() == [18]
    rc, p = h.plan(ctx, g, **prune)
    assert rc == 0
    assert h.lib.gwfa_plan_launch(p, None) == 0 and h.dirs() == [18]
    h.lib.fake_overflow(18, 2)
    h.lib.fake_memory(288 * fake_hip.GIB)
    assert h.lib.gwfa_plan_launch(p, None) == 0 and h.lib.gwfa_plan_finish(p, None) == 0
    assert h.dirs() == [18, 20]
    h.lib.gwfa_plan_destroy(p)
    assert h.lib.gwfa_last_error(ctx) == b"" and h.lib.fake_last_error() == 0


def test_pruned_calls_after_the_small_arenas_made_room(H):
    """An overflow whose tier fits only in the small arenas' place: the calls
    after it run on that tier."""
    h, ctx, g = H
    assert h.align(ctx, g, **PRUNED) == 0 and h.dirs() == [14]
    small = h.lib.fake_used()
    h.lib.fake_overflow(14, 5)
    assert h.align(ctx, g, **PRUNED) == 0
    both = h.lib.fake_used()
    assert h.dirs() == [14, 18]
    # the same on a device that holds one of the two
    h.lib.gwfa_ctx_config(ctx, 64, 0, 18, 1 << 17, 256)
    h.lib.fake_memory(both - small // 2)
    h.lib.fake_overflow(14, 0)
    assert h.align(ctx, g, **PRUNED) == 0 and h.dirs() == [14]
    h.lib.fake_overflow(14, 5)
    assert h.align(ctx, g, **PRUNED) == 0 and h.lib.fake_last_error() == 0
    assert [x[0] for x in h.launches()] == [14, 18]     # the first one's arenas are given back by now
    for _ in range(3):
        assert h.align(ctx, g, **PRUNED) == 0 and h.dirs() == [18]


@pytest.mark.parametrize("cfg", [dict(), dict(lanes=64), dict(lanes=256, dir_log2_max=18, list_cap=1 << 17),
                                 dict(lanes=64, dir_log2_max=18, list_cap=1 << 17), dict(lanes=64, dir_log2_max=19)])
def test_tiers_leave_the_caller_memory(host, cfg):
    """All tiers together take at most 85% of the memory free when the context
    is configured; the configured tier keeps its 60%."""
    host.reset()
    ctx = host.context(**cfg)
    g = host.graph(ctx)
    for d in range(14, 24):
        host.lib.fake_overflow(d, 1)
    before = host.lib.fake_used()
    assert host.align(ctx, g, n=100_000, **PRUNED) == 0
    ls = host.launches()
    assert len(ls) == 4 and all(x[5] for x in ls)
    assert host.lib.fake_used() - before <= 0.85 * 288 * fake_hip.GIB
    host.lib.gwfa_graph_destroy(g)
    host.lib.gwfa_ctx_destroy(ctx)


def _lists(h, ctx, g):
    return h.align(ctx, g, n=20_000_000)


def _host_batch(h, ctx, g):
    n = 1 << 20
    off, res = np.arange(n + 1, dtype=np.int64) * 100, np.zeros(n, gwfa.RESULT_DTYPE)
    return h.lib.gwfa_align_batch(ctx, g, n, np.full(n * 100, 65, np.uint8).ctypes.data_as(fake_hip._P),
                                  off.ctypes.data_as(fake_hip._P), np.zeros(n, np.int32).ctypes.data_as(fake_hip._P),
                                  ctypes.byref(gwfa.opts(traceback=False)), res.ctypes.data_as(fake_hip._P), None, 0,
                                  None)


def _cigar(h, ctx, g, n=1000, dist=3000):
    res = np.zeros(n, gwfa.RESULT_DTYPE)
    res["dist"], res["path_len"] = dist, 10
    off = np.arange(n + 1, dtype=np.int64) * 10_000
    b = h._buf.ctypes.data_as(fake_hip._P)
    return h.lib.gwfa_cigar_dev(ctx, g, n, b, off.ctypes.data_as(fake_hip._P), res.ctypes.data_as(fake_hip._P), b, b,
                                0, b, b, b, None)


def _grad(h, ctx, g):
    b = h._buf.ctypes.data_as(fake_hip._P)
    return h.lib.gwfa_mlp_grad_dev(ctx, b, 1, 8, b, b, 1.0, b, b, b, None)


def _graph(h, ctx, g):
    h.lib.gwfa_graph_destroy(h.graph(ctx, n_vtx=1_000_000))
    return 0


@pytest.mark.parametrize("call", [_lists, _host_batch, _cigar, _grad, _graph])
def test_small_arenas_give_way_to_other_calls(H, call):
    """With the device full, a call's own memory takes the place of the pruned
    runs' arenas; pruned calls then run on the configured tier."""
    h, ctx, g = H
    assert h.align(ctx, g) == 0 and h.align(ctx, g, **PRUNED) == 0 and h.dirs() == [18, 14]
    h.lib.fake_memory(h.lib.fake_used())
    assert call(h, ctx, g) == 0 and h.lib.fake_last_error() == 0
    h.lib.fake_memory(h.lib.fake_used())
    assert h.align(ctx, g, **PRUNED) == 0 and h.dirs()[-1] == 18


@pytest.mark.parametrize("by", ["finish", "call"])
def test_plans_outlive_their_arenas(H, by):
    """A pruned batch's plan whose arenas were given back, by its own finish or
    by another call, is launched again like any other."""
    h, ctx, g = H
    rc, p = h.plan(ctx, g, **PRUNED)
    assert rc == 0 and h.lib.gwfa_plan_launch(p, None) == 0 and h.lib.gwfa_plan_finish(p, None) == 0
    assert h.dirs() == [14]
    h.lib.fake_memory(180 * fake_hip.GIB)      # no room for the configured tier beside them
    if by == "finish":
        h.lib.fake_overflow(14, 3)
        assert h.lib.gwfa_plan_launch(p, None) == 0 and h.lib.gwfa_plan_finish(p, None) == 0
    else:
        assert h.align(ctx, g) == 0
    h.launches()
    for _ in range(2):
        assert h.lib.gwfa_plan_launch(p, None) == 0 and h.lib.gwfa_plan_finish(p, None) == 0
        assert h.dirs() == [18]
    # what ends a plan is what ended it before
    assert h.align(ctx, g, n=200_000) == 0 and h.lib.gwfa_plan_launch(p, None) == gwfa.ERR_ARG
    h.lib.gwfa_plan_destroy(p)


def test_cigars_run_in_the_room_there_is(H):
    """Distances of 3,000 ask for 18 MB a workgroup: the call takes as many
    workgroups as the device has room for, down to one."""
    h, ctx, g = H
    for room, lo, hi in ((64 * fake_hip.GIB, 500, 1000), (8 * fake_hip.GIB, 100, 500), (100 * MIB, 1, 6), (30 * MIB, 1, 1)):
        h.lib.gwfa_ctx_destroy(ctx)
        ctx.value = h.context().value
        h.lib.fake_memory(h.lib.fake_used() + room)
        assert _cigar(h, ctx, g) == 0 and lo <= h.lib.fake_cigar_groups() <= hi, (room, h.lib.fake_cigar_groups())
    h.lib.gwfa_ctx_destroy(ctx)
    ctx.value = h.context().value
    h.lib.fake_memory(h.lib.fake_used() + 10 * MIB)
    assert _cigar(h, ctx, g) == gwfa.ERR_NOMEM


def test_trace_records_count_tiers_from_the_configured_one(H):
    """The tier in a record's `attempt`: 0 on the configured tier, where dumps
    start, pruned or not, then 1 and 2."""
    h, ctx, g = H
    b = h._buf.ctypes.data_as(fake_hip._P)
    h.lib.fake_overflow(18, 5)
    h.lib.fake_overflow(20, 2)
    for o in (gwfa.opts(), gwfa.opts(**PRUNED)):
        assert h.lib.gwfa_align_dump_dev(ctx, g, 100, b, b, b, None, ctypes.byref(o), b, b, 0, b, b, 0, b, None) == 0
        assert [(x[0], x[4]) for x in h.launches()] == [(18, 0), (20, 1), (22, 2)]


@pytest.mark.parametrize("bytes_", [40_000, 160_000, 320_000])
def test_graphs_report_host_memory_that_is_not_there(H, bytes_):
    """10,000 vertices: edge offsets of 40 kB, records of 160 kB, label records
    of their targets of 320 kB."""
    h, ctx, g = H
    before = h.lib.fake_used()
    h.lib.fake_new_limit(bytes_)
    rc = h.graph(ctx, n_vtx=10_000)
    h.lib.fake_new_limit(-1)
    assert rc == gwfa.ERR_NOMEM and h.lib.fake_used() == before


def test_launch_arithmetic_at_the_largest_batch(host):
    """2^31 - 1 queries: the screen pass has a thread for each, and an empty
    take of any counter lies behind the last query."""
    n = 2**31 - 1
    assert host.lib.fake_screen_blocks(n) == 2**23 and host.lib.fake_screen_blocks(1) == 1
    assert host.lib.fake_screen_blocks(256) == 1 and host.lib.fake_screen_blocks(257) == 2
    for slot in range(8):
        last = (n - 1 - slot) // 8                  # the counter's last query
        assert host.lib.fake_queue_place(last, 8, slot) < n
        for empty in (1, 4096):
            assert host.lib.fake_queue_place(last + empty, 8, slot) >= n


@pytest.mark.parametrize("o,first", [
    (dict(prune=gwfa.PRUNE_HEURISTIC, a_diff=1024), 14), (dict(prune=gwfa.PRUNE_HEURISTIC, a_diff=1025), 18),
    (dict(prune=gwfa.PRUNE_LEARNED, keep_threshold=-12.0, mlp_gate=512, mlp_period=32), 14),
    (dict(prune=gwfa.PRUNE_LEARNED, keep_threshold=-12.5, mlp_gate=512, mlp_period=32), 18),
    (dict(prune=gwfa.PRUNE_LEARNED, keep_threshold=float("-inf")), 18),
    (dict(prune=gwfa.PRUNE_LEARNED, keep_threshold=-12.0, mlp_gate=513, mlp_period=32), 18),
    (dict(prune=gwfa.PRUNE_LEARNED, keep_threshold=-12.0, mlp_gate=512, mlp_period=33), 18)])
def test_first_tier_of_what_prunes_enough(H, o, first):
    h, ctx, g = H
    assert h.align(ctx, g, **o) == 0 and h.dirs() == [first]


def test_full_devices_are_not_asked_again_and_again(H):
    h, ctx, g = H
    assert h.align(ctx, g) == 0
    h.lib.fake_memory(h.lib.fake_used() + 64 * MIB)
    before = h.lib.fake_failed()
    for _ in range(5):
        assert h.align(ctx, g, **PRUNED) == 0
    assert h.lib.fake_failed() == before
