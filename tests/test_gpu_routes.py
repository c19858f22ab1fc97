"""GPU parity on each of the routes a step can take (marks as bits or bytes, all hops in one workgroup or a launch per hop): steps that
the caps cut short, and the degenerate shapes - bad seeds, no edges, ragged words and rows - at sizes that reach the hop launches, with the
route asserted."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2605_29346_amd import workloads as W
from paper_2605_29346_amd import zg
from gpu_util import agg_error, compare_blocks, compare_features, compare_truncated, run_and_compare, samples_in_one_workgroup, to_host_graph, truncated_blocks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    zg.lib()


@pytest.mark.parametrize("nodes,draws,batch,fanouts,hop", [
    (20_000, 500_000, 256, (6, 5, 4), 0),        # bytes all the way: the vertices hop 0 drops are found again by hop 1 ...
    (20_000, 500_000, 256, (6, 5, 4), 1),        # ... and those hop 1 drops by the last hop, whose entries carry tags
    (200_000, 4_000_000, 256, (6, 5, 4), 1),     # bits, then bytes in the last hop
    (3_000_000, 12_000_000, 256, (8, 5, 3), 1),  # bits all the way
    (60_000, 1_200_000, 300, (5, 4, 3, 2), 1),   # a hop and a half behind the cut
    (9000, 300_000, 40, (4, 3, 2), 1),           # all hops in one workgroup
])
@pytest.mark.parametrize("dim", [0, 5])
def test_a_cap_in_the_middle_leaves_a_consistent_step(oracle, nodes, draws, batch, fanouts, hop, dim):
    # what the caps drop has no row and col -1, also where a later hop finds it again; the step after it is exact
    g = W.rmat_graph(nodes, draws, 23)
    og = to_host_graph(oracle, g)
    feat = W.feature_table(nodes, dim, 3) if dim else None
    seeds = W.SeedPool(g, batch, 7).batch_for(0).numpy()
    full = og.sample_blocks(seeds, fanouts, 31)
    caps = list(full.n)
    caps[hop + 1] = (full.n[hop] + full.n[hop + 1]) // 2
    want = truncated_blocks(oracle, g, seeds, fanouts, 31, caps)
    deg = np.diff(g.offsets.numpy())
    small = np.concatenate([np.flatnonzero(deg == 0)[: batch - 12], np.flatnonzero(deg == 1)[:12]]).astype(np.int32)
    fits = truncated_blocks(oracle, g, small, fanouts, 32, caps)
    assert len(small) == batch and fits[0] == fits[1] and fits[0][1] > batch
    dropped = set(want[3][hop][1][want[3][hop][2] < 0].tolist())
    assert dropped & set(want[2].tolist())  # some are found again
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), fanouts, batch, zg.make_envelope(zg.ENV_EXPLICIT, node_caps=caps), feat_dim=dim)
    assert samples_in_one_workgroup(plan) == (nodes == 9000)
    if dim:
        plan.bind_features(feat.cuda())
    for rep in range(2):
        plan.step(torch.as_tensor(seeds).cuda(), 31)
        torch.cuda.synchronize()
        assert plan.step_status() == (2 * rep + 1, zg.FLAG_HOP_OVERFLOW(hop))
        compare_truncated(plan, want, f"rep {rep}")
        if dim:
            X_ref = oracle.gather(feat.numpy(), want[2].astype(np.int32))
            assert np.array_equal(plan.view_X()[: len(X_ref), :dim].cpu().numpy(), X_ref)
        # a step that fits: nothing of the cut one is left behind
        plan.step(torch.as_tensor(small).cuda(), 32)
        torch.cuda.synchronize()
        assert plan.step_status() == (2 * rep + 2, 0)
        compare_truncated(plan, fits, f"after rep {rep}")


@pytest.mark.parametrize("nodes,batch,cut,maps_differ", [
    (300_000, 1130, 0.5, True),   # the plan marks bits, its twin - whose caps allow more edges - bytes
    (300_000, 1130, 0.95, True),
    (300_000, 1600, 0.5, False),  # both bytes
    (100_000, 300, 0.5, False),   # both in one workgroup
])
def test_replayed_features_after_the_twins_step(oracle, nodes, batch, cut, maps_differ):
    # the plan's step is cut at the last hop, the twin redoes it over the shared id map, then the plan's own feature launches run
    # again: its outputs are rewritten with the same values and nothing else in the workspace changes
    g = W.rmat_graph(nodes, 20 * nodes, 29)
    feat = W.feature_table(nodes, 16, 3).cuda()
    og = to_host_graph(oracle, g)
    seeds = W.SeedPool(g, batch, 7).batch_for(0)
    ref = og.sample_blocks(seeds.numpy(), (3, 4), 5)
    caps = [0, ref.n[1], ref.n[1] + int(cut * (ref.n[2] - ref.n[1]))]
    dg = zg.Graph(g.offsets.cuda(), g.indices.cuda())
    plan = zg.Plan(dg, (3, 4), batch, zg.make_envelope(zg.ENV_EXPLICIT, flags=zg.PLAN_SAFE_TWIN, node_caps=caps), feat_dim=16)
    plan.bind_features(feat)
    own, worst = (dg.plan_query((3, 4), batch, zg.make_envelope(m, node_caps=caps)).scratch_bytes for m in (zg.ENV_EXPLICIT, zg.ENV_MAX))
    assert (worst - own > nodes) == maps_differ  # a map of bytes instead of bits
    plan.step(seeds.cuda(), 5)
    cut_step = plan.read_step()
    plan.step_safe(seeds.cuda(), 5)
    torch.cuda.synchronize()
    assert cut_step.flags == zg.FLAG_HOP_OVERFLOW(1) and cut_step.n == [batch, caps[1], caps[2]]
    before = plan.workspace.clone()
    plan.replay_features(0)
    plan.replay_features(1)
    torch.cuda.synchronize()
    assert torch.equal(plan.workspace, before)
    again, whole = plan.read_step(), plan.safe_view().read_step()
    compare_blocks(whole, ref, "twin")
    for got, want in zip([again.X, again.agg] + again.col, [cut_step.X, cut_step.agg] + cut_step.col):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("dim", [0, 8])
@pytest.mark.parametrize("batch", [300, 24])  # a launch per hop; all hops in one workgroup
@pytest.mark.parametrize("flags", [0, zg.PLAN_EAGER])
def test_a_queued_step_finds_its_own_inputs_prefetched(oracle, dim, batch, flags):
    # The last launch of a step copies the next step's inputs out of host memory if the host is ahead: what it leaves (the two words
    # behind the fallback word: valid, step number) must name the next step, not the one after it, although the same launch
    # also advances the step counter.
    g = W.rmat_graph(30_000, 600_000, 21)
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), (8, 6), batch, zg.make_envelope(zg.ENV_MAX, flags=flags), feat_dim=dim)
    assert samples_in_one_workgroup(plan) == (batch == 24)
    if dim:
        plan.bind_features(W.feature_table(30_000, dim, 4).cuda())
    pool, og, steps = W.SeedPool(g, batch, 2), to_host_graph(oracle, g), 40
    batches = [pool.batch_for(s).cuda() for s in range(steps)]
    words = plan._view(plan.out.d_active + 4, 2, torch.int32)
    seen = torch.full((steps, 2), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    torch.cuda._sleep(50_000_000)  # the device starts when all steps are queued
    for s in range(steps):
        plan.step(batches[s], 600 + s)
        seen[s].copy_(words)
    torch.cuda.synchronize()
    assert seen.cpu().tolist()[:-1] == [[1, s + 1] for s in range(steps - 1)] and int(seen[-1, 0]) == 0
    log = plan.view_log().cpu().numpy()
    for s in range(steps):
        ref = og.sample_blocks(batches[s].cpu().numpy(), (8, 6), 600 + s)
        assert log[s][0] == s and log[s][1] == 0 and list(log[s][2:5]) == ref.n and list(log[s][5:7]) == ref.E


@pytest.mark.parametrize("flags", [0, zg.PLAN_FUSED_INPUT])
def test_the_stop_watch_of_a_small_step_is_on_its_aggregation_alone(oracle, flags):
    # 1900 rows of 32768 floats and next to no edges: the frontier's copy moves twice the bytes of the aggregation
    nodes, dim, batch = 2000, 32768, 1900
    g = W.rmat_graph(nodes, 400, 3)
    feat = W.feature_table(nodes, dim, 4)
    table = feat.cuda()
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), (1,), batch, zg.make_envelope(zg.ENV_MAX, flags=flags), feat_dim=dim)
    assert samples_in_one_workgroup(plan)
    plan.bind_features(table)
    seeds = W.SeedPool(g, batch, 5).batch_for(0)
    ref = to_host_graph(oracle, g).sample_blocks(seeds.numpy(), (1,), 8)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(), b.record()
    times = {"step": [], 0: [], 1: []}
    for rep in range(12):
        plan.step_timed(seeds.cuda(), 8, a, b)
        torch.cuda.synchronize()
        times["step"].append(a.elapsed_time(b))
        if rep == 0:
            res = plan.read_step()
            compare_blocks(res, ref)
            X_ref = oracle.gather(feat.numpy(), ref.S)
            assert np.array_equal(res.X, X_ref[: res.X.shape[0]])
            assert agg_error(oracle, res.agg, oracle.aggregate_mean(ref.row_ptr[0], ref.col[0], X_ref), ref.row_ptr[0], ref.col[0], X_ref) <= 1e-5
        for which in (0, 1):
            a.record()
            plan.replay_features(which)
            b.record()
            torch.cuda.synchronize()
            times[which].append(a.elapsed_time(b))
    step, copy, mean = (min(times[k]) for k in ("step", 0, 1))
    assert step < mean + 0.5 * copy, (step, copy, mean)


def _plan(g, fanouts, batch, small, feat=None, **more):
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), fanouts, batch, zg.make_envelope(zg.ENV_MAX, **more), feat_dim=0 if feat is None else feat.shape[1])
    assert samples_in_one_workgroup(plan) == small
    if feat is not None:
        plan.bind_features(feat if feat.is_cuda else feat.cuda())
    return plan


@pytest.mark.parametrize("batch,small", [(30, True), (400, False), (1500, False)])  # (the last: two workgroups ingest the seeds)
def test_bad_seeds_on_either_route(oracle, batch, small):
    # flags, and no row for an id out of range; the clean step after it is exact
    g = W.rmat_graph(5000, 80_000, 6)
    plan, og = _plan(g, (4, 4), batch, small), to_host_graph(oracle, g)
    good = W.SeedPool(g, batch, 3).batch_for(0).numpy()
    for at in (0, batch // 2, batch - 1):
        for bad in (5000, -1, -2**31, 2**31 - 1):
            seeds = good.copy()
            seeds[at] = bad
            plan.step(torch.as_tensor(seeds).cuda(), 1)
            torch.cuda.synchronize()
            assert int(plan.view_counts()[3].cpu()[0]) == zg.FLAG_SEED_RANGE
            row_ptr = plan.view_block(0)[0].cpu().numpy()
            assert row_ptr[at + 1] == row_ptr[at] and int(plan.view_S()[at].item()) == -1
            plan.overflow_clear()
        seeds = good.copy()
        seeds[at] = good[(at + 1) % batch]
        plan.step(torch.as_tensor(seeds).cuda(), 1)
        torch.cuda.synchronize()
        assert int(plan.view_counts()[3].cpu()[0]) & zg.FLAG_SEED_DUP
        plan.overflow_clear()
        plan.step(torch.as_tensor(good).cuda(), 2)
        compare_blocks(plan.read_step(), og.sample_blocks(good, (4, 4), 2), f"after bad seeds at {at}")


def test_a_graph_without_edges_on_the_hop_launches(oracle):
    n = 1000
    g = W.Graph(n, torch.zeros(n + 1, dtype=torch.int32), torch.zeros(0, dtype=torch.int32))
    feat = W.feature_table(n, 8, 1)
    seeds = np.arange(300, 800, dtype=np.int32)
    plan = _plan(g, (8, 8), 500, False, feat)
    _, res, _ = run_and_compare(oracle, g, feat, seeds, (8, 8), 7, plan=plan)
    assert res.n == [500, 500, 500] and res.E == [0, 0] and np.all(res.agg == 0)


def test_a_single_seed_on_the_hop_launches(oracle):
    g = W.rmat_graph(300_000, 3_000_000, 2)  # (more vertices than one workgroup's bitmaps hold)
    feat = W.feature_table(300_000, 12, 1)
    deg = np.diff(g.offsets.numpy())
    plan, og = _plan(g, (5, 5, 5), 1, False, feat), to_host_graph(oracle, g)
    for v in (int(np.argmax(deg)), int(np.argmin(deg)), 299_999):
        run_and_compare(oracle, g, feat, np.array([v], dtype=np.int32), (5, 5, 5), 3, plan=plan, og=og)


def test_the_published_known_answer_on_the_hop_launches(oracle):
    # vertex 0 draws 0xe169c58d6627e8d5 / 2^64 at key 0, hop 0, slot 0 (the all-zero Philox input)
    n = 300_000
    for d in (5, 1000):
        off = np.full(n + 1, d, dtype=np.int64)
        off[0] = 0
        g = W.Graph(n, torch.as_tensor(off), torch.arange(1, d + 1, dtype=torch.int32))
        _, res, _ = run_and_compare(oracle, g, None, np.array([0], dtype=np.int32), (1,), 0, plan=_plan(g, (1,), 1, False))
        assert res.nbr_gid[0].tolist() == [((0xE169C58D6627E8D5 * d) >> 64) + 1]


@pytest.mark.parametrize("nodes,batch,fanouts", [
    (31, 31, (64,)), (32, 32, (64,)), (33, 33, (64,)),                            # every vertex a seed; one word, a word and a bit
    (95, 40, (64, 64)), (96, 40, (64, 64)), (97, 40, (64, 64)), (97, 50, (64, 63, 64)),
    (1023, 900, (5, 2)), (1025, 1025, (4, 2)),                                   # a ranking tile of 32 words, and one bit more
])
@pytest.mark.parametrize("flags", [0, zg.PLAN_REPLACE])
def test_ragged_words_on_the_hop_launches(oracle, nodes, batch, fanouts, flags):
    g = W.rmat_graph(nodes, 12 * nodes, nodes)
    feat = W.feature_table(nodes, 5, 1)
    plan, og = _plan(g, fanouts, batch, False, feat, flags=flags), to_host_graph(oracle, g)
    for s in range(2):
        seeds = np.random.RandomState(s).permutation(nodes)[:batch].astype(np.int32)
        run_and_compare(oracle, g, feat, seeds, fanouts, 11 + s, plan=plan, og=og, replace=bool(flags))


def test_more_steps_queued_than_the_mailbox_holds_on_the_hop_launches(oracle):
    g = W.rmat_graph(30_000, 600_000, 21)
    plan, og, pool, steps = _plan(g, (8, 4), 160, False), to_host_graph(oracle, g), W.SeedPool(g, 160, 2), 600
    batches = [pool.batch_for(s).cuda() for s in range(steps)]
    torch.cuda.synchronize()
    for s in range(steps):
        plan.step(batches[s], 9000 + s)
    torch.cuda.synchronize()
    assert plan.step_status() == (steps, 0)
    log = plan.view_log().cpu().numpy()
    for s in range(steps):
        ref = og.sample_blocks(batches[s].cpu().numpy(), (8, 4), 9000 + s)
        assert log[s][0] == s and log[s][1] == 0 and list(log[s][2:5]) == ref.n and list(log[s][5:7]) == ref.E, f"step {s}"


@pytest.mark.parametrize("dim", [1, 3, 4, 5, 7, 75, 102, 600])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_ragged_and_shifted_rows_through_the_closing_launchs_copy(oracle, dim, shift):
    # rows that start at any multiple of four bytes; the frontier's are copied by workgroups of 512 lanes beside the ranking
    g = W.rmat_graph(6000, 90_000, 3)
    feat, og = W.feature_table(6000, dim, 4), to_host_graph(oracle, g)
    seeds = W.SeedPool(g, 200, 2).batch_for(0).numpy()
    wide = torch.full((6000, dim + 5), 1e30, device="cuda")
    wide[:, shift: shift + dim] = feat.cuda()
    ref = og.sample_blocks(seeds, (6, 4), 11)
    X_ref = oracle.gather(feat.numpy(), ref.S)
    agg_ref = oracle.aggregate_mean(ref.row_ptr[-1], ref.col[-1], X_ref)
    for flags in (0, zg.PLAN_X_TWO_PASS, zg.PLAN_FUSED_INPUT):
        plan = _plan(g, (6, 4), 200, False, wide[:, shift: shift + dim], flags=flags)
        out = plan.out
        last = out.d_agg + 4 * ((out.node_cap[1] - 1) * out.ld_agg + (dim + 3) // 4 * 4) - plan.workspace.data_ptr()
        plan.workspace[last: last + 256] = 0xA5
        plan.step(torch.as_tensor(seeds).cuda(), 11)
        res = plan.read_step()
        compare_blocks(res, ref, f"flags {flags}")
        assert np.array_equal(res.X, X_ref[: res.X.shape[0]])
        assert agg_error(oracle, res.agg, agg_ref, ref.row_ptr[-1], ref.col[-1], X_ref) <= 1e-5
        assert bool((plan.workspace[last: last + 256] == 0xA5).all())


@pytest.mark.parametrize("nodes,draws,max_tickets,draw", [(70_000, 1_400_000, 0, False), (3_000_000, 12_000_000, 20, True)])
@pytest.mark.parametrize("flags", [0, zg.PLAN_EAGER, zg.PLAN_AUTO_FALLBACK])
def test_the_kind_of_the_tickets_does_not_depend_on_other_plans(oracle, nodes, draws, max_tickets, draw, flags):
    # drawn where a tile is longer than a word per lane, whichever plan was made first and on whatever handle
    g = W.rmat_graph(nodes, draws, 8)
    og = to_host_graph(oracle, g)
    off, idx = g.offsets.cuda(), g.indices.cuda()
    fanouts, batch = (7, 5), 2000
    pool = W.SeedPool(g, batch, 3)
    graphs = [zg.Graph(off, idx), zg.Graph(off, idx)]
    plans = [zg.Plan(graphs[k], fanouts, batch, zg.make_envelope(zg.ENV_MAX, flags=flags, max_tickets=max_tickets)) for k in (0, 0, 1)]
    assert not samples_in_one_workgroup(plans[0])
    for s in range(3):
        for plan in plans[1:]:  # (the first one does nothing)
            run_and_compare(oracle, g, None, pool.batch_for(s).numpy(), fanouts, 90 + s, plan=plan, og=og)
            assert (int(plan.view_log()[s][zg.LOG_STRIDE - 1]) > 0) == draw


@pytest.mark.parametrize("nodes,draws,hop", [(20_000, 500_000, 0), (20_000, 500_000, 1), (200_000, 4_000_000, 1)])
def test_totals_worked_out_where_a_cap_cuts_the_step(oracle, nodes, draws, hop):
    # two plans on two streams, every total that is not there at a look worked out: the tile in which the cap falls and those behind it too
    g = W.rmat_graph(nodes, draws, 23)
    og = to_host_graph(oracle, g)
    batch, fanouts = 256, (6, 5, 4)
    pool = W.SeedPool(g, batch, 7)
    batches = [pool.batch_for(s).numpy() for s in range(2)]
    caps = [og.sample_blocks(b, fanouts, 31).n for b in batches]
    for c in caps:
        c[hop + 1] = (c[hop] + c[hop + 1]) // 2
    want = [truncated_blocks(oracle, g, b, fanouts, 31, c) for b, c in zip(batches, caps)]
    dg, streams = zg.Graph(g.offsets.cuda(), g.indices.cuda()), [zg.new_stream() for _ in batches]
    plans = [zg.Plan(dg, fanouts, batch, zg.make_envelope(zg.ENV_EXPLICIT, node_caps=c, flags=zg.PLAN_IMPATIENT)) for c in caps]
    seeds = [torch.as_tensor(b).cuda() for b in batches]
    torch.cuda.synchronize()
    for rep in range(3):
        for _ in range(4):
            for plan, s, st in zip(plans, seeds, streams):
                plan.step(s, 31, st)
        torch.cuda.synchronize()
        for plan, w in zip(plans, want):
            assert plan.step_status() == (4 * rep + 4, zg.FLAG_HOP_OVERFLOW(hop))
            compare_truncated(plan, w, f"rep {rep}")


@pytest.mark.parametrize("dim", [0, 8])
@pytest.mark.parametrize("batch", [300, 24])  # a launch per hop; all hops in one workgroup
def test_a_step_recorded_into_the_callers_graph(oracle, dim, batch):
    # replays, each a step of the plan, between steps that are enqueued; one recording is never replayed and counts for nothing
    g = W.rmat_graph(30_000, 600_000, 21)
    feat = W.feature_table(30_000, 8, 4)
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), (8, 6), batch, zg.make_envelope(zg.ENV_MAX), feat_dim=dim)
    assert samples_in_one_workgroup(plan) == (batch == 24)
    if dim:
        plan.bind_features(feat.cuda())
    pool, og, stream = W.SeedPool(g, batch, 2), to_host_graph(oracle, g), torch.cuda.Stream()
    batches = [pool.batch_for(s).cuda() for s in range(3)]
    torch.cuda.synchronize()
    recorded = [torch.cuda.CUDAGraph() for _ in range(2)]
    for s, rec in enumerate(recorded):
        with torch.cuda.graph(rec, stream=stream):
            plan.step(batches[s], 70 + s, stream)
    assert plan.step_status() == (0, 0)
    steps = 0
    for r in range(4):
        for s in (1, 2):
            recorded[1].replay() if s == 1 else plan.step(batches[2], 72)
            steps += 1
            res = plan.read_step()
            ref = og.sample_blocks(batches[s].cpu().numpy(), (8, 6), 70 + s)
            compare_blocks(res, ref, f"replay {r}, batch {s}")
            if dim:
                compare_features(oracle, res, ref, feat.numpy(), f"replay {r}, batch {s}")
            assert plan.step_status() == (steps, 0) and plan.epoch() == steps
    plan.close()  # (waits for nothing that was not replayed)


@pytest.mark.parametrize("enqueued", [0, 1])  # without and with a finished step that was not recorded
def test_destroying_a_plan_waits_for_replays_of_its_steps(oracle, enqueued):
    g = W.rmat_graph(30_000, 600_000, 21)
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), (8, 6), 300, zg.make_envelope(zg.ENV_MAX))
    seeds, key, stream = W.SeedPool(g, 300, 2).batch_for(0), 70, torch.cuda.Stream()
    seeds_d, rec = seeds.cuda(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(rec, stream=stream):
        plan.step(seeds_d, key, stream)
    for _ in range(enqueued):
        plan.step(seeds_d, key)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(200_000_000)  # the replays are still ahead when the plan is closed
        for _ in range(3):
            rec.replay()
    assert not stream.query() and plan.step_status() == (enqueued, 0)
    plan.close()
    assert stream.query()
    ref = to_host_graph(oracle, g).sample_blocks(seeds.numpy(), (8, 6), key)
    assert np.array_equal(plan.view_S()[: ref.n[-1]].cpu().numpy(), ref.S) and int(plan.view_counts()[0][-1]) == ref.n[-1]


def test_replays_do_not_count_against_the_steps_in_flight(oracle):
    # 300 replays later the host still waits when 255 of its own steps are unfinished, and for these alone
    g = W.rmat_graph(30_000, 600_000, 21)
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), (8, 4), 24, zg.make_envelope(zg.ENV_MAX))
    seeds, key, stream = W.SeedPool(g, 24, 2).batch_for(0), 70, torch.cuda.Stream()
    seeds_d, rec, replays, steps = seeds.cuda(), torch.cuda.CUDAGraph(), 300, 300
    torch.cuda.synchronize()
    with torch.cuda.graph(rec, stream=stream):
        plan.step(seeds_d, key, stream)
    for _ in range(replays):
        rec.replay()
    torch.cuda.synchronize()
    assert plan.step_status() == (replays, 0)
    torch.cuda._sleep(50_000_000)
    for s in range(steps):
        plan.step(seeds_d, key)
    assert plan.step_status()[0] >= replays + steps - 255
    compare_blocks(plan.read_step(), to_host_graph(oracle, g).sample_blocks(seeds.numpy(), (8, 4), key))
    assert plan.step_status() == (replays + steps, 0)


_REFUSED_LAUNCHES = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
import torch
from paper_2605_29346_amd import workloads as W, zg

left = ctypes.c_int.in_dll(shim, "launches_until_failure")
g = W.rmat_graph(30_000, 600_000, 21)
dg, seeds = zg.Graph(g.offsets.cuda(), g.indices.cuda()), W.SeedPool(g, 300, 2).batch_for(0).cuda()
def status(call):
    try:
        call()
        return zg.OK
    except zg.ZgError as e:
        return e.status
for launched in (0, 1, 3):
    plan, stream = zg.Plan(dg, (8, 6), 300, zg.make_envelope(zg.ENV_MAX)), torch.cuda.Stream()
    torch.cuda.synchronize()
    step = lambda: plan.step(seeds, 70, stream)
    with torch.cuda.stream(stream):
        torch.cuda._sleep(200_000_000)  # what is enqueued is still ahead when the plan is closed
    left.value = launched
    assert status(step) == zg.EHIP and left.value == 0
    left.value = -1
    torch.zeros(1, device="cuda").add_(1)  # the error is the step's, not the caller's next launch's
    assert status(step) == (zg.ESTATE if launched else zg.OK)  # nothing of the step was enqueued: the plan goes on
    assert not stream.query()
    plan.close()
    assert stream.query()
print("all closed")
"""


def test_a_step_enqueued_in_part_is_waited_for_and_the_last(tmp_path):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    shim = tmp_path / "launch_shim.so"
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(root, "tests", "launch_shim.cpp"), "-o", str(shim), "-ldl"], check=True)
    run = subprocess.run([sys.executable, "-c", _REFUSED_LAUNCHES, str(shim)], cwd=root, timeout=100, capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout.strip() == "all closed", run.stderr[-2000:]


def test_a_step_that_replays_the_plans_graph_is_not_recorded(oracle):
    # refused with nothing enqueued: the caller's recording goes on, and the plan's next steps find their own inputs
    g = W.rmat_graph(30_000, 600_000, 21)
    feat = W.feature_table(30_000, 8, 4)
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), (8, 6), 300, zg.make_envelope(zg.ENV_MAX, flags=zg.PLAN_AUTO_FALLBACK), feat_dim=8)
    plan.bind_features(feat.cuda())
    pool, og, stream = W.SeedPool(g, 300, 2), to_host_graph(oracle, g), torch.cuda.Stream()
    batches = [pool.batch_for(s).cuda() for s in range(3)]
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(), b.record()
    mark = torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    rec = torch.cuda.CUDAGraph()
    with torch.cuda.graph(rec, stream=stream):
        mark += 1
        for refused in (lambda: plan.step(batches[0], 70, stream), lambda: plan.step_timed(batches[0], 70, a, b, stream)):
            with pytest.raises(zg.ZgError) as err:
                refused()
            assert err.value.status == zg.ESTATE
        mark += 1
    for s in (1, 2):
        rec.replay()
        plan.step(batches[s], 70 + s)
        ref, res = og.sample_blocks(batches[s].cpu().numpy(), (8, 6), 70 + s), plan.read_step()
        compare_blocks(res, ref, f"batch {s}")
        compare_features(oracle, res, ref, feat.numpy(), f"batch {s}")
        assert plan.step_status() == (s, 0) and plan.epoch() == s and float(mark) == 2 * s


@pytest.mark.parametrize("nodes,tickets", [
    (32 * 64 * 2, 4),        # closing tiles of 64 words: a lane expands 4 vertices
    (32 * 256 * 2, 4),       # ... 16
    (32 * 257 * 2 - 5, 4),   # 288 words: a vertex per lane, the last word ragged
    (32 * 512 * 2, 4),       # a word per lane, several batches of vertices to a tile
    (32 * 64 * 300 + 1, 0),  # 235 tiles at most: several looks back
])
@pytest.mark.parametrize("dim", [0, 8])  # marks without and with tags
def test_closing_tiles_of_any_width(oracle, nodes, tickets, dim):
    g = W.rmat_graph(nodes, nodes * 30, 31)
    feat = W.feature_table(nodes, dim, 4) if dim else None
    env, plan = zg.make_envelope(zg.ENV_MAX, max_tickets=tickets), None
    og = to_host_graph(oracle, g)
    for s in range(3):  # (marks a step leaves behind show in the next)
        seeds = np.random.RandomState(s).permutation(nodes)[:600].astype(np.int32)
        plan, res, _ = run_and_compare(oracle, g, feat, seeds, (9, 20), 40 + s, env=env, plan=plan, og=og, label=f"step {s}")
    assert not samples_in_one_workgroup(plan)


@pytest.mark.parametrize("dim,batch,tickets", [
    (256, 32767, 0), (256, 32768, 0),  # either side of 32 MB of frontier rows of 1 KB
    (259, 32389, 0),                   # rows that are no whole pieces
    (256, 33000, 2),                   # closing tiles of more than a word per lane
    (8, 32768, 0),                     # 1 MB of frontier rows: copied
])
def test_frontier_rows_the_last_hop_reaches_again(oracle, dim, batch, tickets):
    # sparse rows and a few popular neighbors: the frontier has rows that the hop reaches, once or from many edges, and rows that it does not
    nodes = 50_000
    g = W.rmat_graph(nodes, nodes * 6, 33)
    feat = W.feature_table(nodes, dim, 4)
    og, plan = to_host_graph(oracle, g), None
    for s in range(3):
        seeds = np.random.RandomState(s).permutation(nodes)[:batch].astype(np.int32)
        plan, res, ref = run_and_compare(oracle, g, feat, seeds, (3,), 50 + s, env=zg.make_envelope(zg.ENV_MAX, max_tickets=tickets), plan=plan, og=og,
                                         label=f"step {s}")
        rows = plan.view_X()[: res.n[1], :dim]
        X = rows.clone()
        rows[:] = 7
        plan.replay_features(1)  # the rows the aggregation writes are the same again, the others are the copy's
        torch.cuda.synchronize()
        written = (rows != 7).any(1)
        assert torch.equal(rows[written], X[written]) and bool(written[batch:].all())
        reached = np.isin(seeds, res.nbr_gid[0]) if dim >= 256 and 4 * dim * batch >= 32 << 20 else np.zeros(batch, bool)
        assert np.array_equal(written[:batch].cpu().numpy(), reached)


@pytest.mark.parametrize("dim,batch,by_aggregation", [
    (100, 419_430, False), (100, 419_431, True),  # either side of 160 MB of frontier rows of less than 512 bytes
    (127, 330_260, False), (127, 330_261, True),
    (128, 196_607, False), (128, 196_608, True),  # ... of 96 MB from there on
    (255, 98_689, False), (255, 98_690, True),
])
def test_the_frontier_from_which_reached_rows_are_not_copied(dim, batch, by_aggregation):
    nodes = 700_000
    g = W.rmat_graph(nodes, 3 * nodes, 35)
    table = torch.empty((nodes, dim), device="cuda").normal_()
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), (2,), batch, zg.make_envelope(zg.ENV_MAX), feat_dim=dim)
    plan.bind_features(table)
    for s in range(2):
        plan.step(torch.randperm(nodes, device="cuda")[:batch].int(), 60 + s)
        torch.cuda.synchronize()
        n, E = int(plan.view_counts()[0][1]), int(plan.view_counts()[1][0])
        S, X = plan.view_S()[:n].long(), plan.view_X()[:n, :dim]
        assert plan.step_status()[1] == 0 and torch.equal(X, table[S])
        X[:] = 9  # (further from zero than any entry of the table)
        plan.replay_features(1)
        torch.cuda.synchronize()
        written = (X != 9).any(1)
        reached = torch.isin(S[:batch], plan.view_block(0)[1][:E].long())
        assert bool(written[batch:].all()) and 0 < int(reached.sum()) < batch
        assert torch.equal(written[:batch], reached if by_aggregation else torch.zeros_like(reached)) and torch.equal(X[written], table[S][written])


_LARGE = dict(nodes=100_000, dim=512, batch=15_000, fanouts=(3, 4))  # two hops: more than 32 MB of frontier rows of 2 KB, a third of them reached again


def _large_frontier(oracle, steps):
    """Graph, its host copy, features and per step the seeds and the checker's blocks."""
    g = W.rmat_graph(_LARGE["nodes"], 8 * _LARGE["nodes"], 33)
    og, feat = to_host_graph(oracle, g), W.feature_table(_LARGE["nodes"], _LARGE["dim"], 4)
    seeds = [np.random.RandomState(s).permutation(_LARGE["nodes"])[: _LARGE["batch"]].astype(np.int32) for s in range(steps)]
    refs = [og.sample_blocks(x, _LARGE["fanouts"], 50 + s) for s, x in enumerate(seeds)]
    for r in refs:
        frontier = r.S[: r.n[1]]
        assert 4 * _LARGE["dim"] * (r.n[1] - 1000) > 32 << 20 and 0.2 < np.isin(frontier, r.nbr_gid[1]).mean() < 0.8
    return g, og, feat, seeds, refs


def _rows_written_by_the_aggregation(plan, n):
    """Which of X's first n rows a replay of the aggregation writes; it may not change any."""
    rows = plan.view_X()[:n, : _LARGE["dim"]]
    X = rows.clone()
    rows[:] = 7
    plan.replay_features(1)
    torch.cuda.synchronize()
    written = (rows != 7).any(1)
    assert torch.equal(rows[written], X[written])
    rows[:] = X
    return written.cpu().numpy()


@pytest.mark.parametrize("flags", [0, zg.PLAN_IMPATIENT])
def test_entries_are_relabeled_while_the_frontiers_get_their_tags(oracle, flags):
    # two hops: the closing launch relabels hop 0's edges from the entries to which other workgroups of it add tags
    g, og, feat, seeds, refs = _large_frontier(oracle, 4)
    plan = None
    for s, (x, ref) in enumerate(zip(seeds, refs)):
        plan, res, _ = run_and_compare(oracle, g, feat, x, _LARGE["fanouts"], 50 + s, env=zg.make_envelope(zg.ENV_MAX, flags=flags), plan=plan, og=og, label=f"step {s}")
        assert np.array_equal(_rows_written_by_the_aggregation(plan, ref.n[2]), np.isin(ref.S, ref.nbr_gid[1]))


@pytest.mark.parametrize("flags", [0, zg.PLAN_IMPATIENT])
@pytest.mark.parametrize("cut", [(0,), (1,), (0, 1)])  # hops
def test_reached_frontier_rows_where_a_cap_cuts_the_step(oracle, cut, flags):
    g, og, feat, seeds, refs = _large_frontier(oracle, 3)
    caps = [_LARGE["batch"]] + [min(r.n[h + 1] for r in refs) - 700 if h in cut else max(r.n[h + 1] for r in refs) for h in range(2)]
    table = feat.cuda()
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), _LARGE["fanouts"], _LARGE["batch"], zg.make_envelope(zg.ENV_EXPLICIT, node_caps=caps, flags=flags),
                   feat_dim=_LARGE["dim"])
    plan.bind_features(table)
    for s, x in enumerate(seeds):  # (marks a step leaves behind show in the next)
        want = truncated_blocks(oracle, g, x, _LARGE["fanouts"], 50 + s, caps)
        plan.step(torch.as_tensor(x).cuda(), 50 + s)
        torch.cuda.synchronize()
        assert plan.step_status()[1] == sum(zg.FLAG_HOP_OVERFLOW(h) for h in range(2) if want[1][h + 1] > caps[h + 1])
        compare_truncated(plan, want, f"step {s}")
        n, S = want[0], want[2]
        assert all((n[h + 1] == caps[h + 1]) for h in cut)
        assert torch.equal(plan.view_X()[: n[2], : _LARGE["dim"]], table[torch.as_tensor(S).cuda()]), f"step {s}: X"
        assert np.array_equal(_rows_written_by_the_aggregation(plan, n[2]), np.isin(S, want[3][1][1]))


@pytest.mark.parametrize("how", ["graph", "eager", "recorded"])  # the plan's own graph; launches; launches in the caller's graph
def test_reached_frontier_rows_of_a_step_that_the_twin_redoes(oracle, how):
    g, og, feat, seeds, refs = _large_frontier(oracle, 3)
    table = feat.cuda()
    caps = [0, max(r.n[1] for r in refs), sorted(r.n[2] for r in refs)[1]]  # one of the three steps does not fit
    assert sum(r.n[2] > caps[2] for r in refs) == 1
    flags = zg.PLAN_AUTO_FALLBACK | (0 if how == "graph" else zg.PLAN_EAGER)
    plan = zg.Plan(zg.Graph(g.offsets.cuda(), g.indices.cuda()), _LARGE["fanouts"], _LARGE["batch"], zg.make_envelope(zg.ENV_EXPLICIT, node_caps=caps, flags=flags),
                   feat_dim=_LARGE["dim"])
    plan.bind_features(table)
    twin, stream, batches, recorded = plan.safe_view(), torch.cuda.Stream(), [torch.as_tensor(x).cuda() for x in seeds], []
    torch.cuda.synchronize()
    for s, x in enumerate(batches if how == "recorded" else []):
        recorded.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(recorded[s], stream=stream):
            plan.step(x, 50 + s, stream)
    for rep in range(2):
        for s, ref in enumerate(refs):
            recorded[s].replay() if recorded else plan.step(batches[s], 50 + s)
            torch.cuda.synchronize()
            active = int(plan.view_active().item())
            assert active == (ref.n[2] > caps[2]) and plan.step_status() == (3 * rep + s + 1, zg.FLAG_HOP_OVERFLOW(1) if active else 0)
            res = (twin if active else plan).read_step()
            res.flags &= ~zg.FLAG_HOP_OVERFLOW(1)  # (the plan's sticky word)
            compare_blocks(res, ref, f"{rep}: step {s}")
            compare_features(oracle, res, ref, feat.numpy(), f"{rep}: step {s}")
