"""Helpers shared by the GPU parity tests: run the HIP path through the C-ABI binding and compare
every output with the CPU checker on the same seeded inputs."""
import os
import re

import numpy as np
import torch

from paper_2605_29346_amd import zg

AGG_RTOL = 1e-5  # fp32 mean aggregation: |gpu - ref| <= 1e-5 * max(|ref|, mean over the row of |x|)


def to_host_graph(oracle, g):
    return oracle.Graph(g.offsets.cpu().numpy(), g.indices.cpu().numpy())


def compare_blocks(res, ref, label=""):
    """Bit-exact comparison of counts, vertex list and every hop's block CSR."""
    H = len(ref.E)
    assert res.flags == 0, f"{label}: status flags {res.flags:#x}"
    assert res.n == ref.n, f"{label}: n {res.n} != {ref.n}"
    assert res.E == ref.E, f"{label}: E {res.E} != {ref.E}"
    assert res.n_exact[1:] == ref.n[1:], f"{label}: n_exact"
    assert np.array_equal(res.S, ref.S), f"{label}: S differs"
    for h in range(H):
        assert np.array_equal(res.row_ptr[h], ref.row_ptr[h]), f"{label}: row_ptr[{h}]"
        assert np.array_equal(res.nbr_gid[h], ref.nbr_gid[h]), f"{label}: nbr_gid[{h}]"
        assert np.array_equal(res.col[h], ref.col[h]), f"{label}: col[{h}]"


def agg_error(oracle, got, ref_agg, row_ptr, col, X):
    """max over elements of |got - ref| / max(|ref|, mean_row |x|) (0/0 counts as 0)."""
    denom = np.maximum(np.abs(ref_agg), oracle.aggregate_mean(row_ptr, col, np.abs(X)))
    err = np.abs(got.astype(np.float64) - ref_agg.astype(np.float64))
    with np.errstate(divide="ignore", invalid="ignore"):
        rel = np.where(denom > 0, err / denom, np.where(err == 0, 0.0, np.inf))
    return float(rel.max()) if rel.size else 0.0


def compare_features(oracle, res, ref, feat_host, label=""):
    X_ref = oracle.gather(feat_host, ref.S)
    assert np.array_equal(res.X.view(np.uint32), X_ref.view(np.uint32)), f"{label}: gathered rows differ"
    agg_ref = oracle.aggregate_mean(ref.row_ptr[-1], ref.col[-1], X_ref)
    assert res.agg.shape == agg_ref.shape
    e = agg_error(oracle, res.agg, agg_ref, ref.row_ptr[-1], ref.col[-1], X_ref)
    assert e <= AGG_RTOL, f"{label}: aggregation error {e}"
    return e


def run_and_compare(oracle, g, feat, seeds, fanouts, key, *, env=None, plan=None, og=None, replace=False, label=""):
    """One step on the GPU (new plan unless given) against the checker; returns (plan, result, reference)."""
    dev_g = None
    if plan is None:
        dev_g = zg.Graph(g.offsets.cuda(), g.indices.cuda())
        flags = zg.PLAN_REPLACE if replace else 0
        env = env or zg.make_envelope(zg.ENV_MAX, flags=flags)
        plan = zg.Plan(dev_g, fanouts, len(seeds), env, feat_dim=0 if feat is None else feat.shape[1])
        if feat is not None:
            plan.bind_features(feat.cuda())
    og = og or to_host_graph(oracle, g)
    seeds_d = torch.as_tensor(np.asarray(seeds, dtype=np.int32)).cuda()
    plan.step(seeds_d, key)
    res = plan.read_step()
    ref = og.sample_blocks(np.asarray(seeds, dtype=np.int32), fanouts, key, with_replacement=replace)
    compare_blocks(res, ref, label)
    if feat is not None:
        compare_features(oracle, res, ref, feat.cpu().numpy(), label)
    return plan, res, ref


def samples_in_one_workgroup(plan):
    """Whether the plan's step samples all its hops in one workgroup (the rule zg_plan_info documents beside grid_sample, with the
    planner's own constants): asserted where a test is there for one of the two routes."""
    src = open(os.path.join(os.path.dirname(zg.__file__), "csrc", "zg_internal.h")).read()
    const = {k: int(re.search(rf"\b{k} = (\d+);", src).group(1)) for k in ("kSmallEdgesPerHop", "kSmallMaxWords")}
    H, per_hop = plan.num_hops, const["kSmallEdgesPerHop"]
    return sum(plan.info.edge_cap[h] for h in range(H)) <= per_hop * H - per_hop // 2 and -(-plan.graph.num_nodes // 32) <= const["kSmallMaxWords"]


def truncated_blocks(oracle, g, seeds, fanouts, key, caps):
    """What a step under node caps leaves, built row by row from the checker's sampled positions: a hop's new vertices beyond its
    cap are dropped (no row, col -1) and may be found again by a later hop.  Returns (n, n_exact, S, per hop (row_ptr, nbr, col))."""
    off, idx = g.offsets.cpu().numpy().astype(np.int64), g.indices.cpu().numpy()
    S, n, n_exact, blocks = [int(v) for v in seeds], [len(seeds)], [len(seeds)], []
    for h, F in enumerate(fanouts):
        row_ptr, nbr = [0], []
        for v in S:
            pos = oracle.sample_positions(key, h, v, int(off[v + 1] - off[v]), F)
            nbr += [int(idx[off[v] + p]) for p in pos]
            row_ptr.append(len(nbr))
        new = sorted(set(nbr) - set(S))
        n_exact.append(len(S) + len(new))
        S = S + new[: caps[h + 1] - len(S)]
        n.append(len(S))
        at = {v: i for i, v in enumerate(S)}
        blocks.append((np.array(row_ptr), np.array(nbr, dtype=np.int64), np.array([at.get(v, -1) for v in nbr])))
    return n, n_exact, np.array(S), blocks


def compare_truncated(plan, want, label=""):
    n, n_exact, S, blocks = want
    got_n, got_E, got_exact, _ = [t.cpu().numpy().tolist() for t in plan.view_counts()]
    assert got_n == n and got_exact == n_exact, f"{label}: n {got_n} {n}, exact {got_exact} {n_exact}"
    assert np.array_equal(plan.view_S()[: n[-1]].cpu().numpy(), S), f"{label}: S"
    for h, (row_ptr, nbr, col) in enumerate(blocks):
        got = [t.cpu().numpy() for t in plan.view_block(h)]
        assert got_E[h] == len(nbr), f"{label}: E[{h}]"
        assert np.array_equal(got[0][: len(row_ptr)], row_ptr), f"{label}: row_ptr[{h}]"
        assert np.array_equal(got[1][: len(nbr)], nbr), f"{label}: nbr[{h}]"
        assert np.array_equal(got[2][: len(nbr)], col), f"{label}: col[{h}]"
