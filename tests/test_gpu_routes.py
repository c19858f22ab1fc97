"""GPU parity on the routes a step can take beyond the plain one: steps that the caps cut short, each at the route its sizes lead to
(marks as bits or bytes, all hops in one workgroup or a launch per hop)."""
import numpy as np
import pytest
import torch

from paper_2605_29346_amd import workloads as W
from paper_2605_29346_amd import zg
from gpu_util import compare_truncated, samples_in_one_workgroup, to_host_graph, truncated_blocks

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
