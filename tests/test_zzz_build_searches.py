"""Triplet builds whose passes search by themselves: without neighbour lists (clouds of 2^24 points, small workspaces), with
centres that have more neighbours than their list, with and without a grid."""
import numpy as np
import pytest
import torch

import oracle


def _same(T, ref):
    o, i, k, seg = ref
    assert T.n_triplets == len(o) and np.array_equal(T.seg_offsets.cpu().numpy(), seg)
    for got, want in ((T.tri_k, k), (T.tri_o, o), (T.tri_i, i)):
        assert np.array_equal(got.cpu().numpy(), want)


def _plan(m, n_in, n_out, t, capacity, flags):
    """A plan's buffer of zeros: what a build leaves unwritten compares equal."""
    return torch.zeros(m.library().pcpp_plan_bytes(n_in, n_out, t, capacity, flags), dtype=torch.uint8, device="cuda")


@pytest.mark.gpu
@pytest.mark.parametrize("spatial", [False, True])
@pytest.mark.parametrize("t,batched", [(5, False), (5, True), (6, False), (6, True)])
def test_both_sides_counted_without_lists(t, batched, spatial):
    """A cloud against itself without neighbour lists: one pass counts both sides, in two tables of counters that take 49 KB of
    LDS at 125 cells and 85 KB at 216."""
    import paper_2511_23227_amd as m
    rng = np.random.default_rng(10 * t + spatial)
    p = np.concatenate([rng.random((900, 3)), 0.5 + rng.normal(0.0, 0.02, (300, 3))]).astype(np.float32)
    cuts = np.array([0, 500, len(p)], np.int32) if batched else None
    ref = oracle.build_triplets_general(p, p, np.float32(0.1), t, in_offsets=cuts, out_offsets=cuts)
    d = torch.from_numpy(p).cuda()
    off = torch.from_numpy(cuts).cuda() if batched else None
    flags = m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0)
    plans = []
    for test in (m.BUILD_TEST_WIDE_KEYS, 0):
        plans.append(_plan(m, len(p), len(p), t, len(ref[0]), flags))
        T = m.pcpp_build_triplets(d, d, 0.1, t, plan_flags=flags | test, capacity=len(ref[0]), buffers={"plan": plans[-1]},
                                  in_offsets=off, out_offsets=off)
        _same(T, ref)
    assert torch.equal(plans[0][256:], plans[1][256:])
