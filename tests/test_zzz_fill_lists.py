"""Triplet builds whose tiles of 64 centres hold more neighbours than the fill pass keeps on chip at a time (12 276 with 27
cells, 3 834 with 216): tiles in several parts, and single centres that are past it."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import assert_close, oracle_bwd_input, oracle_fwd

# points in a ball of the radius, outputs among them (0: all), t, what the sizes are for
CASES = [(700, 0, 3, "parts of 17 centres"), (300, 0, 6, "parts of 12 centres, 216 cells"), (12_500, 3, 3, "single centres"),
         (4_000, 70, 6, "single centres, 216 cells, a second tile of 6")]


@pytest.mark.gpu
@pytest.mark.parametrize("spatial", [False, True])
@pytest.mark.parametrize("n,n_out,t,what", CASES)
def test_tiles_past_the_list(n, n_out, t, what, spatial):
    import paper_2511_23227_amd as m
    rng = np.random.default_rng(n + t)
    p = rng.uniform(0.0, 0.57, (n, 3)).astype(np.float32)           # all within 1 of each other
    out = p[:n_out].copy() if n_out else p
    o, i, k, seg = oracle.build_triplets(p, out, np.float32(1.0), t)
    assert len(o) == n * len(out)
    d = torch.from_numpy(p).cuda()
    do = torch.from_numpy(out).cuda() if n_out else d
    T = m.pcpp_build_triplets(d, do, 1.0, t, capacity=len(o),
                              plan_flags=m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0))
    assert T.n_triplets == len(o) and np.array_equal(T.seg_offsets.cpu().numpy(), seg)
    for got, want in ((T.tri_o, o), (T.tri_i, i), (T.tri_k, k)):
        assert np.array_equal(got.cpu().numpy(), want)
    # the plan's own lists, through the two passes that read them
    c, K = 8, t ** 3
    x, dy = rng.standard_normal((n, c)).astype(np.float32), rng.standard_normal((len(out), c)).astype(np.float32)
    w = (rng.standard_normal((K, c, c)) / np.sqrt(K * c)).astype(np.float32)
    y = m.pcpp_mvmr_fwd(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), T)
    dx = m.pcpp_mvmr_bwd_input(torch.from_numpy(dy).cuda(), torch.from_numpy(w).cuda(), T)
    assert_close(y.cpu().numpy(), *oracle_fwd(x, w, o, i, k, len(out)), 1e-4, "y")
    assert_close(dx.cpu().numpy(), *oracle_bwd_input(dy, w, o, i, k, n), 1e-4, "dx")
