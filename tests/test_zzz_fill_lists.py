"""Triplet builds whose tiles of 64 centres hold more neighbours than the fill pass keeps on chip at a time (8 192 in crowded
clouds): tiles in several parts, and single centres that are past it; and neighbour lists of every length."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import assert_close, oracle_bwd_input, oracle_fwd

# points in a ball of the radius, outputs among them (0: all), t, what the sizes are for
CASES = [(700, 0, 3, "parts of 11 centres"), (300, 0, 6, "parts of 27 centres, 216 cells"), (12_500, 3, 3, "single centres"),
         (4_000, 70, 6, "parts of 2 centres, 216 cells, a second tile of 6")]


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


@pytest.mark.gpu
@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("spatial,same", [(False, True), (False, False), (True, True), (True, False)])
@pytest.mark.parametrize("t", [2, 3, 5])
def test_workspace_between_the_sizes(t, spatial, same, batched):
    """Neighbour lists as the workspace has room for: none, inside the tables of the smallest, with shorter strides, as long as the
    capacity asks for; what has no list is searched again: the same triplets and plan."""
    import ctypes
    import paper_2511_23227_amd as m
    from paper_2511_23227_amd import binding as B
    L = m.library()
    rng = np.random.default_rng(7 * t + spatial)
    p = np.concatenate([rng.random((900, 3)) * 1.2, 0.5 + rng.random((300, 3)) * 0.1]).astype(np.float32)
    p = p[rng.permutation(len(p))]
    out = p if same else p[::3].copy()
    r = np.float32(0.2)
    cuts = [0, 500, len(p)] if batched else [0, len(p)]
    ocuts = cuts if same else [-(-c // 3) for c in cuts]
    o, i, k, seg = oracle.build_triplets_general(p, out, r, t, in_offsets=np.array(cuts, np.int32), out_offsets=np.array(ocuts, np.int32))
    n_of = np.bincount(o, minlength=len(out))
    assert n_of.max() > 100 and (n_of < 27).any()
    d = torch.from_numpy(p).cuda()
    do = d if same else torch.from_numpy(out).cuda()
    off_i = torch.tensor(cuts, dtype=torch.int32, device="cuda") if batched else None
    off_o = off_i if same else torch.tensor(ocuts, dtype=torch.int32, device="cuda") if batched else None
    least, most = L.pcpp_build_triplets_workspace_bytes(len(p), len(out), t), L.pcpp_build_triplets_workspace_bytes_for(len(p), len(out), t, len(o))
    flags = B.PLAN_FWD | B.PLAN_BWD_INPUT | (B.PLAN_SPATIAL if spatial else 0)
    plans = []
    for size in (least, least + (most - least) // 4, most):
        ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")
        tri = [torch.empty(len(o), dtype=torch.int32, device="cuda") for _ in range(3)]
        sg = torch.empty(t ** 3 + 1, dtype=torch.int64, device="cuda")
        plan = torch.zeros(L.pcpp_plan_bytes(len(p), len(out), t, len(o), flags), dtype=torch.uint8, device="cuda")
        n = ctypes.c_int64(0)
        rc = L.pcpp_build_triplets_batched(B._ptr(d), len(p), B._ptr(do), len(out), B._ptr(off_i), B._ptr(off_o), len(cuts) - 1,
                                           float(r), t, *[B._ptr(x) for x in tri], len(o), B._ptr(sg), ctypes.byref(n), B._ptr(plan),
                                           plan.numel(), flags, B._ptr(ws), size, B._stream())
        assert rc == 0, L.pcpp_last_error()
        torch.cuda.synchronize()
        assert n.value == len(o) and np.array_equal(sg.cpu().numpy(), seg)
        for got, want in zip(tri, (o, i, k)):
            assert np.array_equal(got.cpu().numpy(), want)
        plans.append(plan.cpu().numpy()[256:])
    assert np.array_equal(plans[0], plans[2]) and np.array_equal(plans[1], plans[2])


def _lattice(n):
    g = np.stack(np.meshgrid(*[np.arange(18)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.float32)
    return g[np.random.default_rng(n).permutation(len(g))[:n]] * 0.25 + 1000.0


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["plain", "batched", "voxel", "lattice"])
@pytest.mark.parametrize("n", [1, 65, 2896, 2897, 4500])
def test_search_with_and_without_a_grid(n, mode):
    """Up to 2^23 pairs the search does without a grid (2896 points against themselves) and passes over far candidates by a test
    in 32 bits; a lattice far from the origin has neighbours at exactly the radius."""
    import paper_2511_23227_amd as m
    rng = np.random.default_rng(n)
    p = _lattice(n) if mode == "lattice" else rng.random((n, 3)).astype(np.float32) * (n / 400.0) ** (1 / 3)
    size = np.float32(0.5 if mode == "lattice" else 0.2 if mode != "voxel" else 0.11)
    cuts = [0, n // 3, n // 3, n] if mode == "batched" else None
    o, i, k, seg = oracle.build_triplets_general(p, p, size, 3, mode=oracle.MODE_VOXEL if mode == "voxel" else oracle.MODE_BALL,
                                                 in_offsets=cuts, out_offsets=cuts)
    d = torch.from_numpy(p).cuda()
    off = torch.tensor(cuts, dtype=torch.int32, device="cuda") if cuts else None
    T = m.pcpp_build_triplets(d, d, float(size), 3, capacity=len(o), in_offsets=off, out_offsets=off,
                              plan_flags=m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.BUILD_VOXEL if mode == "voxel" else 0))
    assert T.n_triplets == len(o) and np.array_equal(T.seg_offsets.cpu().numpy(), seg)
    for got, want in ((T.tri_o, o), (T.tri_i, i), (T.tri_k, k)):
        assert np.array_equal(got.cpu().numpy(), want)
