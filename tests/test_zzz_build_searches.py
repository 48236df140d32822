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


def _uneven(n, seed):
    """A quarter of the points in a small blob: its centres have many times the mean number of neighbours."""
    rng = np.random.default_rng(seed)
    p = rng.random((n, 3)) * 0.6
    p[: n // 4] = 0.3 + rng.normal(0.0, 0.03, (n // 4, 3))
    return p[rng.permutation(n)].astype(np.float32)


# outputs (0: all points), mode, plan order; with and without a grid (up to 8192 points a side and 2^23 pairs), one chunk of 4096
# candidates and two, one centre per wave of the search and several (from 16 384 centres on)
LONG = [(n, n_out, mode, spatial) for n, n_out in [(700, 0), (2896, 0), (3500, 0), (4097, 1000), (1000, 4097), (8192, 1024), (8193, 500), (16_500, 0), (16_500, 4000)]
        for mode, spatial in [("ball", False), ("ball", True), ("batched", False), ("voxel", False)]]


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_out,mode,spatial", LONG)
def test_lists_past_the_stride(n, n_out, mode, spatial):
    """Centres with many times the mean number of neighbours have a list behind the others; every list is complete."""
    import paper_2511_23227_amd as m
    p = _uneven(n, n + n_out)
    q = p if n_out == 0 else (p[:n_out].copy() if n_out <= n else _uneven(n_out, n))
    t, size = 3, np.float32(0.02 if mode == "voxel" else 0.04)
    cuts, ocuts = None, None
    if mode == "batched":                                  # the middle cloud is empty, the last begins in the second chunk
        at = n - n // 3
        cuts = np.array([0, at, at, n], np.int32)
        at = len(q) - len(q) // 3
        ocuts = cuts if n_out == 0 else np.array([0, at, at, len(q)], np.int32)
    ref = oracle.build_triplets_general(p, q, size, t, mode=oracle.MODE_VOXEL if mode == "voxel" else oracle.MODE_BALL,
                                        in_offsets=cuts, out_offsets=ocuts)
    of = np.bincount(ref[0], minlength=len(q))
    assert of.max() > max(32, 3 * len(ref[0]) / len(q))    # past a stride of twice the mean
    d = torch.from_numpy(p).cuda()
    dq = d if n_out == 0 else torch.from_numpy(q).cuda()
    off = torch.from_numpy(cuts).cuda() if cuts is not None else None
    oo = off if n_out == 0 else torch.from_numpy(ocuts).cuda() if cuts is not None else None
    flags = m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0)
    plans = []
    for test in (0, m.BUILD_TEST_WIDE_KEYS):               # with lists, and searched in each pass
        plans.append(_plan(m, len(p), len(q), t, len(ref[0]), flags))
        T = m.pcpp_build_triplets(d, dq, float(size), t, plan_flags=flags | test | (m.BUILD_VOXEL if mode == "voxel" else 0),
                                  capacity=len(ref[0]), buffers={"plan": plans[-1]}, in_offsets=off, out_offsets=oo)
        _same(T, ref)
    assert torch.equal(plans[0][256:], plans[1][256:])
    # too little room: the same count, and nothing written
    tri = {k: torch.full((len(ref[0]) - 1,), -7, dtype=torch.int32, device="cuda") for k in ("tri_o", "tri_i", "tri_k")}
    with pytest.raises(m.PcppError) as e:
        m.pcpp_build_triplets(d, dq, float(size), t, plan_flags=flags | (m.BUILD_VOXEL if mode == "voxel" else 0),
                              capacity=len(ref[0]) - 1, buffers=tri, in_offsets=off, out_offsets=oo)
    assert e.value.code == -2 and str(len(ref[0])) in str(e.value)
    torch.cuda.synchronize()
    assert all(int((v != -7).sum()) == 0 for v in tri.values())


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_out", [(2500, 0), (3500, 0), (3500, 800), (20_000, 0)])
@pytest.mark.parametrize("t", [1, 2, 3, 5])
def test_workspaces_of_every_size(n, n_out, t):
    """Lists behind the tables with and without a grid, with shorter strides, inside the tables of the smallest workspace
    (where the neighbours have room there), and none: the same triplets and plan."""
    import ctypes
    import paper_2511_23227_amd as m
    from paper_2511_23227_amd import binding as B
    L = m.library()
    p = _uneven(n, n + t)
    q = p[:n_out].copy() if n_out else p
    o, i, k, seg = oracle.build_triplets(p, q, np.float32(0.035), t)
    d = torch.from_numpy(p).cuda()
    dq = torch.from_numpy(q).cuda() if n_out else d
    least, most = L.pcpp_build_triplets_workspace_bytes(n, len(q), t), L.pcpp_build_triplets_workspace_bytes_for(n, len(q), t, len(o))
    flags = B.PLAN_FWD | B.PLAN_BWD_INPUT
    first = None
    for share in (0.0, 0.02, 0.1, 0.3, 0.6, 0.9, 0.999, 1.0):
        ws = torch.full((int(least + (most - least) * share),), 255, dtype=torch.uint8, device="cuda")
        tri = [torch.empty(len(o), dtype=torch.int32, device="cuda") for _ in range(3)]
        sg = torch.empty(t ** 3 + 1, dtype=torch.int64, device="cuda")
        plan = _plan(m, n, len(q), t, len(o), flags)
        got = ctypes.c_int64(0)
        rc = L.pcpp_build_triplets(B._ptr(d), n, B._ptr(dq), len(q), 0.035, t, *[B._ptr(x) for x in tri], len(o), B._ptr(sg), ctypes.byref(got),
                                   B._ptr(plan), plan.numel(), flags, B._ptr(ws), ws.numel(), B._stream())
        assert rc == 0, L.pcpp_last_error()
        torch.cuda.synchronize()
        assert got.value == len(o) and np.array_equal(sg.cpu().numpy(), seg)
        for a, b in zip(tri, (o, i, k)):
            assert np.array_equal(a.cpu().numpy(), b)
        first = plan if first is None else first
        assert torch.equal(first[256:], plan[256:])


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_out", [(0, 0), (0, 70), (70, 0), (1, 1), (64, 64), (2896, 2896), (2897, 2897), (8192, 1024), (700, 8256), (17_000, 17_000), (17_000, 4_032)])
@pytest.mark.parametrize("mode,t", [("ball", 1), ("ball", 3), ("batched", 2), ("voxel", 3), ("voxel", 1)])
def test_count_only(n, n_out, mode, t):
    """The number of triplets, with the smallest workspace, into pageable and pinned memory."""
    import ctypes
    import paper_2511_23227_amd as m
    from paper_2511_23227_amd import binding as B
    L = m.library()
    p = _uneven(n, n + t) if n else np.zeros((0, 3), np.float32)
    same = n == n_out
    q = p if same else _uneven(n_out, n) if n_out else np.zeros((0, 3), np.float32)
    size = np.float32(0.02 if mode == "voxel" else 0.04)
    cuts = ocuts = None
    if mode == "batched":
        cuts, ocuts = np.array([0, n // 3, n], np.int32), np.array([0, n_out // 3, n_out], np.int32)
    want = len(oracle.build_triplets_general(p, q, size, t, mode=oracle.MODE_VOXEL if mode == "voxel" else oracle.MODE_BALL,
                                             in_offsets=cuts, out_offsets=ocuts)[0]) if n and n_out else 0
    d = torch.from_numpy(p).cuda()
    dq = d if same else torch.from_numpy(q).cuda()
    off = torch.from_numpy(cuts).cuda() if cuts is not None else None
    oo = off if same else torch.from_numpy(ocuts).cuda() if cuts is not None else None
    ws = torch.full((L.pcpp_build_triplets_workspace_bytes(n, n_out, t),), 255, dtype=torch.uint8, device="cuda")
    word = torch.full((1,), -1, dtype=torch.int64, pin_memory=True)
    pinned = ctypes.cast(word.data_ptr(), ctypes.POINTER(ctypes.c_int64))
    for target in (ctypes.pointer(ctypes.c_int64(-1)), pinned):
        rc = L.pcpp_build_triplets_batched(B._ptr(d), n, B._ptr(dq), n_out, B._ptr(off), B._ptr(oo), 2 if cuts is not None else 1,
                                           float(size), t, None, None, None, 0, None, target, None, 0,
                                           m.BUILD_VOXEL if mode == "voxel" else 0, B._ptr(ws), ws.numel(), B._stream())
        assert rc == 0 and target[0] == want, (L.pcpp_last_error(), target[0], want)


@pytest.mark.gpu
@pytest.mark.parametrize("spatial", [False, True])
@pytest.mark.parametrize("blob,sparse,t", [(3000, 3000, 1), (3000, 3000, 3), (4300, 1000, 1), (4300, 1000, 3)])
def test_centres_past_the_list_of_a_small_block(blob, sparse, t, spatial):
    """Few outputs inside a blob and many in sparse surroundings: the fill takes blocks of 256 or 512 threads, whose list holds 2048
    or 4096 neighbours, and each output in the blob has more; in other tiles nothing of the kind."""
    import paper_2511_23227_amd as m
    rng = np.random.default_rng(blob + t)
    p = np.concatenate([rng.uniform(0.0, 0.05, (blob, 3)), rng.uniform(-1.0, 1.0, (5000, 3))]).astype(np.float32)
    q = np.concatenate([p[rng.choice(blob, 20, replace=False)], rng.uniform(-1.0, 1.0, (sparse, 3)).astype(np.float32)])
    q = np.concatenate([q[20:720], q[:20], q[720:]])                 # the twenty in one tile, or in two
    r = np.float32(0.1)
    ref = oracle.build_triplets(p, q, r, t)
    of = np.bincount(ref[0], minlength=len(q))
    load = len(ref[0]) / (len(q) / 64) * 2 / 3
    assert (of > (2048 if blob == 3000 else 4096)).sum() >= 20 and (load < 2000 if blob == 3000 else 2200 < load < 4000)
    flags = m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0)
    plans = []
    for test in (0, m.BUILD_TEST_SHORT_LISTS):
        plans.append(_plan(m, len(p), len(q), t, len(ref[0]), flags))
        T = m.pcpp_build_triplets(torch.from_numpy(p).cuda(), torch.from_numpy(q).cuda(), float(r), t, plan_flags=flags | test,
                                  capacity=len(ref[0]), buffers={"plan": plans[-1]})
        _same(T, ref)
    assert torch.equal(plans[0][256:], plans[1][256:])
