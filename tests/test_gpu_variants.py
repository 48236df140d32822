"""GPU parity of the variants around the main path: the voxel (degraded) operator, batches of clouds, voxel-grid
down-sampling, and the decoder's up-sampling layer -- each against the oracle, bit for bit where integers are
concerned."""
import numpy as np
import pytest
import torch

import oracle
import scenes
from parity_util import TOL, assert_close, oracle_bwd_input, oracle_bwd_weight, oracle_fwd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pcpp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_23227_amd as m
    m.library()
    return m


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t.to(dtype) if dtype is not None else t


def same_triplets(T, ref):
    o, i, k, seg = ref
    assert T.n_triplets == len(o)
    assert np.array_equal(T.seg_offsets.cpu().numpy(), seg)
    assert np.array_equal(T.tri_k.cpu().numpy(), k)
    assert np.array_equal(T.tri_o.cpu().numpy(), o)
    assert np.array_equal(T.tri_i.cpu().numpy(), i)


def check_ops(m, T, ref, n_in, n_out, K, cin, cout, dt, rng, what):
    o, i, k, _ = ref
    x = rng.standard_normal((n_in, cin)).astype(np.float32)
    w = (rng.standard_normal((K, cout, cin)) / np.sqrt(K * cin)).astype(np.float32)
    dy = rng.standard_normal((n_out, cout)).astype(np.float32)
    tdt = torch.float32
    if dt == "bf16":
        x, w, dy, tdt = scenes.round_to_bf16(x), scenes.round_to_bf16(w), scenes.round_to_bf16(dy), torch.bfloat16
    r, sc = oracle_fwd(x, w, o, i, k, n_out)
    assert_close(m.pcpp_mvmr_fwd(dev(x, tdt), dev(w, tdt), T).cpu().numpy(), r, sc, TOL[dt], what + " fwd")
    r, sc = oracle_bwd_input(dy, w, o, i, k, n_in)
    assert_close(m.pcpp_mvmr_bwd_input(dev(dy, tdt), dev(w, tdt), T).cpu().numpy(), r, sc, TOL[dt], what + " bwd_input")
    r, sc = oracle_bwd_weight(x, dy, o, i, k, K)
    assert_close(m.pcpp_mvmr_bwd_weight(dev(x, tdt), dev(dy, tdt), T).cpu().numpy(), r, sc, TOL[dt], what + " bwd_weight")


@pytest.mark.parametrize("case", [
    dict(n_in=3000, n_out=3000, same=True, pitch=0.05, t=3, cin=32, cout=32, dt="f32", spatial=False),
    dict(n_in=2500, n_out=1200, same=False, pitch=0.08, t=3, cin=64, cout=128, dt="bf16", spatial=False),
    dict(n_in=10400, n_out=10400, same=True, pitch=0.02, t=5, cin=256, cout=256, dt="bf16", spatial=True),
    dict(n_in=900, n_out=1500, same=False, pitch=0.11, t=5, cin=12, cout=20, dt="f32", spatial=True),
    dict(n_in=700, n_out=700, same=True, pitch=0.2, t=1, cin=16, cout=16, dt="f32", spatial=False),
])
def test_voxel_operator(pcpp, case):
    """BUILD_VOXEL: triplets bit-exact against the oracle's voxel mode (points anywhere inside their voxels, several
    per voxel, negative coordinates, points exactly on voxel faces), and all three ops on them."""
    rng = np.random.default_rng(case["n_in"] * 7 + case["t"])
    pitch = float(np.float32(case["pitch"]))

    def cloud(n):
        p = rng.uniform(-0.5, 0.5, (n, 3))
        p[: n // 10] = np.round(p[: n // 10] / pitch) * pitch          # exactly on voxel faces (as far as fp32 allows)
        return p.astype(np.float32)
    pin = cloud(case["n_in"])
    pout = pin if case["same"] else cloud(case["n_out"])
    ref = oracle.build_triplets_general(pin, pout, pitch, case["t"], oracle.MODE_VOXEL)
    din = dev(pin)
    dout = din if case["same"] else dev(pout)
    flags = pcpp.PLAN_FWD | pcpp.PLAN_BWD_INPUT | pcpp.BUILD_VOXEL | (pcpp.PLAN_SPATIAL if case["spatial"] else 0)
    T = pcpp.pcpp_build_triplets(din, dout, pitch, case["t"], plan_flags=flags)
    same_triplets(T, ref)
    assert T.n_triplets > 0
    check_ops(pcpp, T, ref, len(pin), len(pout), case["t"] ** 3, case["cin"], case["cout"], case["dt"], rng, repr(case))
    with pytest.raises(pcpp.PcppError):
        pcpp.pcpp_build_triplets(din, dout, pitch, 4, plan_flags=flags)


def test_voxel_operator_is_sparse_voxel_convolution(pcpp):
    """One point per occupied voxel of a lattice with holes: the library's result equals torch's dense conv3d of the
    occupancy-masked volume at the occupied sites (the special case of Sec. 3.2, checked end to end on the GPU path)."""
    rng = np.random.default_rng(5)
    n, pitch, t, ci, co = 12, 0.1, 3, 32, 32
    occ = rng.random((n, n, n)) < 0.5
    vox = np.argwhere(occ)
    pts = ((vox + rng.uniform(0.05, 0.95, vox.shape)) * pitch).astype(np.float32)
    x = rng.standard_normal((len(pts), ci)).astype(np.float32)
    w = (rng.standard_normal((27, co, ci)) / 30).astype(np.float32)
    d = dev(pts)
    T = pcpp.pcpp_build_triplets(d, d, pitch, t, plan_flags=pcpp.PLAN_FWD | pcpp.BUILD_VOXEL)
    out = pcpp.pcpp_mvmr_fwd(dev(x), dev(w), T).cpu().numpy()
    vol = np.zeros((1, ci, n, n, n), np.float64)
    vol[0, :, vox[:, 0], vox[:, 1], vox[:, 2]] = x
    wd = torch.from_numpy(w.astype(np.float64).reshape(3, 3, 3, co, ci).transpose(3, 4, 0, 1, 2).copy())
    dense = torch.nn.functional.conv3d(torch.from_numpy(vol), wd, padding=1)[0].numpy()
    ref = dense[:, vox[:, 0], vox[:, 1], vox[:, 2]].T
    assert np.abs(out - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("mode,spatial", [("ball", False), ("ball", True), ("voxel", False)])
def test_batches(pcpp, mode, spatial):
    """Clouds that overlap in space, empty clouds, a cloud convolved with itself: triplets bit-exact against the oracle's
    batched construction, ops on the concatenated arrays."""
    rng = np.random.default_rng(12 + spatial)
    sizes_in, sizes_out = [1200, 0, 900, 40, 1500], [800, 30, 0, 40, 1500]
    cin_ = [rng.uniform(0, 1, (n, 3)).astype(np.float32) for n in sizes_in]
    cout_ = [rng.uniform(0, 1, (n, 3)).astype(np.float32) for n in sizes_out]
    cout_[3], cout_[4] = cin_[3], cin_[4]
    pin, pout = np.concatenate(cin_), np.concatenate(cout_)
    io = np.cumsum([0] + sizes_in).astype(np.int32)
    oo = np.cumsum([0] + sizes_out).astype(np.int32)
    size, t = 0.1, 3
    omode = oracle.MODE_BALL if mode == "ball" else oracle.MODE_VOXEL
    ref = oracle.build_triplets_general(pin, pout, size, t, omode, io, oo)
    flags = pcpp.PLAN_FWD | pcpp.PLAN_BWD_INPUT | (pcpp.BUILD_VOXEL if mode == "voxel" else 0) | \
        (pcpp.PLAN_SPATIAL if spatial else 0)
    T = pcpp.pcpp_build_triplets(dev(pin), dev(pout), size, t, plan_flags=flags, in_offsets=dev(io), out_offsets=dev(oo))
    same_triplets(T, ref)
    # fewer triplets than when the clouds see each other
    assert T.n_triplets < oracle.count_triplets(pin, pout, size, t) or mode == "voxel"
    check_ops(pcpp, T, ref, len(pin), len(pout), 27, 64, 64, "bf16", rng, f"batches {mode}")
    # the whole batch as one self-convolution (same arrays, same offsets): the one-pass count of both sides
    d = dev(pin)
    off = dev(io)
    T2 = pcpp.pcpp_build_triplets(d, d, size, t, plan_flags=flags, in_offsets=off, out_offsets=off)
    ref2 = oracle.build_triplets_general(pin, pin, size, t, omode, io, io)
    same_triplets(T2, ref2)
    check_ops(pcpp, T2, ref2, len(pin), len(pin), 27, 32, 32, "f32", rng, f"batches self {mode}")


def test_voxel_subsample_and_strided_and_upsampling_layers(pcpp):
    """Sec. 4.1: down-sampling keeps one original point per voxel (bit-exact against the oracle), the strided layer
    convolves onto those points, the decoder's up-sampling layer goes back to the original points (n_out > n_in)."""
    rng = np.random.default_rng(13)
    pts = np.concatenate([rng.uniform(-1, 1, (4000, 3)), rng.normal(0.2, 0.03, (1500, 3))]).astype(np.float32)
    d = dev(pts)
    for pitch in (0.05, 0.13, 0.5):
        kept = pcpp.pcpp_voxel_subsample(d, pitch).cpu().numpy()
        assert np.array_equal(kept, oracle.voxel_subsample(pts, pitch))
    assert pcpp.pcpp_voxel_subsample(torch.zeros((0, 3), device="cuda"), 0.1).numel() == 0
    pitch, r, t = 0.13, 0.25, 3
    kept = pcpp.pcpp_voxel_subsample(d, pitch)
    coarse = d[kept.long()].contiguous()
    cp = coarse.cpu().numpy()
    assert np.array_equal(cp, pts[kept.cpu().numpy()])                     # original coordinates, not voxel centres
    # strided (down) layer: fine -> coarse
    T = pcpp.pcpp_build_triplets(d, coarse, r, t)
    ref = oracle.build_triplets(pts, cp, np.float32(r), t)
    same_triplets(T, ref)
    check_ops(pcpp, T, ref, len(pts), len(cp), 27, 64, 128, "bf16", rng, "strided layer")
    # up-sampling layer: coarse -> fine
    T = pcpp.pcpp_build_triplets(coarse, d, r, t)
    ref = oracle.build_triplets(cp, pts, np.float32(r), t)
    same_triplets(T, ref)
    check_ops(pcpp, T, ref, len(cp), len(pts), 27, 128, 64, "bf16", rng, "up-sampling layer")
    # the scene generator's strided scene uses the same rule
    s = scenes.make_scene(4)
    g = pcpp.pcpp_voxel_subsample(dev(s.in_xyz), s.meta["pitch"]).cpu().numpy() if "pitch" in s.meta else None
    if g is not None:
        assert np.array_equal(s.in_xyz[g], s.out_xyz)
