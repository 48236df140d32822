"""GPU parity of the kernels that take any channel counts, at the sizes where their tiles, remainders and dispatch lines
lie: channel counts around a lane's vector, a 16-channel tile and a chunk of source channels, point counts on either
side of the line between the split and the cooperative form, lists shorter than one batch per wave."""
import zlib

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


@pytest.mark.parametrize("n_in,n_out,r,t,shapes,dt", [
    (300, 200, 0.2, 3, ((1, 1), (2, 3), (3, 2), (7, 5), (16, 17), (31, 33), (33, 31)), "bf16"),
    (300, 200, 0.2, 3, ((1, 1), (2, 3), (3, 2), (7, 5), (16, 17), (31, 33), (33, 31), (65, 64)), "f32"),
    (400, 300, 0.2, 2, ((63, 65), (65, 63), (127, 129), (130, 96), (257, 48), (300, 270)), "bf16"),
    (400, 300, 0.2, 2, ((63, 65), (127, 129), (96, 260)), "f32"),
    (17000, 16300, 0.06, 3, ((20, 36), (15, 130), (128, 128)), "bf16"),       # split form one way, cooperative the other
    (16300, 17000, 0.06, 3, ((20, 36), (66, 15)), "f32"),
    (300, 66000, 0.15, 3, ((20, 32), (32, 17)), "f32"),                       # many centres with few neighbours
    (2000, 2000, 0.15, 6, ((64, 64), (40, 24)), "bf16"),                       # 216 cells
    (40, 1, 0.5, 3, ((20, 20), (64, 64)), "bf16"),
    (1, 70, 0.5, 3, ((20, 20), (32, 32)), "f32"),
])
@pytest.mark.parametrize("spatial", [False, True])
def test_any_channels(pcpp, n_in, n_out, r, t, shapes, dt, spatial):
    if spatial and n_in > 10000:
        pytest.skip("the line between the forms does not depend on the plan's order")
    rng = np.random.default_rng(zlib.crc32(repr((n_in, n_out, t, dt)).encode()))
    pin = rng.uniform(0, 1, (n_in, 3)).astype(np.float32)
    pout = rng.uniform(0, 1, (n_out, 3)).astype(np.float32)
    K = t ** 3
    o, i, k, seg = oracle.build_triplets(pin, pout, np.float32(r), t)
    flags = pcpp.PLAN_FWD | pcpp.PLAN_BWD_INPUT | (pcpp.PLAN_SPATIAL if spatial else 0)
    T = pcpp.pcpp_build_triplets(dev(pin), dev(pout), r, t, plan_flags=flags)
    assert T.n_triplets == len(o)
    for c_in, c_out in shapes:
        x = rng.standard_normal((n_in, c_in)).astype(np.float32)
        w = (rng.standard_normal((K, c_out, c_in)) / np.sqrt(K * c_in)).astype(np.float32)
        dy = rng.standard_normal((n_out, c_out)).astype(np.float32)
        tdt = torch.float32
        if dt == "bf16":
            x, w, dy, tdt = scenes.round_to_bf16(x), scenes.round_to_bf16(w), scenes.round_to_bf16(dy), torch.bfloat16
        what = f"{n_in}->{n_out} t={t} {c_in}->{c_out} {dt}"
        # run sums are rounded to bf16 in the layers of 64 and 128 channels with up to 64 cells only; elsewhere they keep
        # fp32 precision, and products with bf16 weights are exact
        tol = TOL["bf16" if dt == "bf16" and K <= 64 and (c_in, c_out) in ((64, 64), (64, 128), (128, 64)) else "f32"]
        out = pcpp.pcpp_mvmr_fwd(dev(x, tdt), dev(w, tdt), T)
        assert_close(out.cpu().numpy(), *oracle_fwd(x, w, o, i, k, n_out), tol, what + " fwd")
        gx = pcpp.pcpp_mvmr_bwd_input(dev(dy, tdt), dev(w, tdt), T)
        assert_close(gx.cpu().numpy(), *oracle_bwd_input(dy, w, o, i, k, n_in), tol, what + " bwd_input")
        gw = pcpp.pcpp_mvmr_bwd_weight(dev(x, tdt), dev(dy, tdt), T)
        # bf16 products are exact in fp32 and fp32 layers keep all product terms above 2^-24, so the weight gradient
        # meets the fp32 tolerance whatever the storage type
        assert_close(gw.cpu().numpy(), *oracle_bwd_weight(x, dy, o, i, k, K), TOL["f32"], what + " bwd_weight")
        assert not gw.cpu().numpy()[np.diff(seg) == 0].any()
        again = pcpp.pcpp_mvmr_fwd(dev(x, tdt), dev(w, tdt), T)
        assert torch.equal(out, again)                                        # fixed summation order
        assert torch.equal(gw, pcpp.pcpp_mvmr_bwd_weight(dev(x, tdt), dev(dy, tdt), T))
