"""Feature tensors of 4 GiB and more, which the matrix-core kernels do not take: the kernels on the vector ALUs, all three
operations.  The rows with triplets lie behind the first 4 GiB."""
import numpy as np
import pytest
import torch

import oracle
import scenes
from parity_util import TOL, assert_close, oracle_bwd_input, oracle_bwd_weight, oracle_fwd

pytestmark = pytest.mark.gpu


# c_many: channels of the side with the large tensor
@pytest.mark.parametrize("c_many,c_few,dt,t,spatial", [(1024, 20, "f32", 2, False), (1000, 33, "f32", 2, True), (1024, 70, "bf16", 2, False)])
@pytest.mark.parametrize("many_inputs", [True, False])
def test_beyond_four_gib(c_many, c_few, dt, t, spatial, many_inputs):
    import paper_2511_23227_amd as m
    rng = np.random.default_rng(c_many + c_few)
    K, few, near, r = t ** 3, 300, 333, 0.25
    tdt, size = (torch.float32, 4) if dt == "f32" else (torch.bfloat16, 2)
    lead = (1 << 32) // (c_many * size) + 1                   # rows in front of the near points: far away, without triplets
    p_few = rng.uniform(0, 1, (few, 3)).astype(np.float32)
    p_near = rng.uniform(0, 1, (near, 3)).astype(np.float32)
    p_many = torch.empty(lead + near, 3, device="cuda")
    at = torch.arange(lead, device="cuda")
    p_many[:lead] = torch.stack([at % 128, at // 128 % 128, at // 16384], 1) * 0.5 + 50.0
    p_many[lead:] = torch.from_numpy(p_near).cuda()
    f_few = rng.standard_normal((few, c_few)).astype(np.float32)
    f_near = rng.standard_normal((near, c_many)).astype(np.float32)
    c_in, c_out = (c_many, c_few) if many_inputs else (c_few, c_many)
    w = (rng.standard_normal((K, c_out, c_in)) / np.sqrt(K * c_in)).astype(np.float32)
    if dt == "bf16":
        f_few, f_near, w = (scenes.round_to_bf16(a) for a in (f_few, f_near, w))
    big = torch.zeros(lead + near, c_many, dtype=tdt, device="cuda")
    big[lead:] = torch.from_numpy(f_near).cuda()
    assert big.numel() * size > 1 << 32
    small, dw_ = torch.from_numpy(f_few).cuda().to(tdt), torch.from_numpy(w).cuda().to(tdt)
    d_few = torch.from_numpy(p_few).cuda()
    pin, pout = (p_many, d_few) if many_inputs else (d_few, p_many)
    T = m.pcpp_build_triplets(pin, pout, r, t, plan_flags=m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0))
    hin, hout = (p_near, p_few) if many_inputs else (p_few, p_near)
    o, i, k, seg = oracle.build_triplets(hin, hout, np.float32(r), t)
    many = i if many_inputs else o
    assert T.n_triplets == len(o)
    assert np.array_equal((T.tri_i if many_inputs else T.tri_o).cpu().numpy(), many + lead)
    if many_inputs:                                            # the large tensor is gathered by the forward pass ...
        got = m.pcpp_mvmr_fwd(big, dw_, T)
        assert_close(got.cpu().numpy(), *oracle_fwd(f_near, w, o, i, k, few), TOL["f32"], "fwd")
        x, dy = big, small
    else:                                                      # ... or by the input gradient
        got = m.pcpp_mvmr_bwd_input(big, dw_, T)
        assert_close(got.cpu().numpy(), *oracle_bwd_input(f_near, w, o, i, k, few), TOL["f32"], "bwd_input")
        x, dy = small, big
    gw = m.pcpp_mvmr_bwd_weight(x, dy, T).cpu().numpy()
    hx, hdy = (f_near, f_few) if many_inputs else (f_few, f_near)
    assert_close(gw, *oracle_bwd_weight(hx, hdy, o, i, k, K), TOL["f32"], "bwd_weight")
