"""Which calls run without the workspace that pcpp_mvmr_workspace_bytes asks for, through the C ABI, and what they give: the
kernels that read W as it is and sum on the vector ALUs."""
import numpy as np
import pytest
import torch

import oracle
import scenes
from parity_util import TOL, assert_close, oracle_fwd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pcpp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_23227_amd as m
    m.library()
    return m


class Layer:
    """A small layer and its buffers; op(...) makes one C call with the given workspace."""

    def __init__(self, m, n_in, n_out, r, t, c_in, c_out, dt, seed, spatial=False):
        from paper_2511_23227_amd import binding as B
        self.B, self.L = B, m.library()
        rng = np.random.default_rng(seed)
        self.n_in, self.n_out, self.c_in, self.c_out, self.K = n_in, n_out, c_in, c_out, t ** 3
        pin = rng.uniform(0, 1, (n_in, 3)).astype(np.float32)
        pout = rng.uniform(0, 1, (n_out, 3)).astype(np.float32)
        self.o, self.i, self.k, _ = oracle.build_triplets(pin, pout, np.float32(r), t)
        flags = m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0)
        self.T = m.pcpp_build_triplets(torch.from_numpy(pin).cuda(), torch.from_numpy(pout).cuda(), r, t, plan_flags=flags)
        self.x = rng.standard_normal((n_in, c_in)).astype(np.float32)
        self.w = (rng.standard_normal((self.K, c_out, c_in)) / np.sqrt(self.K * c_in)).astype(np.float32)
        self.dy = rng.standard_normal((n_out, c_out)).astype(np.float32)
        tdt = torch.float32
        if dt == "bf16":
            self.x, self.w, self.dy, tdt = *(scenes.round_to_bf16(a) for a in (self.x, self.w, self.dy)), torch.bfloat16
        self.dx_, self.dw_, self.ddy = (torch.from_numpy(a).cuda().to(tdt) for a in (self.x, self.w, self.dy))
        self.code = B._dtype_code(self.dx_)

    def need(self, op):
        return self.L.pcpp_mvmr_workspace_bytes(op, self.n_in, self.n_out, self.T.n_triplets, self.c_in, self.c_out, self.K,
                                                self.code)

    def run(self, op, ws_bytes):
        """(return code, result) of forward (0), input gradient (1) or weight gradient (2)."""
        P, T = self.B._ptr, self.T
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda") if ws_bytes else None
        rows, cols = ((self.n_out, self.c_out), (self.n_in, self.c_in), (self.K * self.c_out, self.c_in))[op]
        out = torch.full((rows, cols), 7.0, device="cuda")
        tail = (self.n_in, self.n_out, self.c_in, self.c_out, self.K, P(T.tri_o), P(T.tri_i), P(T.tri_k), P(T.seg_offsets),
                T.n_triplets, P(T.plan), T.plan.numel(), T.plan_flags, P(ws), ws_bytes, self.B._stream())
        if op == 2:
            rc = self.L.pcpp_mvmr_bwd_weight(P(self.dx_), P(self.ddy), P(out), self.code, *tail)
        else:
            call = self.L.pcpp_mvmr_bwd_input if op else self.L.pcpp_mvmr_fwd
            rc = call(P(self.ddy if op else self.dx_), P(self.dw_), P(out), self.code, 0, *tail)
        torch.cuda.synchronize()
        return rc, out.cpu().numpy()


@pytest.mark.parametrize("c_in,c_out,dt,t,runs", [
    (32, 32, "f32", 5, True), (64, 64, "f32", 6, True), (64, 64, "bf16", 5, True), (64, 128, "bf16", 5, True),
    (128, 64, "bf16", 6, True), (5, 7, "f32", 3, True), (70, 33, "bf16", 3, True), (128, 128, "bf16", 4, True),
    (32, 32, "f32", 4, False), (64, 64, "f32", 3, False), (64, 64, "bf16", 4, False), (128, 64, "bf16", 3, False),
    (256, 256, "bf16", 2, False), (256, 256, "bf16", 5, False),
])
@pytest.mark.parametrize("spatial", [False, True])
def test_forward_without_workspace(pcpp, c_in, c_out, dt, t, runs, spatial):
    l = Layer(pcpp, 300, 333, 0.2, t, c_in, c_out, dt, 7 * c_in + c_out + t, spatial)
    rc, out = l.run(0, 0)
    if not runs:
        assert rc == -3 and b"workspace" in l.L.pcpp_last_error() and (out == 7.0).all()
        return
    assert rc == 0, l.L.pcpp_last_error()
    assert_close(out, *oracle_fwd(l.x, l.w, l.o, l.i, l.k, l.n_out), TOL["f32"], "forward without workspace")
