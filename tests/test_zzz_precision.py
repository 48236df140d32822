"""Relative error against 64-bit sums of the layers that promise fp32 sums: all fp32 layers, and the bf16 layers whose run
sums are kept exactly.  Values of one sign included: there the roundings of a sum add up instead of cancelling."""
import numpy as np
import pytest
import torch

U = 2.0 ** -24                     # half an ulp of a 32-bit float, relative


def bound(parts):
    """A sum of `parts` parts, each rounded to nearest when it is added: the errors are independent, U / sqrt(3) in the root
    mean square; twice that, and a few U for the parts themselves (32 products, or a run)."""
    return float((4.0 + 2.0 * np.sqrt(parts / 3.0)) * U)


def three_terms(x, drop=()):
    """fp32 values as the bf16 terms that the kernels split them into (each the high half of what the others leave)."""
    terms, rest = [], x.astype(np.float32)
    for _ in range(3):
        hi = (rest.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
        terms.append(hi.astype(np.float64))
        rest = rest - hi
    return sum(t for j, t in enumerate(terms) if j not in drop)


def test_bound_notices_a_lost_term():
    """The bounds below are tight enough that a kernel that loses any term of its operands, or the products of the smaller
    terms, does not pass."""
    rng = np.random.default_rng(3)
    x, w = (rng.standard_normal((64, 256)).astype(np.float32) for _ in range(2))
    for x_, w_ in ((x, w), (abs(x), abs(w))):
        exact = x_.astype(np.float64) @ w_.astype(np.float64).T
        assert np.array_equal(three_terms(x_), x_)
        for drop in (0, 1, 2):
            got = three_terms(x_, (drop,)) @ w_.astype(np.float64).T
            assert np.linalg.norm(got - exact) > 2.0 * bound(27 * 8) * np.linalg.norm(exact)


gpu = pytest.mark.gpu


def layer(n, per, t, c_in, c_out, dt, positive, spatial=False):
    import paper_2511_23227_amd as m
    g = torch.Generator(device="cuda").manual_seed(n + 7 * c_in + c_out)
    xyz = torch.rand(n, 3, generator=g, device="cuda")
    flags = m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0)
    T = m.pcpp_build_triplets(xyz, xyz, (per / (n * 4.18879)) ** (1 / 3), t, plan_flags=flags)
    K = t ** 3
    x = torch.randn(n, c_in, generator=g, device="cuda")
    w = torch.randn(K, c_out, c_in, generator=g, device="cuda") / (K * c_in) ** 0.5
    dy = torch.randn(n, c_out, generator=g, device="cuda")
    if positive:
        x, w, dy = x.abs(), w.abs(), dy.abs()
    if dt == "bf16":
        x, w, dy = x.bfloat16(), w.bfloat16(), dy.bfloat16()
    return m, T, K, x, w, dy


def wide(T, K, x, w, dy, rows):
    """out and dx, or dW, in 64 bits."""
    y = torch.zeros(T.n_out, w.shape[1], dtype=torch.float64, device="cuda")
    dx = torch.zeros(T.n_in, w.shape[2], dtype=torch.float64, device="cuda")
    dw = torch.zeros(w.shape, dtype=torch.float64, device="cuda")
    seg, step = T.seg_offsets.cpu().tolist(), 400000
    for k in range(K):
        wk = w[k].double()
        for s in range(seg[k], seg[k + 1], step):
            e = min(seg[k + 1], s + step)
            o, i = T.tri_o[s:e].long(), T.tri_i[s:e].long()
            xi, do = x[i].double(), dy[o].double()
            if rows:
                y.index_add_(0, o, xi @ wk.t().contiguous())
                dx.index_add_(0, i, do @ wk)
            else:
                dw[k] += do.t().contiguous() @ xi
    return (y, dx) if rows else dw


def err(got, ref):
    return ((got.double() - ref).norm() / ref.norm()).item()


@gpu
@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("n,per,t,c_in,c_out,dt", [
    (2000, 30, 3, 32, 32, "f32"), (9000, 20, 3, 20, 36, "f32"), (9000, 20, 3, 64, 64, "f32"), (3000, 15, 3, 300, 64, "f32"),
    (9000, 20, 3, 96, 96, "f32"), (2000, 30, 3, 256, 256, "f32"), (3000, 25, 3, 512, 520, "f32"), (3000, 60, 6, 64, 200, "f32"),
    (70000, 8, 3, 32, 32, "f32"), (1000, 100, 2, 24, 24, "f32"),
    (3000, 400, 3, 512, 256, "bf16"), (9000, 24, 3, 128, 128, "bf16"), (3000, 25, 3, 200, 200, "bf16"),
    (12500, 20, 3, 40, 136, "f32"), (12500, 60, 2, 128, 136, "bf16"), (12500, 20, 3, 128, 200, "bf16"),     # cooperative
    (3000, 200, 3, 128, 136, "bf16"), (2000, 30, 3, 20, 36, "bf16"), (2000, 300, 3, 24, 160, "bf16"),
])
def test_rows_keep_32_bit_sums(n, per, t, c_in, c_out, dt, positive):
    m, T, K, x, w, dy = layer(n, per, t, c_in, c_out, dt, positive)
    y, dx = wide(T, K, x, w, dy, True)
    e_fwd, e_bwd = err(m.pcpp_mvmr_fwd(x, w, T), y), err(m.pcpp_mvmr_bwd_input(dy, w, T), dx)
    assert e_fwd < bound(K * -(-c_in // 32)) and e_bwd < bound(K * -(-c_out // 32))


# Clouds on either side of a line between two forms of the rows kernel: which form runs may not cost precision.  More waves than the
# form before shorten a wave's sums; the error may not be larger than beyond the line for that (the margin is for other values).
@gpu
@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("n,beyond,per,t,c_in,c_out,dt", [
    (4000, 9000, 24, 3, 128, 128, "f32"), (8000, 9000, 24, 3, 96, 100, "f32"), (4000, 9000, 24, 4, 40, 72, "f32"),
    (8000, 9000, 20, 5, 32, 128, "f32"), (3000, 9000, 24, 2, 512, 128, "f32"),
    (132000, 130000, 12, 3, 128, 128, "bf16"), (132000, 130000, 12, 3, 32, 100, "bf16"),
])
def test_forms_do_not_differ_in_precision(n, beyond, per, t, c_in, c_out, dt, positive):
    errors = []
    for points in (n, beyond):
        m, T, K, x, w, dy = layer(points, per, t, c_in, c_out, dt, positive)
        y, dx = wide(T, K, x, w, dy, True)
        errors.append((err(m.pcpp_mvmr_fwd(x, w, T), y), err(m.pcpp_mvmr_bwd_input(dy, w, T), dx)))
    assert errors[0][0] < 1.1 * errors[1][0] and errors[0][1] < 1.1 * errors[1][1]


# the longest sums: chunks that are summed in three parts (1024 -> 1024: more than 16384 triplets), fp32 chunks of more than 768 triplets
# (256 -> 256), many chunks to one cell
@gpu
@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("n,per,t,c_in,c_out,dt", [
    (3000, 30, 3, 32, 32, "f32"), (20000, 400, 1, 20, 36, "f32"), (60000, 33, 3, 256, 256, "f32"), (9000, 60, 2, 70, 33, "f32"),
    (5000, 330, 1, 1024, 1024, "bf16"), (4000, 130, 3, 512, 520, "bf16"), (20000, 440, 1, 24, 40, "bf16"),
    (9000, 60, 2, 128, 128, "bf16"), (9000, 60, 2, 256, 256, "bf16"),
])
def test_weight_gradient_keeps_32_bit_sums(n, per, t, c_in, c_out, dt, positive):
    m, T, K, x, w, dy = layer(n, per, t, c_in, c_out, dt, positive)
    # a wave adds up to 8192 / (4 * 32) batches; the sums of the waves, the parts and the chunks are added up in two steps
    e = err(m.pcpp_mvmr_bwd_weight(x, dy, T), wide(T, K, x, w, dy, False))
    assert e < bound(64)


# Chunks of the triplet list: a wave adds up a quarter of a chunk, 32 triplets at a time, and the matrix cores cut every addend at the sum's
# last place.  bf16 lists are cut into 1024 chunks over the number of sub-blocks of 128 x 64 channels; a random walk of as many cuts is what
# their sums may be off, half of U each, and U for the rest (the waves' and the chunks' sums).
@gpu
@pytest.mark.parametrize("n,c_in,c_out,blocks", [(24583, 128, 128, 2), (24583, 192, 128, 3), (39583, 64, 128, 1), (100000, 64, 64, 1)])
def test_chunks_are_short_enough(n, c_in, c_out, blocks):
    m, T, K, x, w, dy = layer(n, 24, 3, c_in, c_out, "bf16", False)
    steps = -(-(T.n_triplets * blocks // 1024) // 128) + 1
    e = err(m.pcpp_mvmr_bwd_weight(x, dy, T), wide(T, K, x, w, dy, False))
    assert e < (1.0 + 0.5 * steps ** 0.5) * U
