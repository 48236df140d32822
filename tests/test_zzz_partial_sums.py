"""The sum of a weight gradient's partial sums: each of its forms (elements per lane, waves per block), which are chosen by the size
of dW and by how many chunks of the triplet list a cell has, at sizes on both sides of the lines between them."""
import numpy as np
import pytest
import torch

# c_in, c_out, t, triplets, whole chunks a cell that they make in bf16 (chunks of 256 triplets and more, up to 1024 in all)
CASES = [
    (127, 129, 6, 3_000, 0),        # rows of dW at any address, fewer chunks than cells
    (65, 65, 6, 40_000, 0),
    (65, 65, 1, 300_000, 469),        # the same with many chunks a cell
    (33, 31, 3, 20_000, 2),         # 2.9 chunks a cell, all blocks at a time
    (33, 31, 3, 30_000, 4),         # 4.3
    (47, 61, 5, 40_000, 1),         # 1.3, more blocks
    (47, 61, 3, 130_000, 18),        # 18
    (47, 61, 3, 160_000, 23),        # 22
    (65, 65, 2, 125_000, 61),        # 61 (bf16), 536 blocks
    (65, 65, 2, 131_000, 64),        # 64 (bf16)
    (63, 65, 2, 10_000, 4),         # 4095 and 4096 elements
    (64, 64, 2, 7_000, 3),          # 3.4 chunks a cell
    (64, 64, 2, 9_000, 4),          # 4.4
    (64, 64, 1, 65_000, 253),         # 254
    (64, 64, 1, 66_000, 257),         # 258
    (128, 128, 2, 60_000, 29),       # 16 384 elements: 29
    (128, 128, 2, 72_000, 35),       # 35 (bf16)
    (127, 128, 2, 30_000, 14),
    (2, 2, 1, 200_000, 783),
]


PER = 40                         # neighbours of every centre: groups of points at one place


def points(triplets):
    return -(-triplets // PER)


@pytest.mark.parametrize("c_in,c_out,t,triplets,chunks", CASES)
def test_case_is_on_its_side(c_in, c_out, t, triplets, chunks):
    """The chunks a cell, from the size of the workspace: one slot of dW per chunk and per cell."""
    from paper_2511_23227_amd import binding
    n, K = points(triplets), t ** 3
    exact = n // PER * PER * PER + (n % PER) ** 2
    slots = binding.library().pcpp_mvmr_workspace_bytes(2, 1, 1, exact, c_in, c_out, K, 1) // (4 * c_in * c_out)
    assert (slots - K) // K == chunks


@pytest.mark.gpu
@pytest.mark.parametrize("c_in,c_out,t,triplets,chunks", CASES)
def test_partial_sums(c_in, c_out, t, triplets, chunks):
    """Against sums in 64 bits; a relative error of 1e-6 is what 32-bit sums of this length show (measured: at most 2.1e-7), one
    chunk counted twice or left out would show at 1e-2 and more."""
    import paper_2511_23227_amd as m
    rng = np.random.default_rng(triplets + c_in)
    K = t ** 3
    # triplets around centres that share all their neighbours: their number is known beforehand, and cells differ in length
    n = points(triplets)
    p = np.repeat(np.arange(-(-n // PER), dtype=np.float32), PER)[:n]
    p = np.stack([p * 4.0, np.zeros(n), np.zeros(n)], 1).astype(np.float32)
    p += rng.uniform(-0.28, 0.28, p.shape).astype(np.float32)
    d = torch.from_numpy(p).cuda()
    T = m.pcpp_build_triplets(d, d, 1.0, t, plan_flags=m.PLAN_FWD)
    x = torch.from_numpy(rng.standard_normal((n, c_in)).astype(np.float32)).cuda()
    dy = torch.from_numpy(rng.standard_normal((n, c_out)).astype(np.float32)).cuda()
    for dtype in (torch.float32, torch.bfloat16):
        xd, dyd = x.to(dtype), dy.to(dtype)
        got = m.pcpp_mvmr_bwd_weight(xd, dyd, T).double()
        want = torch.zeros_like(got)
        seg = T.seg_offsets.cpu().tolist()
        for k in range(K):
            a, b = seg[k], seg[k + 1]
            if b > a:
                want[k] = dyd[T.tri_o[a:b].long()].double().t() @ xd[T.tri_i[a:b].long()].double()
        error = float((got - want).norm() / want.norm())
        print(f"{c_in}x{c_out} {K} cells {T.n_triplets} {dtype}: {error:.1e}")
        assert T.n_triplets > 0 and error < 1e-6
