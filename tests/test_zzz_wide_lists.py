"""256 -> 256 bf16 on clouds in which a blob of points holds most of the triplets, on both sides of the line between the
producer/consumer kernel (at most three triplets per cell and centre) and the tile kernel.  The forward pass in spatial order
and the input gradient in either order take the producer/consumer kernel below the line.  (It takes clouds of more than 10240 centres.)"""
import numpy as np
import pytest
import torch

import oracle
import scenes
from test_gpu_spatial import check_all, dev

R, T_, C = 0.12, 2, 256
K = T_ ** 3


def cloud(below):
    """A dense blob and lone points, each its own only neighbour: as many that |T| is on the wanted side of 3 n K, if only just."""
    rng = np.random.default_rng(21)
    blob = rng.normal(0.5, 0.03, (500, 3)).astype(np.float32)
    in_blob = len(oracle.build_triplets(blob, blob, np.float32(R), T_)[0])
    lone = -(-(in_blob - 3 * K * len(blob)) // (3 * K - 1)) - (0 if below else 1)
    grid = np.stack(np.meshgrid(*[np.arange(24)] * 3, indexing="ij"), -1).reshape(-1, 3)[:lone] * 0.25 + 2.0
    p = np.concatenate([blob, grid]).astype(np.float32)
    p = p[rng.permutation(len(p))]
    return p, in_blob + lone


@pytest.mark.parametrize("below", [True, False])
def test_cloud_is_on_its_side(below):
    p, n = cloud(below)
    o, i, k, seg = oracle.build_triplets(p, p, np.float32(R), T_)
    assert len(p) > 10240 and len(o) == n and (n <= 3 * len(p) * K) == below and abs(n - 3 * len(p) * K) < 3 * K
    # in spatial order the blob's points share a few blocks: far more rows per cell and block than a producer has in flight
    # (four producers of 32 rows), and runs longer than its groups of four rows
    assert np.bincount(k).max() > 4 * 4 * 4 * 32 and np.bincount(k.astype(np.int64) * len(p) + o).max() > 64


@pytest.mark.gpu
@pytest.mark.parametrize("below", [True, False])
@pytest.mark.parametrize("spatial", [False, True])
def test_blob_and_lone_points(below, spatial):
    import paper_2511_23227_amd as m
    p, _ = cloud(below)
    rng = np.random.default_rng(5)
    x, dy = (scenes.round_to_bf16(rng.standard_normal((len(p), C)).astype(np.float32)) for _ in range(2))
    w = scenes.round_to_bf16((rng.standard_normal((K, C, C)) / np.sqrt(K * C)).astype(np.float32))
    d = dev(p)
    T = m.pcpp_build_triplets(d, d, R, T_, plan_flags=m.PLAN_FWD | m.PLAN_BWD_INPUT | (m.PLAN_SPATIAL if spatial else 0))
    check_all(m, T, p, p, R, T_, x, w, dy, "bf16", f"blob below={below} spatial={spatial}")
