"""The network's row kernels, the regions' features and the ranking top-k at the
sizes where their tiles, chunks and dispatch rules end, against the FP64 oracle.

Tolerances: a chain of at most 128 FP32 sums with exactly split inputs errs by at
most 128 * 2^-24 = 8e-6 of the sum of absolute values; the network's sums cancel
little, so 2e-5 of the largest logit and of each gradient block's norm.  Indices
are exact.
"""
import numpy as np
import pytest

import synth
from oracle import mlp as om
from oracle import proposal as op

pytestmark = pytest.mark.gpu


def _net(seed, B):
    from paper_2609_12476_amd.mlp import Mlp
    p = synth.mlp_init_params(seed)
    return p, Mlp(max_batch=B, params=p)


# tiles of 16 and 32 rows, the line between them at 16 * 256 rows
@pytest.mark.parametrize("B", [1, 15, 16, 17, 4095, 4096, 4097, 4111, 8193])
def test_forward_at_tile_edges(gpu, B):
    import torch
    print(f"forward B={B}", flush=True)
    p, net = _net(21, 8)
    x = np.random.default_rng(B).standard_normal((B, 64)).astype(np.float32)
    z = net.forward(torch.from_numpy(x).to(gpu)).cpu().numpy().astype(np.float64)
    zr, _ = om.forward(om.weights_as_used(p), x)
    assert z.shape == zr.shape
    assert np.max(np.abs(z - zr)) <= 2e-5 * max(1.0, np.max(np.abs(zr)))
    net.close()


# one chunk of 256 rows, its edges, several chunks with a ragged last one, and
# both row tiles in training
@pytest.mark.parametrize("B", [15, 17, 255, 256, 257, 513, 4097])
def test_gradient_at_chunk_edges(gpu, B):
    import torch
    print(f"gradient B={B}", flush=True)
    p, net = _net(22, B)
    rng = np.random.default_rng(B)
    x = rng.standard_normal((B, 64)).astype(np.float32)
    y = (rng.random(B) < 0.5).astype(np.float32)
    g, loss = net.gradient(torch.from_numpy(x).to(gpu), torch.from_numpy(y).to(gpu))
    g = g.cpu().numpy().astype(np.float64)
    d = om.weights_as_used(p)
    lr, gr = om.loss_and_grad(d, x, y)
    size = sum(np.abs(om.loss_and_grad(d, x[r:r + 1], y[r:r + 1])[1]) for r in range(B)) / B
    assert abs(float(loss.cpu()) - lr) <= 2e-6 * max(1.0, abs(lr))
    o = 0
    for name, shape in om.SHAPES:
        n = int(np.prod(shape))
        assert np.linalg.norm(g[o:o + n] - gr[o:o + n]) <= 8e-6 * np.linalg.norm(size[o:o + n]), name
        o += n
    net.close()


# rows * n at the line between ranking and sorting (32768), odd lengths, k = n,
# equal scores, signed zeros, infinities and NaN
@pytest.mark.parametrize("rows,n,k", [(1, 1, 1), (3, 17, 17), (1, 16384, 64), (2, 16384, 16384), (3, 16384, 5),
                                      (32, 1024, 64), (33, 1024, 64), (8, 4095, 100), (128, 256, 1)])
def test_topk_on_both_sides_of_the_line(gpu, rows, n, k):
    import torch
    from paper_2609_12476_amd import proposal as pp
    print(f"topk rows={rows} n={n} k={k}", flush=True)
    rng = np.random.default_rng(rows * n + k)
    s = np.round(rng.standard_normal((rows, n)) * 50).astype(np.float32)
    special = np.array([np.nan, np.inf, -np.inf, 0.0, -0.0, np.finfo(np.float32).min, np.finfo(np.float32).max],
                       dtype=np.float32)
    at = rng.integers(0, n, size=(rows, 14))
    if n > 1:
        for r in range(rows):
            s[r, at[r]] = np.tile(special, 2)
    got = pp.nr_prop_topk(torch.from_numpy(s).to(gpu), rows, n, k).cpu().numpy()
    assert np.array_equal(got, op.topk(s.astype(np.float64), k))


# bins below, at and past one wave's width; equal loudest bins; rows of the
# type's lowest values
@pytest.mark.parametrize("n_mc,n_sub,K", [(1, 1, 1), (3, 5, 63), (9, 3, 64), (2, 1, 65), (5, 7, 600)])
def test_region_features_at_wave_edges(gpu, n_mc, n_sub, K):
    import torch
    from paper_2609_12476_amd.mlp import nr_mlp_region_features
    print(f"features {n_mc} x {n_sub} x {K}", flush=True)
    rng = np.random.default_rng(K)
    T, L = n_mc * n_sub, 7680
    stat = rng.gamma(50.0, L, size=(T, K)).astype(np.float32)
    stat[0] = stat[0, 0]                                  # every bin is the loudest
    stat[T - 1, [K // 3, K - 1]] = 1e9                    # two are
    stat[T // 2] = -np.inf
    used = rng.integers(0, 60, size=T).astype(np.int32)
    used[T // 2] = 0
    f = nr_mlp_region_features(torch.from_numpy(stat.ravel()).to(gpu), torch.from_numpy(used).to(gpu),
                               n_mc, n_sub, K, 1.0 / L).cpu().numpy()
    ref = op.region_features(stat.astype(np.float64).ravel(), used, n_mc, n_sub, K, 1.0 / L)
    assert np.allclose(f, ref, rtol=1e-5, atol=1e-5)
