"""The fold's shared evaluation of the inverse time map: every sample it picks is
the plain evaluation's, bit for bit (float32 sums in the order of the points)."""
import numpy as np
import pytest

from oracle import strobo as ost

pytestmark = pytest.mark.gpu


def _fold(x, idx, fold):
    ref = np.zeros(fold, x.dtype)
    for m0 in range(0, len(idx), fold):
        part = idx[m0:m0 + fold]
        ref[:len(part)] += np.where(part >= 0, x[np.maximum(part, 0)], x.dtype.type(0))
    return ref


# one slot and eight a thread (at and past the line between them), folds of one
# slot and of more than 64 multiples, folds past the last point, a segment that
# ends shortly before coalescence (the series is too long there), none at all
@pytest.mark.parametrize("n,fs,mc,f0,fold,n_seg", [
    (1, 256.0, 1e-2, 50.0, 3, 1), (4099, 1024.0, 1e-1, 40.0, 1, 2), (4099, 256.0, 3e-2, 40.0, 37, 3),
    (65537, 4096.0, 1e-2, 50.0, 16385, 2), (300001, 1024.0, 1e-2, 40.0, 75001, 20), (300001, 1024.0, 1e-1, 20.0, 131072, 8),
    (262144, 4096.0, 0.0, 50.0, 65537, 32), (100000, 4096.0, 1.0, 40.0, 200000, 6)])
@pytest.mark.parametrize("cplx", [False, True])
def test_fold_picks_the_plain_samples(gpu, n, fs, mc, f0, fold, n_seg, cplx):
    import torch
    from paper_2609_12476_amd import strobo
    print(f"fold n={n} fs={fs} mc={mc} fold={fold} n_seg={n_seg} complex={cplx}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n_seg, n)).astype(np.float32)
    if cplx:
        x = (x + 1j * rng.standard_normal((n_seg, n)).astype(np.float32)).astype(np.complex64)
    got = strobo.nr_strobo_fold(torch.from_numpy(x.ravel()).to(gpu), n, fs, mc, f0, fold, n_seg=n_seg).cpu().numpy()
    _, t = ost.tau_points(mc, f0, fs, n)
    idx = ost.nearest(t, fs, n)
    for i in range(n_seg):
        assert np.array_equal(got[i], _fold(x[i], idx, fold).astype(np.complex64)), i
