"""Calls on both sides of the lines between two kernels of the fold and of top-k:
the results are the same integers and float32 sums on either side."""
import numpy as np
import pytest

from oracle import proposal as op
from oracle import strobo as ost

pytestmark = pytest.mark.gpu


def _fold(x, idx, fold):
    ref = np.zeros(fold, x.dtype)
    for m0 in range(0, len(idx), fold):
        part = idx[m0:m0 + fold]
        ref[:len(part)] += np.where(part >= 0, x[np.maximum(part, 0)], x.dtype.type(0))
    return ref


# workgroups of 2048 slots: 511, 512 and 513 of them, one slot short of and past a
# workgroup; the identity past the line
@pytest.mark.parametrize("n,fs,mc,fold,n_seg", [
    (40000, 1024.0, 1e-2, 2048, 511), (40000, 1024.0, 1e-2, 2048, 512), (40000, 1024.0, 1e-2, 2049, 256),
    (40000, 1024.0, 1e-2, 2047, 513), (40000, 1024.0, 0.0, 2048, 513)])
@pytest.mark.parametrize("cplx", [False, True])
def test_fold_on_both_sides_of_the_line(gpu, n, fs, mc, fold, n_seg, cplx):
    import torch
    from paper_2609_12476_amd import strobo
    print(f"fold line n={n} mc={mc} fold={fold} n_seg={n_seg} complex={cplx}", flush=True)
    rng = np.random.default_rng(n_seg)
    x = rng.standard_normal((n_seg, n)).astype(np.float32)
    if cplx:
        x = (x + 1j * rng.standard_normal((n_seg, n)).astype(np.float32)).astype(np.complex64)
    got = strobo.nr_strobo_fold(torch.from_numpy(x.ravel()).to(gpu), n, fs, mc, 40.0, fold, n_seg=n_seg).cpu().numpy()
    _, t = ost.tau_points(mc, 40.0, fs, n)
    idx = ost.nearest(t, fs, n)
    for i in (0, 1, n_seg // 2, n_seg - 1):
        assert np.array_equal(got[i], _fold(x[i], idx, fold).astype(np.complex64)), i


# rows of one to four scores are sorted, of five and more ranked
@pytest.mark.parametrize("rows,n,k", [(1, 1, 1), (4097, 1, 1), (8192, 4, 4), (6553, 5, 3), (5, 4, 2), (5, 5, 5)])
def test_topk_of_short_rows(gpu, rows, n, k):
    import torch
    from paper_2609_12476_amd import proposal as pp
    print(f"topk short rows={rows} n={n} k={k}", flush=True)
    rng = np.random.default_rng(rows + n)
    s = np.round(rng.standard_normal((rows, n)) * 2).astype(np.float32)
    s[::7, 0] = np.nan
    s[::5, n - 1] = -np.inf
    got = pp.nr_prop_topk(torch.from_numpy(s).to(gpu), rows, n, k).cpu().numpy()
    assert np.array_equal(got, op.topk(s.astype(np.float64), k))
