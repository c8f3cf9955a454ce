"""The stack-slide gather where its blocks of 64 lags and of 8 values end, whole
and over segment ranges, with values that no track of a lane may pick up
(NaN in every segment but the range's tracks').  The statistic is an FP64 sum
rounded to float32: 2e-6 of max(1, |n_sigma|) as everywhere for it."""
import numpy as np
import pytest

import synth
from oracle import stackslide as oss

pytestmark = pytest.mark.gpu

BETAS, _ = synth.beta_bank(69)


@pytest.mark.parametrize("n_seg,S", [(1, 1), (7, 2), (9, 1), (63, 1), (64, 2), (65, 1), (129, 3)])
@pytest.mark.parametrize("layout", [0, 1])
def test_gather_at_block_edges(gpu, n_seg, S, layout):
    import torch
    from paper_2609_12476_amd import stackslide as ss
    print(f"gather n_seg={n_seg} S={S} layout={layout}", flush=True)
    n_bins, L = 600, 15360
    mcs = np.array([5e-4, 2e-2, 9e-2])
    P = synth.noise_power(len(BETAS), n_seg, n_bins, L, seed=n_seg)
    g = ss.geometry(n_seg=n_seg, n_beta=len(BETAS), n_bins=n_bins, t_coh=30.0, f_lo=40.0, df=1.0 / 30.0,
                    f_start=40.0, f_max=60.0, norm=2.0 / L, layout=layout)
    dev = lambda q: (lambda t: ss.nr_ss_transpose(t, *q.shape) if layout else t)(
        torch.from_numpy(np.ascontiguousarray(q)).to(gpu))
    ref, cnt = oss.n_sigma(P, mcs, S, 30.0, BETAS, 40.0, 1.0 / 30.0, 40.0, 60.0, 2.0 / L)
    with ss.StackSlide(g, BETAS, mcs, S) as p:
        ns, used = (v.cpu().numpy() for v in p.execute(dev(P)))
        assert np.array_equal(used, cnt)
        assert np.all(np.abs(ns - ref) <= 2e-6 * np.maximum(1.0, np.abs(ref)))
        # ranges add up; a NaN segment reaches only the tracks that pass it
        part = torch.zeros(ref.shape, device=gpu)
        for lo in range(0, n_seg, 50):
            q = P[:, lo:lo + 50]
            p.execute_range(dev(q), lo, q.shape[1], part)
        assert np.all(np.abs(part.cpu().numpy() - ref) <= 4e-6 * np.maximum(1.0, np.abs(ref)))
        P2 = P.copy()
        P2[:, n_seg // 2] = np.nan
        ns2 = p.execute(dev(P2))[0].cpu().numpy()
        start = np.arange(n_seg * S) // S
        hit = (start[None, :] <= n_seg // 2) & (start[None, :] + cnt > n_seg // 2)
        assert np.array_equal(np.isnan(ns2), hit)
        assert np.array_equal(ns2[~hit], ns[~hit])
