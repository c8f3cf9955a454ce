"""The stack-slide gather over spectra of 4 GiB and more (64-bit offsets) against the
same spectra in two ranges of less (32-bit offsets).  The whole and its two halves
are the same FP64 sums rounded to float32 once and twice: 4e-6 of max(1,
|n_sigma|), as for other ranges.  Over one range of everything the sums are equal."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, 1])
def test_wide_gather_matches_ranges(gpu, layout):
    import torch
    from paper_2609_12476_amd import stackslide as ss
    print(f"wide gather layout={layout}", flush=True)
    betas, _ = synth.beta_bank(69)
    n_seg, n_bins, L = 792, 20000, 15360
    assert len(betas) * n_seg * n_bins * 4 >= 1 << 32 > len(betas) * (n_seg // 2) * n_bins * 4
    # tracks that stay in the first templates and such that end in the last
    mcs = np.array([1e-4, 2e-3, 1e-2, 2e-2])
    g = ss.geometry(n_seg=n_seg, n_beta=len(betas), n_bins=n_bins, t_coh=30.0, f_lo=40.0, df=1.0 / 30.0, f_start=40.0,
                    f_max=700.0, norm=2.0 / L, layout=layout)
    gen = torch.Generator(device="cuda").manual_seed(3)
    P = torch.empty((len(betas), n_seg, n_bins) if layout == 0 else (len(betas), n_bins, n_seg), device=gpu)
    P.exponential_(1.0 / L, generator=gen)
    with ss.StackSlide(g, betas, mcs, 2) as p:
        k, _, _, ln = p.tables()
        assert k[-1, 0, :ln[-1, 0]].max() >= len(betas) - 2
        whole, used = p.execute(P.view(-1))
        one = torch.zeros_like(whole)
        ou = torch.zeros_like(used)
        p.execute_range(P.view(-1), 0, n_seg, one, ou)
        two = torch.zeros_like(whole)
        tu = torch.zeros_like(used)
        for lo, n in ((0, n_seg // 2), (n_seg // 2, n_seg - n_seg // 2)):
            q = P.narrow(1 if layout == 0 else 2, lo, n).contiguous()
            p.execute_range(q.view(-1), lo, n, two, tu)
        torch.cuda.synchronize()
    assert torch.equal(whole, one) and torch.equal(used, ou) and torch.equal(used, tu)
    assert bool(torch.all((whole - two).abs() <= 4e-6 * whole.abs().clamp(min=1.0)))
    assert int(used.max()) == n_seg and float(whole.abs().max()) > 0.5
