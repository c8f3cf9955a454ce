"""Complex strain in FP32 cell runs on both sides of the line between unaligned and
aligned quads (24 samples a cell), with runs that begin at every place of a quad,
end in the copy's padding or hold no whole quad, in rounds with records and with
grids, against the oracle.  Bound: the tolerance plus the FP32 rounding of the
spectra (1e-6)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


# 17 cells (one bin on 16): 23.5, 24 and 24.1 samples a cell; long runs of many
# rounds; a copy without padding and one with 63 samples of it
@pytest.mark.parametrize("L,K", [(399, 1), (408, 1), (409, 1), (1601, 8), (4096, 30), (15361, 130), (30719, 250)])
@pytest.mark.parametrize("kw", [{}, {"parts": 1}, {"parts": 4}])
def test_complex_cell_runs(gpu, L, K, kw):
    import torch
    from paper_2609_12476_amd import Plan, complex_view
    print(f"complex cell runs L={L} K={K} {kw}", flush=True)
    w = synth.random_small(5, L, K, 1e-2, f0=45.0, fs=128.0, complex_strain=True)
    w.strain = w.strain.astype(np.complex64).astype(np.complex128)
    with Plan.from_workload(w, precision="fp32", tol=1e-6, method="cellrun", **kw) as p:
        sp, _, _ = p.execute(p.strain_tensor(w.strain, gpu))
        torch.cuda.synchronize()
        X, off = complex_view(sp).cpu().numpy().astype(np.complex128), p.bin_offsets()
    Xr, roff, ok = oracle.spectra(w)
    assert ok.all()
    for i in range(len(ok)):
        a, b = X[off[i]:off[i + 1]], Xr[roff[i]:roff[i + 1]]
        assert np.linalg.norm(a - b) <= 2e-6 * np.linalg.norm(b)
