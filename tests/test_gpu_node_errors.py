"""Spectra from band-limited nodes are no further from the oracle than those from
the samples, by the root mean square over instances of the relative l2 error
(the two paths' errors are independent, so single instances may go either way).
The samples are placed by cell runs of one wave an instance."""
import numpy as np
import pytest

import oracle

from test_gpu_nodes import SHAPES, workload

pytestmark = pytest.mark.gpu


def _rms_errors(gpu, name, prec, tol):
    import torch
    from paper_2609_12476_amd import Plan, complex_view
    *args, kw = SHAPES[name]
    sq = {"nodes": [], "samples": []}
    for seed in (1, 2):
        w = workload(seed, *args, **kw)
        X = {}
        for path, opt in (("nodes", {}), ("samples", dict(method="cellrun", parts=1))):
            with Plan.from_workload(w, precision=prec, tol=tol, **opt) as p:
                assert any(c.width for c in p.nodes()) == (path == "nodes")
                sp, _, _ = p.execute(p.strain_tensor(w.strain, gpu))
                torch.cuda.synchronize()
                X[path] = complex_view(sp).cpu().numpy().astype(np.complex128)
                off, ok = p.bin_offsets(), p.valid_mask().astype(bool)
        idx = np.flatnonzero(ok)
        idx = np.sort(np.random.default_rng(seed).choice(idx, min(len(idx), 150), False))
        Xr, roff, _ = oracle.spectra(w, inst_idx=idx)
        for path, Y in X.items():
            sq[path] += [(np.linalg.norm(Y[off[i]:off[i + 1]] - Xr[roff[j]:roff[j + 1]]) /
                          np.linalg.norm(Xr[roff[j]:roff[j + 1]])) ** 2 for j, i in enumerate(idx)]
    return [float(np.sqrt(np.mean(sq[p]))) for p in ("nodes", "samples")]


# several tiles of reference frequencies a workgroup; the longest small DFT
@pytest.mark.parametrize("name", ["many_refs", "largest_small_grid", "search"])
def test_fp32_nodes_err_no_more_than_samples(gpu, name):
    print(f"node errors fp32 {name}", flush=True)
    nodes, samples = _rms_errors(gpu, name, "fp32", 1e-6)
    print(f"  nodes {nodes:.2e}, samples {samples:.2e}", flush=True)
    assert nodes <= samples


# the loosest and the tightest class that samples spread with width 12, on small
# grids and past them
@pytest.mark.parametrize("name", ["search", "few_bins", "one_bin", "first_fft_grid"])
@pytest.mark.parametrize("tol", [6e-10, 7e-11])
def test_fp64_width_12_errs_no_more_than_samples(gpu, name, tol):
    import paper_2609_12476_amd.nufft_resample as nr
    print(f"node errors fp64 {name} {tol}", flush=True)
    assert nr.nufft_resample_kernel_params(tol, 2.0, "fp64", 30).w == 12
    nodes, samples = _rms_errors(gpu, name, "fp64", tol)
    print(f"  nodes {nodes:.2e}, samples {samples:.2e}", flush=True)
    assert nodes <= samples
