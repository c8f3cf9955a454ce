"""The shortest segments that cell runs store in records (bins so close that a few
samples share a cell; which lengths do is checked by test_plan_paths.py), and the
length below, against the oracle.  Bound: the tolerance plus the FP32 rounding of
the spectra (1e-6), in FP64 the tolerance."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [3, 4, 5, 6, 7, 63, 64, 65])
@pytest.mark.parametrize("prec,tol", [("fp32", 1e-6), ("fp64", 1e-9)])
@pytest.mark.parametrize("cplx", [False, True])
def test_short_records_match_oracle(gpu, L, prec, tol, cplx):
    import torch
    from paper_2609_12476_amd import Plan, complex_view
    print(f"short records L={L} {prec} complex={cplx}", flush=True)
    w = synth.random_small(L, L, 2, 1e-3, f0=100.0, fs=256.0, f_lo=100.0, df=1e-3, complex_strain=cplx)
    w.strain = w.strain.astype(np.complex64).astype(np.complex128) if cplx else w.strain.astype(np.float32).astype(float)
    with Plan.from_workload(w, precision=prec, tol=tol, method="cellrun") as p:
        sp, _, _ = p.execute(p.strain_tensor(w.strain, gpu))
        torch.cuda.synchronize()
        X = complex_view(sp).cpu().numpy().astype(np.complex128)
    Xr, _, ok = oracle.spectra(w)
    assert ok.all()
    # (against the segment's norm: two bins of so few samples may cancel)
    size = np.sqrt(2.0 * np.sum(np.abs(w.strain) ** 2))
    assert np.linalg.norm(X - Xr) <= (tol + (1e-6 if prec == "fp32" else 0.0)) * size
