"""The measured cases of the resampling library: the calls that a transient
search makes, over the sizes that it makes them at.

A case is a dict of plain values with a "kind":

  search   one semicoherent sum (Plan.semicoherent_sum) over n_seg segments of
           t_coh seconds and n_mc chirp masses x n_sub sub-bands of 1 Hz: the
           search itself, and the coarse and fine passes of the proposal
  spectra  Plan.execute of a bank of n_beta templates over the 40-60 Hz band,
           every segment its own reference: the spectra that the stack-slide
           reads; n_seg = n_beta = 1 is one segment and one template
  ragged   Plan.execute of n_inst independent instances of mixed length, rate
           and tolerance (precision "auto"), replayed from a HIP graph
  stack    StackSlide.execute: n_sigma along the tracks through stored spectra
  rank     the ranking of a coarse grid: region features, the network's logits,
           the largest z of every template and the best regions by it
  train    one training step of the network: Mlp.gradient, then Mlp.adam_step
  fold     nr_strobo_fold, the stroboscopic baseline's resampling

Strain is white Gaussian noise with one injected Newtonian chirp.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_12476_amd import mlp, proposal, stackslide, strobo
from paper_2609_12476_amd import nufft_resample as nr

MC_LO, MC_HI = 5e-4, 1e-1                 # chirp masses searched, Msun
BAND_LO, BAND_HI = 40.0, 60.0             # band searched, Hz
BETA_LO, BETA_HI = 3e-8, 7e-4             # bank of the coherent stage, 1/s at 50 Hz
T_SUN = 1.3271244e20 / 299792458.0 ** 3   # GM_sun / c^3, s
DEV = "cuda"


def listed():
    return [
        # the smallest call: one segment, one template, the whole band in double precision
        {"name": "segment_fp64", "kind": "spectra", "n_seg": 1, "n_beta": 1, "t_coh": 30.0, "fs": 256.0,
         "precision": "fp64", "tol": 1e-9},
        # one injection's data (35 segments of 30 s) against a small coarse grid
        {"name": "search_35seg", "kind": "search", "n_seg": 35, "n_mc": 16, "n_sub": 20, "t_coh": 30.0,
         "fs": 256.0, "precision": "fp32", "tol": 1e-6},
        # an hour of data, 64 chirp masses: the benchmark's default workload
        {"name": "search_1h", "kind": "search", "n_seg": 120, "n_mc": 64, "n_sub": 20, "t_coh": 30.0,
         "fs": 256.0, "precision": "fp32", "tol": 1e-6},
        # the largest: two hours against a full coarse grid of the proposal
        {"name": "search_2h", "kind": "search", "n_seg": 240, "n_mc": 256, "n_sub": 20, "t_coh": 30.0,
         "fs": 256.0, "precision": "fp32", "tol": 1e-6},
        # double precision, as a search's reference is computed
        {"name": "search_fp64", "kind": "search", "n_seg": 60, "n_mc": 32, "n_sub": 20, "t_coh": 30.0,
         "fs": 256.0, "precision": "fp64", "tol": 1e-9},
        # the paper's bank over an hour: spectra for the stack-slide
        {"name": "bank_1h", "kind": "spectra", "n_seg": 120, "n_beta": 69, "t_coh": 30.0, "fs": 512.0,
         "precision": "fp32", "tol": 1e-6},
        # a batch of unlike requests, every one its own segment
        {"name": "ragged_512", "kind": "ragged", "n_inst": 512},
        # stack-slide of an hour's spectra, 2048 chirp masses x 8 start times per segment
        {"name": "stack_1h", "kind": "stack", "n_seg": 120, "n_beta": 69, "n_bins": 600, "n_mc": 2048,
         "t0_steps": 8, "layout": 1},
        # the same spectra as execute stores them, a smaller track grid
        {"name": "stack_layout0", "kind": "stack", "n_seg": 120, "n_beta": 69, "n_bins": 600, "n_mc": 500,
         "t0_steps": 4, "layout": 0},
        # ranking of one coarse grid of 256 x 20 regions
        {"name": "rank_5120", "kind": "rank", "n_mc": 256, "n_sub": 20, "n_bins": 30, "k": 128},
        # the network's training batch
        {"name": "train_1024", "kind": "train", "batch": 1024},
        # the baseline, 8-fold oversampled segments of 256 s
        {"name": "fold_256s", "kind": "fold", "n_seg": 8, "n_samples": 1048576, "fs_o": 4096.0, "complex": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "spectra", "spectra", "ragged", "stack", "rank", "train", "fold"])
    t_coh, fs = rng.choice([10.0, 30.0, 30.0, 45.0, 60.0]), rng.choice([256.0, 256.0, 512.0])
    fp64 = rng.random() < 0.25
    acc = {"precision": "fp64", "tol": 1e-9} if fp64 else {"precision": "fp32", "tol": rng.choice([1e-6, 1e-6, 1e-4])}
    if kind == "search":
        # no more samples than the largest listed case, an eighth of them in double precision
        most = 240 * 256 * 20 * 7680 // (8 if fp64 else 1)
        while True:
            c = {"kind": kind, "n_seg": _log(rng, 8, 240), "n_mc": _log(rng, 4, 256), "n_sub": rng.randint(1, 20),
                 "t_coh": t_coh, "fs": fs, **acc}
            inst = c["n_seg"] * c["n_mc"] * c["n_sub"]
            if inst * t_coh * fs <= most and inst <= 240 * 256 * 20:
                return c
    if kind == "spectra":
        return {"kind": kind, "n_seg": _log(rng, 1, 120), "n_beta": _log(rng, 1, 69), "t_coh": t_coh, "fs": fs, **acc}
    if kind == "ragged":
        return {"kind": kind, "n_inst": _log(rng, 8, 512)}
    if kind == "stack":
        return {"kind": kind, "n_seg": _log(rng, 30, 240), "n_beta": rng.randint(20, 69),
                "n_bins": rng.choice([200, 600, 900]), "n_mc": _log(rng, 64, 2048), "t0_steps": rng.randint(1, 8),
                "layout": rng.randint(0, 1)}
    if kind == "rank":
        n_mc, n_sub = _log(rng, 8, 256), rng.randint(1, 20)
        return {"kind": kind, "n_mc": n_mc, "n_sub": n_sub, "n_bins": rng.choice([10, 30, 45, 60]),
                "k": rng.randint(1, n_mc * n_sub)}
    if kind == "train":
        return {"kind": kind, "batch": _log(rng, 1, 4096)}
    return {"kind": kind, "n_seg": rng.randint(1, 8), "n_samples": _log(rng, 4096, 1048576),
            "fs_o": rng.choice([256.0, 1024.0, 4096.0]), "complex": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs --

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _beta(mc, f0):
    return 19.2 * math.pi ** (8.0 / 3.0) * (T_SUN * mc) ** (5.0 / 3.0) * f0 ** (8.0 / 3.0)


def _masses(n):
    return MC_LO * (MC_HI / MC_LO) ** (np.arange(n) / max(n - 1.0, 1.0))


def _bank(n):
    betas = np.linspace(BETA_LO, BETA_HI, n) if n > 1 else np.array([1e-4])
    return betas, (betas / _beta(1.0, 50.0)) ** 0.6


def _chirp(n, fs, rng, amp):
    """A Newtonian chirp sampled at fs for n samples (zero past 0.45 fs)."""
    mc, f = 10.0 ** rng.uniform(math.log10(MC_LO), math.log10(MC_HI)), rng.uniform(BAND_LO, BAND_HI)
    b, t = _beta(mc, f), torch.arange(n, dtype=torch.float64, device=DEV) / fs
    y = (8.0 / 3.0) * b * t
    on = y < 1.0 - (f / (0.45 * fs)) ** (8.0 / 3.0)
    y = torch.where(on, y, torch.zeros_like(y))
    ph = -(0.6 * f / b) * torch.expm1(0.625 * torch.log1p(-y))
    return torch.where(on, amp * torch.cos(2.0 * math.pi * torch.frac(ph) + rng.uniform(0.0, 6.28)), 0.0 * t)


def _strain(n, fs, seed, precision, amp=0.05):
    x = torch.randn(n, generator=_gen(seed), dtype=torch.float64, device=DEV)
    x += _chirp(n, fs, np.random.default_rng(seed), amp)
    return x.to(torch.float64 if precision != "fp32" else torch.float32)


def _describe(case, seed=0):
    """Segments (offset, samples, rate, start), templates (mc, f0, f_lo, df, bins, f_max) and,
    where they are not the full product, instances (segment, template, tolerance)."""
    if case["kind"] == "ragged":
        # shapes are the batch's own, not the seed's: a program that replays a graph keeps them
        rng = np.random.default_rng(2)
        c = rng.integers(27, size=case["n_inst"])
        T, fs = np.array([10.0, 30.0, 60.0])[c // 9], np.array([256.0, 512.0, 1024.0])[c // 3 % 3]
        n = len(c)
        L = np.rint(T * fs).astype(np.int64)
        seg = (np.concatenate([[0], np.cumsum(L)[:-1]]), L, fs, np.zeros(n))
        mc = 10.0 ** rng.uniform(math.log10(MC_LO), math.log10(MC_HI), n)
        tm = (mc, rng.uniform(BAND_LO, BAND_HI, n), np.full(n, BAND_LO), np.zeros(n),
              np.rint(20.0 * T).astype(np.int32), np.zeros(n))
        return seg, tm, (np.arange(n), np.arange(n), np.array([1e-3, 1e-6, 1e-9])[c % 3])
    n, L = case["n_seg"], int(round(case["t_coh"] * case["fs"]))
    off, T = np.arange(n, dtype=np.int64) * L, case["t_coh"]
    if case["kind"] == "search":
        mc, b = np.repeat(_masses(case["n_mc"]), case["n_sub"]), np.tile(np.arange(case["n_sub"]), case["n_mc"])
        m = len(mc)
        tm = (mc, BAND_LO + b + 0.5, BAND_LO + b, np.full(m, 1.0 / T), np.full(m, int(round(T)), np.int32),
              np.full(m, BAND_HI))
        return (off, np.full(n, L), np.full(n, case["fs"]), np.arange(n) * T), tm, None
    _, mc = _bank(case["n_beta"])
    m = len(mc)
    tm = (mc, np.full(m, 50.0), np.full(m, BAND_LO), np.full(m, 1.0 / T),
          np.full(m, int(round((BAND_HI - BAND_LO) * T)), np.int32), np.zeros(m))
    return (off, np.full(n, L), np.full(n, case["fs"]), np.zeros(n)), tm, None


def _he_uniform(seed):
    """Initial weights of the 64-256-256-1 network: W1, b1, W2, b2, w3, b3, flat."""
    rng, parts = np.random.default_rng(seed), []
    for rows, cols in ((256, 64), (256, 256), (1, 256)):
        lim = math.sqrt(6.0 / cols)
        parts += [rng.uniform(-lim, lim, rows * cols), rng.uniform(-0.1, 0.1, rows)]
    return np.concatenate(parts).astype(np.float32)


def _net_parts(p):
    """The flat parameters as (W1, b1, W2, b2, w3, b3)."""
    at, out = 0, []
    for shape in ((256, 64), (256,), (256, 256), (256,), (256,), (1,)):
        n = int(np.prod(shape))
        out.append(p[at:at + n].reshape(shape))
        at += n
    return out


def _train_inputs(case, seed):
    g = _gen(seed)
    x = torch.randn(case["batch"], 64, generator=g, device=DEV)
    return x, (torch.rand(case["batch"], generator=g, device=DEV) < 0.5).float()


def _rank_inputs(case, seed):
    """A summed grid over 120 segments: S norm of noise has mean and variance 120."""
    n = case["n_mc"] * case["n_sub"]
    z = torch.randn(n * case["n_bins"], generator=_gen(seed), dtype=torch.float64, device=DEV)
    used = torch.full((n,), 120, dtype=torch.int32, device=DEV)
    used[::17] = 77
    N = used.double().repeat_interleave(case["n_bins"])
    return ((N + N.sqrt() * z).clamp_min(1.0) * 7680.0).float(), used


def _stack_inputs(case, seed):
    """Noise spectra |X|^2 of segments of 15360 samples, in layout 0."""
    u = torch.rand(case["n_beta"] * case["n_seg"] * case["n_bins"], generator=_gen(seed), dtype=torch.float64, device=DEV)
    return (-15360.0 * torch.log1p(-u)).float()


def _fold_input(case, seed):
    n = case["n_seg"] * case["n_samples"]
    x = torch.randn(n * (2 if case["complex"] else 1), generator=_gen(seed), device=DEV)
    return torch.view_as_complex(x.view(-1, 2)) if case["complex"] else x


FOLD_MC, FOLD_F0 = 1e-2, 20.0


def _fold_size(case):
    return case["n_samples"] // 4 + 1     # four grid points a slot


# ------------------------------------------------------------- preparation --

def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("search", "spectra", "ragged"):
        seg, tm, inst = _describe(case)
        prec = case.get("precision", "auto")
        total = int(seg[0][-1] + seg[1][-1])
        kw = dict(precision=prec, tol=case.get("tol", 1e-6), strain_length=total)
        if kind == "ragged":
            s["stream"] = torch.cuda.Stream()
            kw.update(stream=s["stream"], use_graph=True)
        s["x"] = _strain(total, float(seg[2][0]), seed, prec)
        s["plan"] = p = nr.Plan(nr.make_segments(*seg), nr.make_templates(*tm),
                                nr.make_instances(*inst) if inst else None, **kw)
        if kind == "search":
            s["stat"] = torch.zeros(p.info.stat_bins, dtype=p.out_dtype, device=DEV)
            s["used"] = torch.zeros(p.n_tmpls, dtype=torch.int32, device=DEV)
        else:
            s["spectra"] = torch.empty(2 * p.info.total_bins, dtype=p.out_dtype, device=DEV)
            s["power"] = torch.empty(p.info.total_bins, dtype=p.out_dtype, device=DEV)
            s["valid"] = torch.empty(p.n_inst, dtype=torch.uint8, device=DEV)
    elif kind == "stack":
        P = _stack_inputs(case, seed)
        dims = (case["n_beta"], case["n_seg"], case["n_bins"])
        s["power"] = stackslide.nr_ss_transpose(P, *dims) if case["layout"] else P
        g = stackslide.geometry(case["n_seg"], case["n_beta"], case["n_bins"], 30.0, BAND_LO, 20.0 / case["n_bins"],
                                BAND_LO, BAND_HI, 2.0 / 15360.0, layout=case["layout"])
        s["plan"] = p = stackslide.StackSlide(g, _bank(case["n_beta"])[0], _masses(case["n_mc"]), case["t0_steps"])
        shape = (case["n_mc"], case["n_seg"] * case["t0_steps"])
        s["out"] = torch.empty(shape, device=DEV)
        s["used"] = torch.empty(shape, dtype=torch.int32, device=DEV)
    elif kind == "rank":
        s["stat"], s["used"] = _rank_inputs(case, seed)
        n = case["n_mc"] * case["n_sub"]
        s["net"] = mlp.Mlp(max_batch=1024, params=_he_uniform(seed))
        s["features"] = torch.empty(n, 64, device=DEV)
        s["logits"], s["z"] = torch.empty(n, device=DEV), torch.empty(n, device=DEV)
        s["arg"] = torch.empty(n, dtype=torch.int32, device=DEV)
        s["top"] = torch.empty(1, case["k"], dtype=torch.int32, device=DEV)
    elif kind == "train":
        s["x"], s["y"] = _train_inputs(case, seed)
        s["net"] = mlp.Mlp(max_batch=case["batch"], params=_he_uniform(seed))
    else:
        s["x"] = _fold_input(case, seed)
        s["out"] = torch.empty(case["n_seg"], _fold_size(case), dtype=torch.complex64, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "search":
        s["stat"].zero_()
        s["used"].zero_()
        s["plan"].semicoherent_sum(s["x"], None, s["stat"], s["used"])
        return {"stat": s["stat"], "used": s["used"]}
    if kind in ("spectra", "ragged"):
        s["plan"].execute(s["x"], s["spectra"], s["power"], s["valid"])
        return {"spectra": s["spectra"], "power": s["power"], "valid": s["valid"]}
    if kind == "stack":
        s["plan"].execute(s["power"], s["out"], s["used"])
        return {"n_sigma": s["out"], "used": s["used"]}
    if kind == "rank":
        n_mc, n_sub, K = case["n_mc"], case["n_sub"], case["n_bins"]
        mlp.nr_mlp_region_features(s["stat"], s["used"], n_mc, n_sub, K, 1.0 / 7680.0, s["features"])
        s["net"].forward(s["features"], s["logits"])
        proposal.nr_prop_max_z(s["stat"], s["used"], n_mc * n_sub, 1, K, 1.0 / 7680.0, s["z"], s["arg"])
        proposal.nr_prop_topk(s["z"], 1, n_mc * n_sub, case["k"], s["top"])
        return {"features": s["features"], "logits": s["logits"], "z": s["z"], "arg": s["arg"], "top": s["top"]}
    if kind == "train":
        g, loss = s["net"].gradient(s["x"], s["y"])
        s["net"].adam_step(g, 1e-4)
        return {"grad": g, "loss": loss}
    strobo.nr_strobo_fold(s["x"], case["n_samples"], case["fs_o"], FOLD_MC, FOLD_F0, _fold_size(case),
                          n_seg=case["n_seg"], out=s["out"])
    return {"fold": s["out"]}


# ------------------------------------------------------------------- work --

def work(case):
    kind = case["kind"]
    if kind in ("search", "spectra", "ragged"):
        seg, tm, inst = _describe(case)
        size = {"fp32": 4, "fp64": 8, "auto": 8}[case.get("precision", "auto")]
        n_inst = len(inst[0]) if inst else len(seg[0]) * len(tm[0])
        K = tm[4].astype(np.float64)
        strain = float(np.sum(seg[1])) * size
        # every instance at the least: a transform of 2 K points and its power
        per = np.sum(10.0 * K * np.log2(2.0 * K) + 5.0 * K) * (n_inst / len(tm[0]))
        if kind == "search":
            return {"bytes": strain + float(np.sum(K)) * size + 4.0 * len(K), "flops": float(per)}
        return {"bytes": strain + float(np.sum(K)) * (n_inst / len(tm[0])) * 3 * size + n_inst, "flops": float(per)}
    if kind == "stack":
        tracks = case["n_mc"] * case["n_seg"] * case["t0_steps"]
        reads = int(_tracks(case)[3].sum())
        return {"bytes": 4.0 * case["n_beta"] * case["n_seg"] * case["n_bins"] + 8.0 * tracks, "flops": 4.0 * reads}
    if kind == "rank":
        n = case["n_mc"] * case["n_sub"]
        return {"bytes": n * (4.0 * case["n_bins"] + 4 + 256 + 12) + 4.0 * case["k"] + 165e3,
                "flops": n * (2.0 * (64 * 256 + 256 * 256 + 256) + 4.0 * case["n_bins"])}
    if kind == "train":
        B = case["batch"]
        return {"bytes": B * 260.0 + 82689 * 28.0, "flops": 2.0 * B * (2 * 64 * 256 + 3 * 256 * 256 + 3 * 256)}
    size = 8 if case["complex"] else 4
    return {"bytes": case["n_seg"] * (case["n_samples"] * float(size) + _fold_size(case) * 8.0),
            "flops": 40.0 * case["n_seg"] * case["n_samples"]}


# ------------------------------------------------------ values in 64 bits --

def _dtau(b, t_start, L, fs):
    """tau(t_j) - tau(t_start) of Eq. (new_t), one row a start time, in double precision."""
    us = 1.0 - (8.0 / 3.0) * b * torch.as_tensor(t_start, dtype=torch.float64, device=DEV)[:, None]
    j = torch.arange(L, dtype=torch.float64, device=DEV)[None, :]
    return -(0.6 / b) * us ** 0.625 * torch.expm1(0.625 * torch.log1p(-(8.0 / 3.0) * b / (us * fs) * j))


def _phasor(f, tau):
    ph = f * tau
    ph = (ph - torch.round(ph)) * (-2.0 * math.pi)
    return torch.complex(torch.cos(ph), torch.sin(ph))


def _valid(b, f0, t_start, L, fs, f_max):
    us = 1.0 - (8.0 / 3.0) * b * t_start
    ul = 1.0 - (8.0 / 3.0) * b * (t_start + (L - 1) / fs)
    ok = (ul > 0.0) & (us > 0.0)
    return ok & (f0 * np.maximum(ul, 1e-300) ** -0.375 <= f_max) if f_max > 0.0 else ok


def _sums(x, tau, f_lo, df, K):
    """sum_j x_j exp(-2 pi i (f_lo + k df) tau_j), [rows][K]."""
    z, r = x * _phasor(f_lo, tau), _phasor(df, tau)
    out = torch.empty(x.shape[0], K, dtype=torch.complex128, device=DEV)
    for k in range(K):
        out[:, k] = z.sum(1)
        z = z * r
    return out


def _exact_plan(case, seed):
    seg, tm, inst = _describe(case)
    prec = case.get("precision", "auto")
    x = _strain(int(seg[0][-1] + seg[1][-1]), float(seg[2][0]), seed, prec).double()
    mc, f0, f_lo, df, K, f_max = tm
    if case["kind"] == "ragged":
        sp, ok = [], torch.ones(len(mc), dtype=torch.uint8)
        for i in range(len(mc)):
            L, fs = int(seg[1][i]), float(seg[2][i])
            b = _beta(mc[i], f0[i])
            ok[i] = bool(_valid(b, f0[i], np.zeros(1), L, fs, 0.0)[0])
            X = torch.zeros(int(K[i]), dtype=torch.complex128, device=DEV)
            if ok[i]:
                tau, xi = _dtau(b, [0.0], L, fs), x[seg[0][i]:seg[0][i] + L][None]
                for k0 in range(0, int(K[i]), 64):
                    k1 = min(int(K[i]), k0 + 64)
                    X[k0:k1] = _sums(xi, tau, f_lo[i] + k0 * fs / L, fs / L, k1 - k0)[0]
            sp.append(X)
        X = torch.cat(sp)
        return {"spectra": torch.view_as_real(X).reshape(-1), "power": X.real ** 2 + X.imag ** 2, "valid": ok}
    n, L, fs = len(seg[0]), int(seg[1][0]), float(seg[2][0])
    x = x.view(n, L)
    if case["kind"] == "search":
        stat, used = torch.zeros(int(K.sum()), dtype=torch.float64, device=DEV), np.zeros(len(mc), np.int32)
        for m in range(len(mc)):
            b = _beta(mc[m], f0[m])
            ok = np.flatnonzero(_valid(b, f0[m], seg[3], L, fs, f_max[m]))
            used[m] = len(ok)
            if len(ok):
                X = _sums(x[torch.as_tensor(ok, device=DEV)], _dtau(b, seg[3][ok], L, fs), f_lo[m], df[m], int(K[m]))
                stat[m * K[m]:(m + 1) * K[m]] = (X.real ** 2 + X.imag ** 2).sum(0)
        return {"stat": stat, "used": torch.from_numpy(used)}
    out = torch.empty(len(mc), n, int(K[0]), dtype=torch.complex128, device=DEV)
    for m in range(len(mc)):               # every segment has the same resampled times
        tau = _dtau(_beta(mc[m], f0[m]), [0.0], L, fs)
        z = _phasor(f_lo[m], tau)
        for k0 in range(0, int(K[0]), 200):
            k = torch.arange(k0, min(k0 + 200, int(K[0])), dtype=torch.float64, device=DEV)[:, None]
            E = _phasor(k * df[m], tau) * z
            out[m, :, k0:k0 + len(k)] = torch.complex(x @ E.real.T.contiguous(), x @ E.imag.T.contiguous())
    X = out.reshape(-1)
    return {"spectra": torch.view_as_real(X).reshape(-1), "power": X.real ** 2 + X.imag ** 2,
            "valid": torch.ones(n * len(mc), dtype=torch.uint8)}


def _tracks(case):
    """(template, bin, weight) [mass][offset][lag] of the tracks and the segments on each, [mass][segment][offset]."""
    n, S = case["n_seg"], case["t0_steps"]
    betas, b0 = _bank(case["n_beta"])[0], _beta(_masses(case["n_mc"]), BAND_LO)[:, None, None]
    dt = (np.arange(n)[None, None, :] + np.arange(S)[None, :, None] / S) * 30.0
    u = 1.0 - (8.0 / 3.0) * b0 * dt
    f = BAND_LO * np.where(u > 0.0, u, 1.0) ** -0.375
    j = np.floor((f - BAND_LO) / (20.0 / case["n_bins"]) + 0.5)
    on = np.logical_and.accumulate((u > 0.0) & (f <= BAND_HI) & (j >= 0) & (j < case["n_bins"]), axis=2)
    b = b0 / np.where(on, u, 1.0)
    hi = np.clip(np.searchsorted(betas, b), 1, len(betas) - 1)
    k = np.where(np.abs(betas[hi - 1] - b) <= np.abs(betas[hi] - b), hi - 1, hi)
    lags = on.sum(2)                                                     # [mass][offset]
    used = np.minimum(lags[:, None, :], (n - np.arange(n))[None, :, None])
    return np.where(on, k, 0), np.where(on, j, 0).astype(np.int64), np.where(on, f ** (4.0 / 3.0), 0.0), used


def exact(case, seed):
    kind = case["kind"]
    if kind in ("search", "spectra", "ragged"):
        seg, tm, inst = _describe(case)
        n_inst = len(inst[0]) if inst else len(seg[0]) * len(tm[0])
        if float(np.mean(seg[1])) * float(np.mean(tm[4])) * n_inst > 8e10:
            return None                                                  # over the time a check may take
        return _exact_plan(case, seed)
    if kind == "stack":
        n, S, P = case["n_seg"], case["t0_steps"], _stack_inputs(case, seed).double()
        P = P.view(case["n_beta"], n, case["n_bins"])
        k, j, w, used = _tracks(case)
        kt, jt, wt = (torch.as_tensor(a, device=DEV) for a in (k, j, w))
        out = torch.empty(case["n_mc"], n, S, dtype=torch.float64, device=DEV)
        for i in range(n):                                               # start segment
            seg = torch.arange(i, n, device=DEV)
            v = (P[kt[..., :n - i], seg, jt[..., :n - i]] * (2.0 / 15360.0) - 2.0) / 2.0
            ww = wt[..., :n - i]
            norm = (ww * ww).sum(2).sqrt()
            out[:, i, :] = torch.where(norm > 0, (ww * v).sum(2) / norm.clamp_min(1e-300), torch.zeros_like(norm))
        return {"n_sigma": out.view(case["n_mc"], n * S),
                "used": torch.as_tensor(used.astype(np.int32)).view(case["n_mc"], n * S)}
    if kind == "rank":
        n_mc, n_sub, K = case["n_mc"], case["n_sub"], case["n_bins"]
        stat, used = _rank_inputs(case, seed)
        S, N = stat.double().view(n_mc, n_sub, K), used.double().view(n_mc, n_sub, 1)
        z = (S / 7680.0 - N) / N.sqrt()
        ks = stat.view(n_mc, n_sub, K).cpu().numpy().argmax(2)
        rows = np.clip(np.arange(n_mc)[:, None] - 3 + np.arange(8), 0, n_mc - 1)
        cols = np.clip(ks[..., None] - 3 + np.arange(8), 0, K - 1)       # [mass][sub][8]
        f = z.cpu().numpy()[rows[:, None, :, None], np.arange(n_sub)[None, :, None, None], cols[:, :, None, :]]
        f = torch.from_numpy(f.reshape(n_mc * n_sub, 64))
        W1, b1, W2, b2, w3, b3 = _net_parts(torch.from_numpy(_he_uniform(seed)))
        W1, W2, w3 = (a.bfloat16().double() for a in (W1, W2, w3))       # the weights as the products hold them
        h = torch.relu(torch.relu(f @ W1.T + b1.double()) @ W2.T + b2.double())
        return {"features": f, "logits": h @ w3 + b3.double(), "z": z.amax(2).view(-1), "arg": None, "top": None}
    if kind == "train":
        x, y = (a.double().cpu() for a in _train_inputs(case, seed))
        p = [a.double() for a in _net_parts(torch.from_numpy(_he_uniform(seed)))]
        for i in (0, 2, 4):
            p[i] = p[i].float().bfloat16().double()
        p = [a.requires_grad_() for a in p]
        t = torch.relu(torch.relu(x @ p[0].T + p[1]) @ p[2].T + p[3]) @ p[4] + p[5]
        loss = torch.nn.functional.binary_cross_entropy_with_logits(t, y)
        g = torch.autograd.grad(loss, p)
        return {"grad": torch.cat([a.reshape(-1) for a in g]), "loss": loss.detach().view(1)}
    x = _fold_input(case, seed).cpu().numpy().reshape(case["n_seg"], -1)
    n, fs, fold = case["n_samples"], case["fs_o"], _fold_size(case)
    b = _beta(FOLD_MC, FOLD_F0)
    a = 3.0 / (5.0 * b)
    M = int(math.floor(-a * math.expm1(0.625 * math.log1p(-(8.0 / 3.0) * b * ((n - 1) / fs))) * fs)) + 1
    q = np.rint(-np.expm1(1.6 * np.log1p(-(np.arange(M) / fs) / a)) * (3.0 / (8.0 * b)) * fs).astype(np.int64)
    y = np.where((q >= 0) & (q < n), x[:, np.clip(q, 0, n - 1)], 0.0).astype(np.complex128)
    y = np.pad(y, ((0, 0), (0, -M % fold))).reshape(case["n_seg"], -1, fold)
    return {"fold": y.sum(1)}
