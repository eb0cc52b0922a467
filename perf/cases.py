"""Performance cases: the work that a search, an injection campaign and the surrogate do
through the package's public entry points, with seeded inputs and 64-bit expectations.

Every case is a dict of plain values; its "kind" says which calls a pass makes:

grid      one frequency band of an all-sky search: load the band's SFT table, evaluate the
          f0 x f1 x sky bank, read the statistics and every sub-band's toplist
list      follow-up of an unstructured list of isolated-source templates on loaded data
bank      a random bank of binary-system templates on loaded data (the paper's timed work)
boxes     the hyperbox search of such a bank: the loudest template of every box
trial     one mismatch / sensitivity trial: generate data with a signal, evaluate the
          signal's own template, then a small random bank around it
campaign  a batch of uneven injection-recovery runs (generated tables, one call)
labels    detection labels of the surrogate: many small local banks on a long SFT set
train     the surrogate's training from given initial parameters
predict   surrogate queries
"""
import math

import numpy as np
import torch

from paper_2411_18370_amd import fasttracks as ft
from paper_2411_18370_amd import mismatch, surrogate, synth

T_SFT = 1800.0


def listed():
    return [
        # the smallest search call there is (the smoke test's bank): launches and host latency
        {"name": "grid_smallest", "kind": "grid", "n_det": 1, "n_per_det": 100, "f_lo": 100.0, "n_f0": 180,
         "n_f1": 3, "n_sky": 20, "k": 10, "n_sub": 1, "sft_weights": False, "sky_weights": False, "count": False},
        # an ordinary weighted search: noise weights per SFT, all-sky weights, odd sizes
        {"name": "grid_weighted", "kind": "grid", "n_det": 2, "n_per_det": 1500, "f_lo": 150.0, "n_f0": 437,
         "n_f1": 3, "n_sky": 1201, "k": 20, "n_sub": 4, "sft_weights": True, "sky_weights": True, "count": False},
        # a part of the sky of the benchmark's all-sky band (200-200.5 Hz, 11 spindowns, 1e4 SFTs)
        {"name": "grid_allsky", "kind": "grid", "n_det": 2, "n_per_det": 5000, "f_lo": 200.0, "n_f0": 900,
         "n_f1": 11, "n_sky": 4000, "k": 100, "n_sub": 10, "sft_weights": False, "sky_weights": False,
         "count": False},
        # follow-up of candidates: templates without structure, in a band of 0.25 Hz
        {"name": "list_followup", "kind": "list", "n": 200_000, "n_per_det": 2500, "f_lo": 200.0, "width": 0.25,
         "k": 50, "sft_weights": False, "count": False},
        # the mismatch study's loop body at its oversampling 3.44 (about 1.2e4 templates per bank)
        {"name": "trial", "kind": "trial", "n_per_det": 5000, "o": 3.44, "k": 1},
        # the paper's benchmark banks of binary-system templates: a small and a large batch
        {"name": "bank_1e5", "kind": "bank", "n": 100_000, "n_per_det": 5000, "k": 10, "n_sub": 5,
         "sky_weights": False, "count": False},
        {"name": "bank_2e6", "kind": "bank", "n": 2_000_000, "n_per_det": 5000, "k": 10, "n_sub": 5,
         "sky_weights": False, "count": False},
        # the search step over hyperboxes (the benchmark's partition), in one batch of its bank
        {"name": "boxes_4e6", "kind": "boxes", "n": 4_000_000, "n_per_det": 5000, "n_div": "1,12,4,1,24,9",
         "count": False},
        # injection-recovery runs of uneven sizes (the benchmark's ranges), an eighth of its batch
        {"name": "campaign_64", "kind": "campaign", "n_runs": 64, "n_pool": 5000, "nt_hi": 1e5},
        # a quarter of one chunk of the label campaign on the all-sky SFT set
        {"name": "labels_1024", "kind": "labels", "n_runs": 1024, "n_per_det": 5000},
        # the surrogate: a pass of its training at the schedule's batch, and a block of queries
        {"name": "train_131072", "kind": "train", "n": 131_072, "batch": 2048, "epochs": 1},
        {"name": "predict_200000", "kind": "predict", "n": 200_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["grid", "grid", "grid", "list", "list", "trial", "bank", "bank", "bank", "boxes", "campaign",
                       "labels", "train", "predict"])
    if kind == "grid":
        c = {"kind": kind, "n_det": rng.choice([1, 2]), "n_per_det": _log_int(rng, 30, 5000),
             "f_lo": round(rng.uniform(60.0, 400.0), 3), "n_f0": _log_int(rng, 20, 2000), "n_f1": rng.randint(1, 12),
             "n_sky": _log_int(rng, 4, 4000), "k": _log_int(rng, 1, 100), "n_sub": rng.randint(1, 10),
             "sft_weights": rng.random() < 0.4, "sky_weights": rng.random() < 0.3, "count": rng.random() < 0.3}
        # at most the largest listed bank and half its evaluations
        while c["n_f0"] * c["n_f1"] * c["n_sky"] * c["n_det"] * c["n_per_det"] > 2e11 or \
                c["n_f0"] * c["n_f1"] * c["n_sky"] > 2e7:
            c["n_sky"] = max(4, c["n_sky"] // 2)
        return c
    if kind == "list":
        return {"kind": kind, "n": _log_int(rng, 200, 400_000), "n_per_det": _log_int(rng, 50, 4000),
                "f_lo": round(rng.uniform(60.0, 400.0), 3), "width": round(rng.uniform(0.05, 0.5), 3),
                "k": _log_int(rng, 1, 100), "sft_weights": rng.random() < 0.4, "count": rng.random() < 0.3}
    if kind == "trial":
        return {"kind": kind, "n_per_det": _log_int(rng, 400, 5000), "o": round(rng.uniform(1.0, 10.0), 2),
                "k": rng.choice([1, 1, 16])}
    if kind == "bank":
        return {"kind": kind, "n": _log_int(rng, 1000, 2_000_000), "n_per_det": _log_int(rng, 50, 5000),
                "k": _log_int(rng, 1, 100), "n_sub": rng.randint(1, 10), "sky_weights": rng.random() < 0.2,
                "count": rng.random() < 0.3}
    if kind == "boxes":
        return {"kind": kind, "n": _log_int(rng, 20_000, 2_000_000), "n_per_det": _log_int(rng, 100, 5000),
                "n_div": rng.choice(["1,12,4,1,24,9", "2,3,5,1,7,2", "1,40,16,1,32,5"]), "count": rng.random() < 0.3}
    if kind == "campaign":
        return {"kind": kind, "n_runs": rng.randint(2, 64), "n_pool": _log_int(rng, 800, 5000),
                "nt_hi": float(_log_int(rng, 3000, 100_000))}
    if kind == "labels":
        return {"kind": kind, "n_runs": _log_int(rng, 16, 1024), "n_per_det": _log_int(rng, 250, 5000)}
    if kind == "train":
        return {"kind": kind, "n": _log_int(rng, 3000, 100_000), "batch": rng.choice([256, 1000, 2048, 4096]),
                "epochs": 1}
    return {"kind": "predict", "n": _log_int(rng, 1, 200_000)}


# --- inputs ------------------------------------------------------------------------------
def _times(n_det, n_per_det, t_sft, stride, rng):
    """Mid-times, velocities and arms of the detectors' SFTs (10% of the slots missing)."""
    t, v, a = [], [], []
    for d in range(n_det):
        slots = np.sort(rng.choice(int(math.ceil(n_per_det / 0.9)), size=n_per_det, replace=False))
        td = synth.EPOCH + slots.astype(np.float64) * stride + 0.5 * t_sft
        t.append(td)
        v.append(synth.detector_velocity(td, synth.DETECTORS[d]))
        a.append(synth.detector_arms(td, synth.DETECTORS[d]))
    return np.concatenate(t), np.concatenate(v), np.concatenate(a)


def _noise(n_sft, n_bins, seed):
    """chi^2 noise power with two degrees of freedom, float32 [n_sft, n_bins], on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    u = torch.rand((n_sft, n_bins), generator=g, device="cuda", dtype=torch.float64)
    return (-2.0 * torch.log1p(-u)).to(torch.float32).contiguous()


def _sft_weights(n, rng):
    return rng.uniform(0.5, 1.5, n).astype(np.float32)


def _grid_inputs(case, seed):
    rng = np.random.default_rng(seed)
    t, v, arms = _times(case["n_det"], case["n_per_det"], T_SFT, T_SFT, rng)
    n_f0, n_sub = case["n_f0"], min(case["n_sub"], case["n_f0"])
    f0 = case["f_lo"] + np.arange(n_f0) / T_SFT
    f1 = np.linspace(-1e-9, 0.0, case["n_f1"]) if case["n_f1"] > 1 else np.array([-1e-10])
    sky = synth.isotropic_sky(case["n_sky"], rng)
    dt = t - synth.EPOCH
    vmax = float(np.max(np.linalg.norm(v, axis=1)))
    first, n_bins = synth.table_range(f0.min(), f0.max(), f1.min(), f1.max(), dt.min(), dt.max(), vmax, T_SFT)
    w = _sft_weights(t.size, rng) if case["sft_weights"] else None
    per = n_f0 // n_sub
    edges = np.array([f0[0] + (j * per - 0.5) / T_SFT for j in range(n_sub)] + [f0[-1] + 0.5 / T_SFT])
    return dict(n_det=case["n_det"], t=t, v=v, arms=arms, t_sft=T_SFT, first=first, n_bins=n_bins,
                power=_noise(t.size, n_bins, seed), weight=w, f0=f0, f1=f1, sky=sky, edges=edges)


def _list_inputs(case, seed):
    rng = np.random.default_rng(seed)
    n = case["n"]
    t, v, arms = _times(2, case["n_per_det"], T_SFT, T_SFT, rng)
    f0 = rng.uniform(case["f_lo"], case["f_lo"] + case["width"], n)
    f1 = rng.uniform(-1e-9, 0.0, n)
    sky = synth.isotropic_sky(n, rng)
    dt = t - synth.EPOCH
    vmax = float(np.max(np.linalg.norm(v, axis=1)))
    first, n_bins = synth.table_range(case["f_lo"], case["f_lo"] + case["width"], -1e-9, 0.0, dt.min(), dt.max(),
                                      vmax, T_SFT)
    w = _sft_weights(t.size, rng) if case["sft_weights"] else None
    edges = np.array([case["f_lo"], case["f_lo"] + 0.5 * case["width"], case["f_lo"] + case["width"]])
    return dict(n_det=2, t=t, v=v, arms=arms, t_sft=T_SFT, first=first, n_bins=n_bins,
                power=_noise(t.size, n_bins, seed), weight=w, f0=f0, f1=f1, sky=sky, edges=edges)


def _binary_inputs(case, seed, noise=True):
    """The search set-up of half-overlapping 1024-s SFTs in 110.5-110.625 Hz, periods 7-15 d,
    a_p 5-15 light-seconds, the whole sky and orbital phase."""
    w = synth.binary_band(seed=seed, n_tmpl=1, n_per_det=case["n_per_det"], with_noise=False,
                          n_sub=case.get("n_sub", 1))
    power = _noise(w.n_sft, w.n_bins, seed) if noise else None
    return w, power


def _trial_inputs(case, seed):
    w, _ = _binary_inputs(case, seed, noise=False)
    rng = np.random.default_rng(seed)
    t_obs = float(w.t_mid.max() - w.t_mid.min() + w.t_sft)
    vmax = float(np.max(np.linalg.norm(w.v, axis=1)))
    inner = dict(w.region, f0_lo=w.region["f0_lo"] + 0.01, f0_hi=w.region["f0_hi"] - 0.01)
    lam = mismatch.draw_signal(rng, inner)
    f0, alpha, sdec, ap, om, pb = lam
    cd = math.sqrt(1.0 - sdec * sdec)
    n = np.array([cd * math.cos(alpha), cd * math.sin(alpha), sdec])
    n /= np.linalg.norm(n)
    inj = dict(amp=1.0, cos_iota=float(rng.uniform(-1, 1)), psi=float(rng.uniform(-np.pi / 4, np.pi / 4)), sky=n,
               f0=f0, f1=0.0, ap=ap, omega=om, phib=pb)
    box = mismatch.box_around(lam, 2.0, w, t_obs, vmax)
    # the box at shorter SFT sets is wider in templates' units: keep the study's bank sizes
    n_bank = min(max(1, int(round(case["o"] * mismatch.n_templates(box, w.t_sft, t_obs, vmax)))), 40_000)
    seeds = (int(rng.integers(1, 2 ** 62)), int(rng.integers(1, 2 ** 62)))
    edges = np.array([w.region["f0_lo"] - 1.0, w.region["f0_hi"] + 1.0])
    return w, inj, box, n_bank, seeds, edges


def _mlp_inputs(case, seed):
    """Raw inputs over the label campaign's ranges, labels that fall off with depth, and
    He-initialised parameters."""
    rng = np.random.default_rng(seed)
    n = case["n"]
    lo, hi = surrogate.AMP_RANGE
    raw = np.stack([np.exp(rng.uniform(math.log(lo), math.log(hi), n)), rng.uniform(-1, 1, n),
                    rng.uniform(-np.pi / 4, np.pi / 4, n), rng.uniform(-1, 1, n), rng.uniform(0, 2 * np.pi, n),
                    rng.uniform(100.0, 300.0, n)], axis=1).astype(np.float32)
    eff = raw[:, 0] * np.sqrt(0.25 * (1.0 + raw[:, 1] ** 2) ** 2 + raw[:, 1] ** 2)
    y = (eff + rng.normal(0.0, 0.004, n) > 0.02).astype(np.float32)
    parts = []
    for fan, cnt, bias in ((6, 256 * 6, 256), (256, 256 * 256, 256), (256, 256 * 256, 256), (256, 256, 1)):
        parts += [rng.normal(0.0, math.sqrt(2.0 / fan), cnt), np.zeros(bias)]
    return raw, y, np.concatenate(parts).astype(np.float32)


# --- preparation and one pass --------------------------------------------------------------
def _context():
    return ft.Context(0, torch.cuda.current_stream().cuda_stream)


def _load(c, d):
    c.set_sfts([d["t"].size // d["n_det"]] * d["n_det"], d["t"], d["t_sft"], d["first"], d["power"], d["weight"])
    c.set_velocities(d["v"])


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "c": _context()}
    c = s["c"]
    if kind == "grid":
        s["d"] = _grid_inputs(case, seed)
        s["stats"] = torch.empty(case["n_f0"] * case["n_f1"] * case["n_sky"], dtype=torch.float32, device="cuda")
    elif kind == "list":
        s["d"] = _list_inputs(case, seed)
        s["stats"] = torch.empty(case["n"], dtype=torch.float32, device="cuda")
        _load(c, s["d"])
    elif kind in ("bank", "boxes"):
        w, power = _binary_inputs(case, seed)
        s["w"], s["seed"] = w, seed
        c.set_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, w.first_bin, power)
        c.set_velocities(w.v)
        s["stats"] = torch.empty(case["n"], dtype=torch.float32, device="cuda")
        if kind == "bank" and case["sky_weights"]:
            c.set_arms(w.arms)
        if kind == "boxes":
            s["n_div"] = [int(x) for x in case["n_div"].split(",")]
            s["region"] = dict(w.region, alpha_lo=0.0, alpha_hi=2 * np.pi, sdec_lo=-1.0, sdec_hi=1.0, phib_lo=0.0,
                               phib_hi=2 * np.pi)
        torch.cuda.synchronize()
    elif kind == "trial":
        s["in"] = _trial_inputs(case, seed)
    elif kind == "campaign":
        s["cp"] = synth.campaign(case["n_runs"], seed=seed, n_pool=case["n_pool"],
                                 n_sft_range=(case["n_pool"] // 10, case["n_pool"]), nt_range=(1e3, case["nt_hi"]))
    elif kind == "labels":
        base = synth.allsky_band(seed=2, n_sky=1, n_per_det=case["n_per_det"])
        s["cp"], _ = synth.label_campaign(case["n_runs"], seed, base)
    elif kind == "train":
        s["raw"], s["y"], s["params"] = _mlp_inputs(case, seed)
        s["seed"] = seed
    elif kind == "predict":
        s["raw"], _, params = _mlp_inputs(case, seed)
        s["net"] = ft.Mlp(c, surrogate.FEAT_SHIFT, surrogate.FEAT_SCALE, max_batch=8192, params=params)
        s["net"].owner = c  # the network is closed before its context
    return s


def _tops(c, n_sub, k):
    tops = [c.toplist(j, k) for j in range(n_sub)]
    return {"index": [np.array([e.index for e in t], np.int64) for t in tops],
            "s64": [np.array([e.s64 for e in t]) for t in tops], "z": [np.array([e.z for e in t]) for t in tops]}


def _stat(case):
    return ft.FT_STAT_NUMBER_COUNT if case.get("count") else ft.FT_STAT_POWER


def _wts(case):
    return ft.FT_WEIGHTS_SKY if case.get("sky_weights") else ft.FT_WEIGHTS_SFT


def run(s):
    case, c = s["case"], s["c"]
    kind = case["kind"]
    if kind == "grid":
        d = s["d"]
        _load(c, d)
        if case["sky_weights"]:
            c.set_arms(d["arms"])
        c.eval_templates(d["f0"], d["f1"], d["sky"], synth.EPOCH, case["k"], d["edges"], stats=s["stats"],
                         statistic=_stat(case), weights=_wts(case))
        return dict(_tops(c, len(d["edges"]) - 1, case["k"]), stats=s["stats"])
    if kind == "list":
        d = s["d"]
        c.eval_templates(d["f0"], d["f1"], d["sky"], synth.EPOCH, case["k"], d["edges"], kind=ft.FT_BANK_LIST,
                         stats=s["stats"], statistic=_stat(case))
        return dict(_tops(c, len(d["edges"]) - 1, case["k"]), stats=s["stats"])
    if kind == "bank":
        w = s["w"]
        c.eval_binary_random(w.region, s["seed"], case["n"], w.t_ref, case["k"], w.sub_edges, stats=s["stats"],
                             statistic=_stat(case), weights=_wts(case))
        return dict(_tops(c, len(w.sub_edges) - 1, case["k"]), stats=s["stats"])
    if kind == "boxes":
        r = c.eval_binary_boxes(s["region"], s["seed"], case["n"], s["w"].t_ref, s["n_div"], statistic=_stat(case),
                                stats=s["stats"])
        return {"index": r["index"].copy(), "count": r["count"].copy(), "s32": r["s32"].copy(),
                "s64": r["s64"].copy(), "z": r["z"].copy(), "stats": s["stats"]}
    if kind == "trial":
        w, inj, box, n_bank, seeds, edges = s["in"]
        c.gen_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, w.first_bin, w.n_bins, w.v, w.arms, seeds[0], 0, w.t_ref, inj)
        c.eval_binary(np.array([inj["f0"]]), inj["sky"][None, :], np.array([inj["ap"]]), np.array([inj["omega"]]),
                      np.array([inj["phib"]]), w.t_ref, 1, edges)
        own = _tops(c, 1, 1)
        c.eval_binary_random(box, seeds[1], n_bank, w.t_ref, case["k"], edges)
        return {"own": own, "bank": _tops(c, 1, case["k"])}
    if kind in ("campaign", "labels"):
        c.eval_campaign(s["cp"])
        labels, max_z = c.batch_labels(9.5, s["cp"].n_runs)
        return {"labels": labels, "max_z": max_z}
    if kind == "train":
        net = ft.Mlp(c, surrogate.FEAT_SHIFT, surrogate.FEAT_SCALE, max_batch=8192, params=s["params"])
        loss = net.train(s["raw"], s["y"], batch=case["batch"], epochs=case["epochs"], lr=2e-3, seed=s["seed"])
        out = {"params": net.params(), "loss": loss}
        net.close()
        return out
    return {"p": s["net"].predict(s["raw"])}


# --- the work a pass cannot do without -----------------------------------------------------
def work(case):
    """Inputs read and outputs written once; operations per template-SFT pair: one addition
    (grids, whose bins follow from one per run), 10 with an own bin (lists), 20 with an
    orbital phase (binary banks); 150 per generated table cell; the network's products."""
    kind = case["kind"]
    if kind in ("train", "predict"):
        macs = 256 * 6 + 2 * 256 * 256 + 256
        n = case["n"]
        if kind == "predict":
            return {"bytes": n * 28.0 + 4 * 133_633, "flops": 2.0 * macs * n}
        return {"bytes": case["epochs"] * n * 28.0 + 2 * 4 * 133_633, "flops": 6.0 * macs * n * case["epochs"]}
    if kind == "campaign":
        # means of the uneven ranges: SFTs, template count (log-uniform), table columns
        n_sft = 0.55 * case["n_pool"]
        n_t = (case["nt_hi"] - 1e3) / math.log(case["nt_hi"] / 1e3)
        cells = n_sft * 300
        return {"bytes": case["n_runs"] * 4.0 * (cells + n_t), "flops": case["n_runs"] * (n_sft * n_t + 150.0 * cells)}
    if kind == "labels":
        n_sft = 2 * case["n_per_det"]
        return {"bytes": case["n_runs"] * 4.0 * n_sft * 20,
                "flops": case["n_runs"] * n_sft * (5 * 11 * 16 + 150.0 * 20)}
    n_sft = case.get("n_det", 2) * case["n_per_det"]
    if kind == "grid":
        n_t = case["n_f0"] * case["n_f1"] * case["n_sky"]
        cols = case["n_f0"] + 2e-4 * case["f_lo"] * T_SFT + 1e-9 * n_sft * T_SFT * T_SFT / case["n_det"]
        return {"bytes": 4.0 * n_sft * cols + 32.0 * n_sft + 24.0 * case["n_sky"] + 4.0 * n_t, "flops": 1.0 * n_t * n_sft}
    if kind == "list":
        cols = (case["width"] + 2e-4 * case["f_lo"] + 1e-9 * n_sft / 2 * T_SFT) * T_SFT
        return {"bytes": 4.0 * n_sft * cols + 32.0 * n_sft + 44.0 * case["n"], "flops": 10.0 * case["n"] * n_sft}
    cols = 190.0
    if kind == "trial":
        n_t = 3500.0 * case["o"]
        return {"bytes": 4.0 * n_sft * cols + 80.0 * n_sft, "flops": n_sft * (20.0 * n_t + 150.0 * cols)}
    return {"bytes": 4.0 * n_sft * cols + 32.0 * n_sft + 4.0 * case["n"], "flops": 20.0 * case["n"] * n_sft}


# --- 64-bit expectations ---------------------------------------------------------------------
def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _ab(arms, n):
    """a^2 + b^2 of one SFT's detector for the directions n [m, 3]."""
    u, w = arms[:3], arms[3:]
    x, y, c = n @ u, n @ w, float(u @ w)
    return (1 - c * c) - (x * x + y * y - 2 * c * x * y) + 0.25 * (x * x - y * y) ** 2


def _sums(t, v, t_sft, t_ref, first, table, weight, arms, track, n_dir, shape):
    """Sum over the SFTs of w_k P_k[B_k] and of w_k and w_k^2; track(k, dt, g) gives f(t_k),
    g = 1 + v.n per direction; with arms the weights are u_k (a^2 + b^2) (not normalised)."""
    acc = torch.zeros(shape, dtype=torch.float64, device="cuda")
    w1 = torch.zeros(n_dir.shape[0] if arms is not None else 1, dtype=torch.float64, device="cuda")
    w2 = torch.zeros_like(w1)
    for k in range(t.size):
        vx, vy, vz = (float(x) for x in v[k])
        g = 1.0 + ((vx * n_dir[:, 0] + vy * n_dir[:, 1]) + vz * n_dir[:, 2])
        b = torch.floor(track(float(t[k] - t_ref), g) * t_sft + 0.5).to(torch.int64) - first
        val = table[k][b]
        u = 1.0 if weight is None else float(weight[k])
        if arms is None:
            acc += u * val
            w1 += u
            w2 += u * u
        else:
            wk = u * _ab(arms[k], n_dir)
            acc += wk.view(-1, *([1] * (len(shape) - 1))) * val
            w1 += wk
            w2 += wk * wk
    return acc, w1, w2


def _finish(case, acc, w1, w2, f0_of, edges, k):
    """Statistics, and per sub-band the k largest with their critical ratios."""
    sky = bool(case.get("sky_weights"))
    if sky:
        full = (-1,) + (1,) * (acc.dim() - 1)
        acc = acc / w1.view(full)
        ones, w2 = torch.ones_like(w1), w2 / (w1 * w1)
        w1 = ones
    p = math.exp(-1.6)
    mu = p * w1 if case.get("count") else 2.0 * w1
    sd = torch.sqrt(p * (1 - p) * w2) if case.get("count") else 2.0 * torch.sqrt(w2)
    per = acc[0].numel() if sky else acc.numel()
    flat = acc.reshape(-1)
    s64, z = [], []
    for lo, hi in zip(edges[:-1], edges[1:]):
        idx = torch.nonzero((f0_of >= lo) & (f0_of < hi)).reshape(-1)
        top = torch.topk(flat[idx], min(k, idx.numel()))
        at = idx[top.indices] // per
        s64.append(top.values.cpu().numpy())
        z.append(((top.values - mu[at]) / sd[at]).cpu().numpy())
    return {"index": [None] * len(s64), "s64": s64, "z": z, "stats": flat}


def _indicator(case, table):
    return (table > 3.2).to(torch.float64) if case.get("count") else table


def _philox(c, seed):
    """Philox-4x32-10 (Salmon et al., SC'11) on arrays of four 32-bit counter words."""
    m32 = np.uint64(0xFFFFFFFF)
    c = [np.asarray(x, np.uint64) for x in c]
    k0, k1 = np.uint64(seed & 0xFFFFFFFF), np.uint64(seed >> 32)
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        s = np.uint64(32)
        c = [(p1 >> s) ^ c[1] ^ k0, p1 & m32, (p0 >> s) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + np.uint64(0x9E3779B9)) & m32, (k1 + np.uint64(0xBB67AE85)) & m32
    s11 = np.uint64(11)
    return [((((c[2 * j] << np.uint64(32)) | c[2 * j + 1]) >> s11).astype(np.float64) + 0.5) * 2.0 ** -53
            for j in (0, 1)]


def _random_bank(region, seed, n):
    """Templates uniform in (f0^6, alpha, sin delta, a_p^3, Omega^4, phi_b)."""
    r = dict(alpha_lo=0.0, alpha_hi=2 * np.pi, sdec_lo=-1.0, sdec_hi=1.0, phib_lo=0.0, phib_hi=2 * np.pi)
    r.update(region)
    i = np.arange(n, dtype=np.uint64)
    z = np.zeros_like(i)
    u = []
    for j in range(3):
        u += _philox([i, z, z, z + np.uint64(1 + j)], seed)

    def root(lo, hi, x, p):  # Newton from the closed form, so the root is good to the last bits
        y = lo ** p + x * (hi ** p - lo ** p)
        q = y ** (1.0 / p)
        return q - (q ** p - y) / (p * q ** (p - 1))

    alpha = r["alpha_lo"] + u[1] * (r["alpha_hi"] - r["alpha_lo"])
    sd = r["sdec_lo"] + u[2] * (r["sdec_hi"] - r["sdec_lo"])
    cd = np.sqrt(1.0 - sd * sd)
    sky = np.stack([cd * np.cos(alpha), cd * np.sin(alpha), sd], axis=1)
    return (root(r["f0_lo"], r["f0_hi"], u[0], 6), sky, root(r["ap_lo"], r["ap_hi"], u[3], 3),
            root(r["omega_lo"], r["omega_hi"], u[4], 4), r["phib_lo"] + u[5] * (r["phib_hi"] - r["phib_lo"]))


def _binary_sums(w, table, weight, arms, bank):
    f0, sky, ap, om, pb = (_dev(x) for x in bank)

    def track(dt, g):
        return f0 * (g - (ap * om) * torch.cos(om * dt - pb))

    acc, w1, w2 = _sums(w.t_mid, w.v, w.t_sft, w.t_ref, w.first_bin, table, weight, arms, track, sky, (len(bank[0]),))
    return acc, w1, w2, f0


def _trial_table(w, inj, seed):
    """Noise from the published generator and Box-Muller, plus the signal's three bins per SFT."""
    n = w.t_mid.size
    k, b = np.meshgrid(np.arange(n, dtype=np.uint64), np.arange(w.n_bins, dtype=np.uint64), indexing="ij")
    u1, u2 = _philox([b, k, np.zeros_like(b), np.zeros_like(b)], seed)
    r = np.sqrt(-2.0 * np.log(u1))
    re, im = r * np.cos(2 * np.pi * u2), r * np.sin(2 * np.pi * u2)
    sky = np.asarray(inj["sky"])
    dt = w.t_mid - w.t_ref
    f = inj["f0"] * (1.0 + w.v @ sky - inj["ap"] * inj["omega"] * np.cos(inj["omega"] * dt - inj["phib"]))
    x = f * w.t_sft
    B = np.floor(x + 0.5)
    rho = math.hypot(sky[0], sky[1])
    ea = np.array([-sky[1] / rho, sky[0] / rho, 0.0])
    ed = np.array([-sky[2] * sky[0] / rho, -sky[2] * sky[1] / rho, rho])
    cp, sp = math.cos(inj["psi"]), math.sin(inj["psi"])
    p, q = cp * ea + sp * ed, -sp * ea + cp * ed
    up, uq, wp, wq = w.arms[:, :3] @ p, w.arms[:, :3] @ q, w.arms[:, 3:] @ p, w.arms[:, 3:] @ q
    fp, fx = 0.5 * ((up * up - uq * uq) - (wp * wp - wq * wq)), up * uq - wp * wq
    ci = inj["cos_iota"]
    amp = np.sqrt(w.t_sft * inj["amp"] ** 2 * (fp * fp * (0.5 * (1 + ci * ci)) ** 2 + fx * fx * ci * ci))
    for m in (-1, 0, 1):
        col = (B + m).astype(np.int64) - w.first_bin
        ok = (col >= 0) & (col < w.n_bins)
        re[np.nonzero(ok)[0], col[ok]] += (amp * np.abs(np.sinc(x - B - m)))[ok]
    return _dev((re * re + im * im).astype(np.float32).astype(np.float64))


class _Mt64:
    """The 64-bit Mersenne Twister (Matsumoto and Nishimura), as the C++ standard states it."""

    def __init__(self, seed):
        mask = (1 << 64) - 1
        self.x = [seed & mask]
        for i in range(1, 312):
            p = self.x[-1]
            self.x.append((6364136223846793005 * (p ^ (p >> 62)) + i) & mask)
        self.i = 312

    def next(self):
        if self.i == 312:
            lo = (1 << 31) - 1
            for i in range(312):
                y = (self.x[i] & ~lo & ((1 << 64) - 1)) | (self.x[(i + 1) % 312] & lo)
                self.x[i] = self.x[(i + 156) % 312] ^ (y >> 1) ^ (0xB5026F5AA96619E9 if y & 1 else 0)
            self.i = 0
        y = self.x[self.i]
        self.i += 1
        y ^= (y >> 29) & 0x5555555555555555
        y ^= (y << 17) & 0x71D67FFFEDA60000
        y ^= (y << 37) & 0xFFF7EEE000000000
        return y ^ (y >> 43)


def _mlp_features(raw):
    g = _dev(raw.astype(np.float64))
    g = torch.cat([torch.log(g[:, :1]), g[:, 1:]], dim=1)
    return (g - _dev(surrogate.FEAT_SHIFT.astype(np.float32))) / _dev(surrogate.FEAT_SCALE.astype(np.float32))


def _mlp_logit(th, x):
    o = 0
    for fan, width in ((6, 256), (256, 256), (256, 256), (256, 1)):
        wt = th[o:o + fan * width].view(width, fan)
        x = x @ wt.t() + th[o + fan * width:o + fan * width + width]
        if width > 1:
            x = 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))
        o += (fan + 1) * width
    return x[:, 0]


def _train64(case, seed):
    raw, y, params = _mlp_inputs(case, seed)
    x, y, th = _mlp_features(raw), _dev(y), _dev(params)
    n, rng, step, hist = case["n"], _Mt64(seed), 0, []
    m, v = torch.zeros_like(th), torch.zeros_like(th)
    for _ in range(case["epochs"]):
        a = 1 + rng.next() % max(n - 1, 1)
        while math.gcd(a, n) != 1:
            a = a % n + 1
        b = rng.next() % n
        order = (torch.arange(n, device="cuda", dtype=torch.int64) * a + b) % n
        total, batches = 0.0, 0
        for b0 in range(0, n, case["batch"]):
            at = order[b0:b0 + case["batch"]]
            th.requires_grad_(True)
            loss = torch.nn.functional.binary_cross_entropy_with_logits(_mlp_logit(th, x[at]), y[at])
            (g,) = torch.autograd.grad(loss, th)
            th = th.detach()
            step += 1
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            th = th - 2e-3 * (m / (1 - 0.9 ** step)) / (torch.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
            total, batches = total + float(loss), batches + 1
        hist.append(total / batches)
    return {"params": th.cpu().numpy(), "loss": np.array(hist)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("grid", "list"):
        d = _grid_inputs(case, seed) if kind == "grid" else _list_inputs(case, seed)
        sky, f0, f1 = _dev(d["sky"]), _dev(d["f0"]), _dev(d["f1"])
        table = _indicator(case, d["power"].to(torch.float64))
        arms = [_dev(x) for x in d["arms"]] if case.get("sky_weights") else None
        if kind == "list":
            if case["n"] * d["t"].size > 4e9:
                return None
            shape, f0_of = (case["n"],), f0

            def track(dt, g):
                return (f0 + f1 * dt) * g
        else:
            shape = (case["n_sky"], case["n_f1"], case["n_f0"])
            if math.prod(shape) * d["t"].size > 2e10:
                return None
            f0_of = f0.repeat(shape[0] * shape[1])

            def track(dt, g):
                return (f0[None, None, :] + (f1 * dt)[None, :, None]) * g[:, None, None]
        acc, w1, w2 = _sums(d["t"], d["v"], T_SFT, synth.EPOCH, d["first"], table, d["weight"], arms, track, sky, shape)
        return _finish(case, acc, w1, w2, f0_of, d["edges"], case["k"])
    if kind == "bank":
        if case["n"] * case["n_per_det"] > 2e9:
            return None
        w, power = _binary_inputs(case, seed)
        arms = [_dev(x) for x in w.arms] if case["sky_weights"] else None
        bank = _random_bank(w.region, seed, case["n"])
        acc, w1, w2, f0 = _binary_sums(w, _indicator(case, power.to(torch.float64)), None, arms, bank)
        return _finish(case, acc, w1, w2, f0, w.sub_edges, case["k"])
    if kind == "trial":
        w, inj, box, n_bank, seeds, edges = _trial_inputs(case, seed)
        table = _trial_table(w, inj, seeds[0])
        out = {}
        own = tuple(np.array([x]) for x in (inj["f0"], inj["sky"], inj["ap"], inj["omega"], inj["phib"]))
        for name, bank, k in (("own", own, 1), ("bank", _random_bank(box, seeds[1], n_bank), case["k"])):
            acc, w1, w2, f0 = _binary_sums(w, table, None, None, bank)
            out[name] = _finish({}, acc, w1, w2, f0, edges, k)
            out[name].pop("stats")
        return out
    if kind == "train":
        return _train64(case, seed)
    if kind == "predict":
        raw, _, params = _mlp_inputs(case, seed)
        return {"p": torch.sigmoid(_mlp_logit(_dev(params), _mlp_features(raw))).cpu().numpy()}
    return None
