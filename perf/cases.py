"""Performance cases of the library: what programs have it compute, from one
short series to batches of thousands, through the public Python entry points.

A case names a kind of work and its sizes:
  single   one series (Periodogram without offsets), periodogram and peak
  batch    a CSR batch on one grid (Periodogram with offsets), periodograms or
           peaks only
  rows     chosen frequency bands of every object of a batch (Rows), the
           refinement step of the learned path
  features band-proposal features of a batch (Features)
  forward  the proposal network on standardised features (BandNet.forward)
  train    one training step of that network (BandNet.train_step)
`form` is "fp32" or "fp64", `method` "standard" or "generalized" (errors and a
floating mean).  Sizes are those of the synthetic workloads that the benchmark
and the tests use (single_256, single_4096, batch_10k, learned_100k, lsst_200k,
asteroids_1k), the batches with fewer objects.

Peak records are returned by field.  The power of the FP32 form is a single
rounded value (the record widens it), so it is returned as float32 where no
periodogram holds it.
"""
import math

import numpy as np
import torch

from paper_2105_04006_amd import learned, lsp

DEV = "cuda"
F_WIDE, F_MID = (0.5, 24.0), (1.0, 12.0)  # cycles per day
AST_GRID = (1.005, 150.796)               # rad per day


# ------------------------------------------------------------------- the cases

def listed():
    return [
        # one short series, everything at hand: the call of an interactive tool
        # or a serving loop; launches and latency
        dict(name="single_short", kind="single", form="fp32", method="standard", n_t=256,
             n_f=10_000),
        # the same with the library's default options, the FP64 form
        dict(name="single_fp64", kind="single", form="fp64", method="standard", n_t=256,
             n_f=10_000),
        # one well-observed object on a fine grid
        dict(name="single_wide", kind="single", form="fp32", method="standard", n_t=4096,
             n_f=500_000),
        # the same with photometric errors
        dict(name="single_gen", kind="single", form="fp32", method="generalized", n_t=4096,
             n_f=500_000),
        # a survey's batch, peaks only, on the wide grid (sinusoids, second
        # harmonics, noise; 20 to 500 points each)
        dict(name="batch_survey", kind="batch", form="fp32", method="standard", n_obj=2500,
             n_lo=20, n_hi=500, n_f=250_000, mix="lsst", pgram=False),
        # objects of 50 to 1,000 points, whole periodograms kept; an odd grid
        dict(name="batch_pgram", kind="batch", form="fp32", method="standard", n_obj=300,
             n_lo=50, n_hi=1000, n_f=100_003, mix="sine", pgram=True),
        # asteroid-like series with errors (nightly cadence, angular grid)
        dict(name="batch_gen", kind="batch", form="fp32", method="generalized", n_obj=300,
             n_lo=20, n_hi=1500, n_f=200_000, mix="asteroid", pgram=True),
        # FP64 periodograms of a small batch
        dict(name="batch_fp64", kind="batch", form="fp64", method="standard", n_obj=48,
             n_lo=50, n_hi=1000, n_f=40_000, mix="sine", pgram=True),
        # the refinement of three proposed bands per object
        dict(name="rows_refine", kind="rows", form="fp32", method="standard", n_obj=4000,
             n_lo=20, n_hi=500, n_f=200_000, bands=3),
        # features of a batch for the band proposal
        dict(name="features", kind="features", n_obj=1500, n_lo=50, n_hi=500),
        # the proposal network on a batch's features
        dict(name="net_forward", kind="forward", n_obj=20_000),
        # one training step at the minibatch size the training uses
        dict(name="net_train", kind="train", n_obj=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "batch", "batch", "batch", "rows", "features",
                       "forward", "train"])
    if kind == "single":
        form = rng.choice(["fp32", "fp32", "fp64"])
        c = dict(kind=kind, form=form, method=rng.choice(["standard", "standard", "generalized"]),
                 n_t=_log(rng, 50, 4096))
        c["n_f"] = _log(rng, 2_000, 50_000 if form == "fp64" else 500_000)
        return c
    if kind == "batch":
        form = rng.choice(["fp32", "fp32", "fp32", "fp64"])
        method = rng.choice(["standard", "standard", "generalized"])
        mix = rng.choice(["sine", "lsst", "asteroid"])
        n_hi = _log(rng, 60, 1000)
        n_f = _log(rng, 5_000, 250_000)
        most = 1.0e9 if form == "fp64" else 2.0e10  # evaluations
        n_obj = _log(rng, 2, max(3.0, min(2500.0, most / (0.5 * n_hi * n_f))))
        pgram = rng.random() < 0.5 and n_obj * n_f <= 60_000_000
        return dict(kind=kind, form=form, method=method, n_obj=n_obj,
                    n_lo=max(20, n_hi // rng.randint(2, 20)), n_hi=n_hi, n_f=n_f, mix=mix,
                    pgram=pgram)
    if kind == "rows":
        n_lo = rng.randint(20, 100)
        return dict(kind=kind, form="fp32", method="standard", n_obj=_log(rng, 50, 4000),
                    n_lo=n_lo, n_hi=n_lo + _log(rng, 20, 400), n_f=_log(rng, 20_000, 200_000),
                    bands=rng.randint(1, 4))
    if kind == "features":
        n_lo = rng.randint(20, 100)
        return dict(kind=kind, n_obj=_log(rng, 20, 1500), n_lo=n_lo,
                    n_hi=n_lo + _log(rng, 20, 400))
    if kind == "forward":
        return dict(kind=kind, n_obj=_log(rng, 100, 20_000))
    return dict(kind=kind, n_obj=_log(rng, 64, 2048))


# ------------------------------------------------------------------ the inputs

def _seasonal(u):
    """Days of a ten-year span without each year's 120-day gap from u in [0, 2450)."""
    yr = torch.floor(u / 245.0)
    r = u - yr * 245.0
    return yr * 365.0 + torch.where(r < 120.0, r, r + 120.0)


def _series(n_t, mix, seed, errors):
    """CSR series: offsets, t, y, dy (None without errors), seeded, on the GPU."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + 17)
    k = len(n_t)
    cnt = torch.as_tensor(np.asarray(n_t, np.int64), device=DEV)
    off = torch.zeros(k + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(cnt, 0)
    n = int(np.sum(n_t))
    own = torch.repeat_interleave(torch.arange(k, device=DEV), cnt)

    def rand(m):
        return torch.rand(m, generator=g, device=DEV, dtype=torch.float64)

    def normal(m):
        return torch.randn(m, generator=g, device=DEV, dtype=torch.float64)

    if mix == "asteroid":  # three years of nightly visits, half of them in pairs
        t = torch.floor(_seasonal(rand(n) * 735.0)) + 0.15 + 0.2 * rand(n)
        t[1:] = torch.where((rand(n - 1) < 0.5) & (own[1:] == own[:-1]), t[:-1] + 30.0 / 1440.0,
                            t[1:])
        freq = 2.0 * 24.0 / torch.clamp(8.0 * torch.exp(0.9 * normal(k)), min=2.0)
        amp = 0.05 * torch.exp(math.log(6.0) * rand(k))
        sigma = 0.02 * torch.exp(math.log(7.5) * rand(k))
    else:
        t = _seasonal(rand(n) * 2450.0)
        freq = 10.0 ** rand(k)
        amp = torch.full((k,), 0.3, dtype=torch.float64, device=DEV)
        sigma = torch.full((k,), 0.05, dtype=torch.float64, device=DEV)
    order = torch.argsort(own.double() * 1.0e4 + t)
    t = t[order].contiguous()
    phi, phi2, ratio, kind = (2 * math.pi * rand(k), 2 * math.pi * rand(k), 0.1 + 0.4 * rand(k),
                              rand(k))
    if mix == "sine":
        ratio = torch.zeros_like(ratio)
    elif mix == "lsst":  # 60% sinusoids, 30% with a second harmonic, 10% noise
        ratio = torch.where((kind >= 0.6) & (kind < 0.9), ratio, torch.zeros_like(ratio))
        amp = torch.where(kind < 0.9, amp, torch.zeros_like(amp))
    w = 2 * math.pi * freq[own] * t
    y = amp[own] * (torch.sin(w + phi[own]) + ratio[own] * torch.sin(2 * w + phi2[own]))
    dy = None
    if errors:
        dy = torch.clamp(sigma[own] * 10.0 ** (0.2 * normal(n)), 0.005, 0.5)
        y = y + dy * normal(n)
    else:
        y = y + sigma[own] * normal(n)
    return off, t, y.contiguous(), dy


def _counts(case, seed):
    r = np.random.default_rng(77_000 + int(seed))
    if case.get("mix") == "asteroid":
        n = np.round(110.0 * np.exp(0.9 * r.standard_normal(case["n_obj"])))
        return np.clip(n, case["n_lo"], case["n_hi"]).astype(np.int64)
    return r.integers(case["n_lo"], case["n_hi"] + 1, case["n_obj"])


def _inputs(case, seed):
    """What prepare() and exact() share: the case's data and grid."""
    gen = case.get("method") == "generalized"
    if case["kind"] == "single":
        off, t, y, dy = _series([case["n_t"]], "sine", seed, gen)
        grid = F_WIDE if case["n_f"] > 100_000 else F_MID
        return off, t, y, dy, grid, lsp.CYCLES
    mix = case.get("mix", "lsst")
    off, t, y, dy = _series(_counts(case, seed), mix, seed, gen)
    if mix == "asteroid":
        return off, t, y, dy, AST_GRID, lsp.ANGULAR
    return off, t, y, dy, F_WIDE if mix == "lsst" else F_MID, lsp.CYCLES


def _bands(case, seed):
    """Distinct bands of 64 for every object, -1 for a slot that was not kept."""
    r = np.random.default_rng(55_000 + int(seed))
    b = np.argsort(r.random((case["n_obj"], 64)), axis=1)[:, :case["bands"]].astype(np.int32)
    if case["bands"] > 1:
        b[:, 1:][r.random((case["n_obj"], case["bands"] - 1)) < 0.3] = -1
    return b


def _net_inputs(case, seed):
    """Standardised features in BF16 bits, labels, and the network's seed."""
    g = torch.Generator(device=DEV)
    g.manual_seed(999_983 * int(seed) + 5)
    n = case["n_obj"]
    x = torch.randn((n, learned.DIMS[0]), generator=g, device=DEV)
    labels = torch.randint(0, 64, (n,), generator=g, device=DEV, dtype=torch.int32)
    # the coarse columns of the label's band stand out, as a peak does
    cols = labels.long()[:, None] * 16 + torch.arange(16, device=DEV)[None, :]
    x.scatter_add_(1, cols, 2.0 * torch.rand((n, 16), generator=g, device=DEV))
    return x.to(torch.bfloat16).view(torch.int16).contiguous(), labels


def _fields(raw, power32):
    """The fields of device peak records (40 bytes each) as tensors."""
    i = raw.view(torch.int64).view(-1, 5)
    d = raw.view(torch.float64).view(-1, 5)
    out = {"index": i[:, 0], "freq": d[:, 1], "period": d[:, 2], "status": i[:, 4]}
    if power32 is not None:
        out["power"] = d[:, 3].float() if power32 else d[:, 3]
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("forward", "train"):
        x, labels = _net_inputs(case, seed)
        net = learned.BandNet(torch.device(DEV), seed=7)
        if kind == "train":  # in the middle of training: moments that are not zero
            for m, v, p in zip(net.m, net.v, net.master):
                m.copy_(1.0e-4 * torch.sin(torch.arange(p.numel(), device=DEV)).view(p.shape))
                v.fill_(1.0e-4)
            net.step = 50
        return {"case": case, "net": net, "x": x, "labels": labels}
    off, t, y, dy, (f_min, f_max), unit = _inputs(case, seed)
    form = lsp.FORM_FP64 if case.get("form") == "fp64" else lsp.FORM_FP32P
    if kind == "features":
        return {"case": case, "call": lsp.Features(off, t, y, *F_MID)}
    if kind == "rows":
        geo = learned.BandGeometry(case["n_f"])
        bands = torch.as_tensor(_bands(case, seed), device=DEV).view(-1)
        call = lsp.Rows(off, t, y, f_min, f_max, case["n_f"], None, bands, geo.band_bins,
                        case["bands"], unit=unit, form=form)
        return {"case": case, "call": call}
    keep = kind == "single" or case["pgram"]
    call = lsp.Periodogram(
        t, y, f_min, f_max, case["n_f"], offsets=None if kind == "single" else off, unit=unit,
        form=form, pgram=keep, peaks=kind == "single" or not case["pgram"],
        pgram_dtype=lsp.PGRAM_F64 if form == lsp.FORM_FP64 else lsp.PGRAM_F32,
        method=case["method"], dy=dy)
    return {"case": case, "call": call}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "forward":
        return state["net"].forward(state["x"])
    if kind == "train":
        net = state["net"]
        loss = net.train_step(state["x"], state["labels"])
        return {"loss": loss, "grads": list(net.grads), "weights": list(net.master)}
    call = state["call"]
    call()
    if kind == "features":
        return call.out
    narrow = case["form"] != "fp64"
    if kind == "rows":
        return _fields(call.peaks_raw, narrow)
    out = {}
    if call.pgram is not None:
        out["pgram"] = call.pgram
    if call.peaks_raw is not None:
        # beside a periodogram, which holds the peak's power, the other fields
        out.update(_fields(call.peaks_raw, None if call.pgram is not None else narrow))
    return out


def work(case):
    kind = case["kind"]
    d = learned.DIMS
    macs = sum(a * b for a, b in zip(d[:-1], d[1:]))
    par = macs + sum(d[1:])
    if kind == "forward":
        n = case["n_obj"]
        return {"bytes": n * (2.0 * d[0] + 4.0 * d[-1]) + 2.0 * macs, "flops": 2.0 * n * macs}
    if kind == "train":
        n = case["n_obj"]
        # forward, weight gradients, and input gradients of the upper two layers
        flops = 2.0 * n * (3.0 * macs - d[0] * d[1])
        # parameters, moments and gradients in FP32, the BF16 copy read and written
        return {"bytes": n * (2.0 * d[0] + 8.0) + par * (6 * 4.0 + 4.0) + 4.0 * macs,
                "flops": flops}
    if kind == "features":
        n_obs = case["n_obj"] * 0.5 * (case["n_lo"] + case["n_hi"])
        return {"bytes": 16.0 * n_obs + 4.0 * lsp.FEAT_DIM * case["n_obj"],
                "flops": 8.0 * n_obs * lsp.FEAT_COARSE * lsp.FEAT_POOL}
    gen = case["method"] == "generalized"
    sums = 6.0 if gen else 4.0  # multiply-adds per observation and bin
    per_obs = 24.0 if gen else 16.0
    width = 8.0 if case["form"] == "fp64" else 4.0
    if kind == "single":
        return {"bytes": per_obs * case["n_t"] + width * case["n_f"] + 40.0,
                "flops": 2.0 * sums * case["n_t"] * case["n_f"]}
    if case.get("mix") == "asteroid":
        mean = min(case["n_hi"], 165.0)  # log-normal, median 110
    else:
        mean = 0.5 * (case["n_lo"] + case["n_hi"])
    n_obs = case["n_obj"] * mean
    if kind == "rows":
        kept = 1.0 + 0.7 * (case["bands"] - 1)
        return {"bytes": per_obs * n_obs + 40.0 * case["n_obj"] + 4.0 * case["n_obj"] * case["bands"],
                "flops": 2.0 * sums * n_obs * kept * case["n_f"] / 64.0}
    out = width * case["n_obj"] * case["n_f"] if case["pgram"] else 40.0 * case["n_obj"]
    return {"bytes": per_obs * n_obs + out, "flops": 2.0 * sums * n_obs * case["n_f"]}


# ------------------------------------------------------- the results in 64 bits

def _split(x):
    """x = h + l with h on 26 bits, so that products of two such halves are exact."""
    c = 134217729.0 * x
    h = c - (c - x)
    return h, x - h


def _phase(f, t):
    """f t mod 1 for every pair, the products taken exactly."""
    fh, fl = _split(f[:, None])
    th, tl = _split(t[None, :])
    r = fh * th
    r = r - torch.round(r)
    q = fh * tl
    r = r + (q - torch.round(q))
    q = fl * th
    r = r + (q - torch.round(q))
    return r + fl * tl


def _powers(t, y, w, f, floating, norm):
    """Normalised power at frequencies f (cycles): the least-squares sinusoid
    (with an offset if `floating`) under weights w, as a fraction of `norm`."""
    out = torch.empty_like(f)
    tc = t - t.mean()
    step = max(1, int(2.0e7) // max(1, t.numel()))
    for a in range(0, f.numel(), step):
        ph = 2 * math.pi * _phase(f[a:a + step], tc)
        c, s = torch.cos(ph), torch.sin(ph)
        if floating:
            tot = w.sum()
            c = c - ((c @ w) / tot)[:, None]
            s = s - ((s @ w) / tot)[:, None]
        cc, ss, cs = (c * c) @ w, (s * s) @ w, (c * s) @ w
        yc, ys = c @ (w * y), s @ (w * y)
        # rotated so that the cross term vanishes, a vanishing direction dropped
        half = 0.5 * torch.atan2(2 * cs, cc - ss)
        ca, sa = torch.cos(half), torch.sin(half)
        d1 = ca * ca * cc + 2 * ca * sa * cs + sa * sa * ss
        d2 = sa * sa * cc - 2 * ca * sa * cs + ca * ca * ss
        tiny = 1.0e-12 * w.sum()
        zero = torch.zeros_like(d1)
        p = torch.where(d1 > tiny, (ca * yc + sa * ys) ** 2 / d1, zero)
        p = p + torch.where(d2 > tiny, (ca * ys - sa * yc) ** 2 / d2, zero)
        out[a:a + step] = p / norm
    return out


def _object_powers(case, t, y, dy, f):
    if case["method"] == "generalized":
        w = 1.0 / (dy * dy)
        w = w * (w.numel() / w.sum())
        yc = y - (w * y).sum() / w.sum()
        return _powers(t, yc, w, f, True, (w * yc * yc).sum())
    yc = y - y.mean()
    return _powers(t, yc, torch.ones_like(t), f, False, (yc * yc).sum())


def _grid(lo, hi, n_f, unit):
    df = (hi - lo) / n_f
    f = lo + df * torch.arange(n_f, device=DEV, dtype=torch.float64)
    return f, f if unit == lsp.CYCLES else f * (1.0 / (2.0 * math.pi))


def _coarse(t, yc, gap, least):
    """The 1,024 pooled coarse features of one object."""
    f = F_MID[0] + (F_MID[1] - F_MID[0]) / 8192 * torch.arange(8192, device=DEV,
                                                               dtype=torch.float64)
    th = t.cpu().numpy()
    starts = np.concatenate([[0], 1 + np.nonzero(np.diff(th) > gap)[0], [len(th)]])
    total = torch.zeros(1024, device=DEV, dtype=torch.float64)
    a, good = 0, 0
    for e in starts[1:]:
        if e - a < least:
            continue
        tg, yg = t[a:e], yc[a:e]
        p = _powers(tg, yg, torch.ones_like(tg), f, False, (yg * yg).sum())
        total += torch.clamp(p, 0.0, 1.0).view(1024, 8).max(dim=1).values
        good += 1
        a = e
    return total / max(1, good), starts


def _window(t, y, gap, least, starts):
    """The 64 sampling and magnitude statistics of one object."""
    n = t.numel()
    th = t.cpu().numpy()
    yc = (y - y.mean()).cpu().numpy()
    d = np.diff(th)
    d = d[d <= gap]
    ld = np.log10(np.maximum(d, 1e-6))
    sizes = np.diff(starts)
    var = float(np.mean(yc * yc))
    sig = math.sqrt(var)
    w = [math.log10(n), math.log10(max(th.max() - th.min(), 1e-3)), float(len(sizes)),
         float((sizes >= least).sum()), math.log10(max(d.mean(), 1e-6)) if len(d) else 0.0,
         float(ld.std()) if len(d) else 0.0, float(sizes[sizes >= least].sum()) / n,
         math.log10(sig), float(np.mean(yc ** 3)) / (var * sig),
         float(np.mean(yc ** 4)) / (var * var) - 3.0, float(np.abs(yc).max()) / sig]
    step = (math.log10(30.0) + 3.0) / 52
    fp = torch.as_tensor([10.0 ** (-3.0 + q * step) for q in range(53)], dtype=torch.float64,
                         device=DEV)
    ph = 2 * math.pi * _phase(fp, t)
    win = (torch.cos(ph).sum(1) ** 2 + torch.sin(ph).sum(1) ** 2) / (n * n)
    return torch.cat([torch.as_tensor(w, dtype=torch.float64, device=DEV), win])


def _net_exact(case, seed):
    x, labels = _net_inputs(case, seed)
    x = (x.to(torch.int32) << 16).view(torch.float32).double()
    par = [torch.as_tensor(np.asarray(p, np.float32), device=DEV).double()
           for p in learned.banded_init(7)]
    w = [p.float().to(torch.bfloat16).double() for p in par[0::2]]
    h1 = torch.relu(x @ w[0] + par[1])
    h2 = torch.relu(h1 @ w[1] + par[3])
    z = h2 @ w[2] + par[5]
    if case["kind"] == "forward":
        return z
    n = x.shape[0]
    lab = labels.long()
    logp = torch.log_softmax(z, dim=1)
    loss = -logp.gather(1, lab[:, None])[:, 0]
    g3 = torch.exp(logp)
    g3[torch.arange(n, device=DEV), lab] -= 1.0
    g3 = g3 / n
    g2 = (g3 @ w[2].T) * (h2 > 0)
    g1 = (g2 @ w[1].T) * (h1 > 0)
    grads = [x.T @ g1, g1.sum(0), h1.T @ g2, g2.sum(0), h2.T @ g3, g3.sum(0)]
    new = []
    for p, g in zip(par, grads):
        m = 1.0e-4 * torch.sin(torch.arange(p.numel(), device=DEV)).double().view(p.shape)
        m = 0.9 * m + 0.1 * g
        v = 0.999 * 1.0e-4 + 0.001 * g * g
        new.append(p - 1e-3 * (m / (1 - 0.9 ** 51)) / (torch.sqrt(v / (1 - 0.999 ** 51)) + 1e-8))
    return {"loss": loss, "grads": grads, "weights": new}


def exact(case, seed):
    """What run() returns for the first pass on these inputs, in 64 bits by
    plain torch; None for fields that are whole numbers or follow from them."""
    kind = case["kind"]
    if kind in ("forward", "train"):
        return _net_exact(case, seed)
    off, t, y, dy, (f_min, f_max), unit = _inputs(case, seed)
    ends = off.cpu().numpy()
    if kind == "features":
        if ends[-1] > 600_000:
            return None
        rows = []
        for a, b in zip(ends[:-1], ends[1:]):
            coarse, starts = _coarse(t[a:b], y[a:b] - y[a:b].mean(), 60.0, 8)
            rows.append(torch.cat([coarse, _window(t[a:b], y[a:b], 60.0, 8, starts)]))
        return torch.stack(rows)
    n_f = case["n_f"]
    none = {"index": None, "freq": None, "period": None, "status": None}
    f, f_cyc = _grid(f_min, f_max, n_f, unit)
    if kind == "rows":
        bb = -(-n_f // 64)
        bands = _bands(case, seed)
        best = []
        for o, (a, b) in enumerate(zip(ends[:-1], ends[1:])):
            at = np.concatenate([np.arange(k * bb, min((k + 1) * bb, n_f))
                                 for k in bands[o] if k >= 0])
            at = torch.as_tensor(at, device=DEV)
            best.append(_object_powers(case, t[a:b], y[a:b], None, f_cyc[at]).max())
        return dict(none, power=torch.stack(best))
    if float(ends[-1]) * n_f > 2.0e11:
        return None
    p = [_object_powers(case, t[a:b], y[a:b], None if dy is None else dy[a:b], f_cyc)
         for a, b in zip(ends[:-1], ends[1:])]
    if kind == "single":
        return dict(none, pgram=p[0][None])
    if case["pgram"]:
        return {"pgram": torch.stack(p)}
    return dict(none, power=torch.stack([q.max() for q in p]))
