"""What the time of this framework is measured on: the calls its users make, over the sizes they
make them at.

Every case is one pass through the public binding (`fsmp.Sampler`, `fsmp.Server`): sampling the
photo-electron sequences of a batch of PMT waveforms and reducing the chains to posteriors, serving
one trigger event from host memory, or deconvolving a batch for its start states.  The workloads are
the shapes of `synth.PRESETS` (window lengths, light curves, charge laws, intensities), cut to a
number of waveforms that a few passes fit in seconds.
"""
import math

import numpy as np
import torch

from paper_2403_03156_amd import fsmp, synth

# the five-component charge law of MCP-PMTs, in units of the single-electron amplitude
MIX = ((0.041, 0.516, 0.187, 0.195, 0.061), (0.92, 1.98, 3.01, 4.70, 6.79), (0.22, 0.48, 0.80, 1.30, 2.04))
EVENT_ID = 7


def _case(name, kind, preset, n_wave, length_lo, length_hi, lam_lo, lam_hi, n_steps, n_chains=1, form="fp64",
          adaptive=False, wide=False, summary=False, records=False):
    """kind: sample | event | lucy.  length_lo == length_hi: every window that long; otherwise each
    waveform's own length between them.  adaptive: every waveform's sweeps from the chain-length
    tuner, n_steps at most.  wide: the wide kernel groups at the capacities where the design tuner
    keeps them for windows of unequal sweeps.  summary: convergence diagnostics and the intensity
    estimates beside the means.  records: start lists, traces, charge draws and grid occupancy."""
    return {"name": name, "kind": kind, "preset": preset, "n_wave": n_wave, "length_lo": length_lo,
            "length_hi": length_hi, "lam_lo": lam_lo, "lam_hi": lam_hi, "n_steps": n_steps, "n_chains": n_chains,
            "form": form, "adaptive": adaptive, "wide": wide, "summary": summary, "records": records}


def listed():
    return [
        # one trigger on a handful of channels, sampled as it comes in: nothing but the latency of a sweep
        _case("few_channels", "sample", "plain", 16, 256, 256, 0.5, 5.0, 500),
        # the smallest standard workload: 1,000 short windows, exponential light curve
        _case("plain", "sample", "plain", 1000, 256, 256, 0.5, 5.0, 2000),
        # one event of a running detector through the serving loop, host memory in and out
        _case("event", "event", "serving", 1200, 1024, 1024, 0.0, 20.0, 1000),
        # offline batch, four chains a waveform for the convergence checks and the intensity estimates
        _case("batched_chains", "sample", "batched", 8000, 1024, 1024, 0.1, 30.0, 600, n_chains=4, summary=True),
        # offline batch of ragged windows with chain lengths from the tuner: the headline workload's shape
        _case("uneven", "sample", "uneven", 16000, 128, 2048, 0.05, 100.0, 4000, adaptive=True, wide=True),
        # the same windows at equal chain lengths and default settings, odd lengths
        _case("ragged", "sample", "uneven", 20000, 101, 1531, 0.05, 60.0, 500),
        # bright events, tens of photo-electrons in every window
        _case("pileup", "sample", "pileup", 3000, 1024, 1024, 20.0, 100.0, 500),
        # the mixed-precision form on moderately bright windows
        _case("fp32_refresh", "sample", "batched", 4000, 1024, 1024, 0.1, 60.0, 400, form="fp32"),
        # MCP-PMT charge law
        _case("mixture", "sample", "batched", 8000, 1024, 1024, 0.1, 30.0, 600, form="mix"),
        # start states by deconvolution, ragged windows
        _case("deconvolution", "lucy", "uneven", 3000, 128, 2048, 0.05, 100.0, 500),
        # a study of single waveforms: chains from the deconvolution's lists, with traces, charge draws and
        # the occupancy of the grid
        _case("study", "sample", "batched", 300, 1024, 1024, 0.5, 30.0, 600, n_chains=4, summary=True, records=True),
    ]


def _log_between(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    what = rng.choice(["plain", "event", "batched", "uneven", "ragged", "pileup", "fp32", "mix", "lucy", "study"])
    if what == "plain":
        length = rng.randint(128, 511)
        return _strip(_case("", "sample", "plain", int(_log_between(rng, 1, 2000)), length, length, 0.5,
                            rng.uniform(2.0, 8.0), int(_log_between(rng, 200, 2000))))
    if what == "event":
        length = rng.randint(500, 1024)
        return _strip(_case("", "event", "serving", rng.randint(50, 2000), length, length, 0.0,
                            rng.uniform(10.0, 20.0), int(_log_between(rng, 300, 1000))))
    if what == "batched":
        length = rng.randint(257, 1024)
        return _strip(_case("", "sample", "batched", int(_log_between(rng, 100, 8000)), length, length, 0.1,
                            rng.uniform(10.0, 30.0), int(_log_between(rng, 200, 600)), n_chains=rng.randint(2, 4),
                            summary=True))
    if what == "uneven":
        return _strip(_case("", "sample", "uneven", int(_log_between(rng, 1000, 14000)), rng.randint(100, 200),
                            rng.randint(800, 2048), 0.05, rng.uniform(30.0, 100.0), rng.randint(1000, 4000),
                            adaptive=True, wide=True))
    if what == "ragged":
        return _strip(_case("", "sample", "uneven", int(_log_between(rng, 300, 18000)), rng.randint(70, 200),
                            rng.randint(400, 1531), 0.05, rng.uniform(5.0, 60.0), rng.randint(200, 500)))
    if what == "pileup":
        length = rng.randint(400, 1024)
        return _strip(_case("", "sample", "pileup", int(_log_between(rng, 50, 3000)), length, length, 20.0,
                            rng.uniform(40.0, 100.0), rng.randint(200, 500)))
    if what == "fp32":
        length = rng.randint(257, 1024)
        return _strip(_case("", "sample", "batched", int(_log_between(rng, 100, 4000)), length, length, 0.1,
                            rng.uniform(10.0, 60.0), rng.randint(150, 400), form="fp32"))
    if what == "mix":
        length = rng.randint(257, 1024)
        return _strip(_case("", "sample", "batched", int(_log_between(rng, 100, 8000)), length, length, 0.1,
                            rng.uniform(5.0, 30.0), rng.randint(200, 600), form="mix"))
    if what == "lucy":
        return _strip(_case("", "lucy", "uneven", int(_log_between(rng, 10, 3000)), rng.randint(70, 200),
                            rng.randint(400, 2048), 0.05, rng.uniform(10.0, 100.0), rng.randint(50, 500)))
    length = rng.randint(400, 1024)
    return _strip(_case("", "sample", "batched", rng.randint(10, 300), length, length, 0.5, rng.uniform(5.0, 30.0),
                        rng.randint(200, 600), n_chains=rng.randint(2, 4), summary=True, records=True))


def _strip(case):
    del case["name"]
    return case


# ------------------------------------------------------------------ inputs
def _inputs(case, seed):
    """Waveforms of the preset's forward model on the host: N ~ Poisson(lambda), times from the
    light curve after t0, charges from the charge law, the response and white noise."""
    wl = synth.PRESETS[case["preset"]]
    rng = np.random.default_rng([seed, case["n_wave"]])
    n = case["n_wave"]
    lo, hi = case["lam_lo"], case["lam_hi"]
    if wl.lam_dist == "loguniform":
        lam = np.exp(rng.uniform(math.log(lo), math.log(hi), n))
    elif wl.lam_dist == "mixture":  # channels of an event: mostly dark, some lit
        lam = np.where(rng.uniform(size=n) < 0.7, rng.uniform(0.0, 1.0, n), rng.uniform(1.0, hi, n))
    else:
        lam = rng.uniform(lo, hi, n)
    fixed = np.random.default_rng(n)  # the windows' lengths belong to the case, not to its inputs
    if case["length_lo"] == case["length_hi"]:
        lengths = np.full(n, case["length_lo"], np.int64)
    elif case["adaptive"] or case["kind"] == "lucy":  # windows of a few standard lengths
        lengths = np.array([case["length_lo"] << k for k in range(12) if case["length_lo"] << k <= case["length_hi"]])
        lengths = lengths[fixed.integers(0, len(lengths), n)]
    else:
        lengths = fixed.integers(case["length_lo"], case["length_hi"] + 1, n)
    offsets = np.zeros(n + 1, np.int64)
    offsets[1:] = np.cumsum(lengths)
    owner = np.repeat(np.arange(n), rng.poisson(lam))
    tot = len(owner)
    times = rng.uniform(wl.t0_min, wl.t0_max, n)[owner] + rng.exponential(wl.tau_decay, tot)
    if wl.phi_kind == synth.PHI_BIEXP:
        times += rng.exponential(wl.tau_rise * wl.tau_decay / (wl.tau_rise + wl.tau_decay), tot)
    if case["form"] == "mix":
        e = rng.choice(len(MIX[0]), size=tot, p=MIX[0])
        charge = np.abs(rng.normal(np.array(MIX[1])[e], np.array(MIX[2])[e]))
    elif wl.charge == "gamma":
        charge = rng.gamma((wl.mu_q / wl.sigma_q) ** 2, wl.sigma_q ** 2 / wl.mu_q, tot)
    else:
        charge = np.abs(rng.normal(wl.mu_q, wl.sigma_q, tot))
    # the response at 1/32 of a sample
    fine, span = 32, 128
    dist, peak = synth.ser_peak(*wl.ser)
    table = dist.pdf(np.arange(fine * (span + 1)) / fine) / peak
    at = np.rint(times * fine).astype(np.int64)
    first = -(-at // fine)  # the first sample at or after the photo-electron
    phase = first * fine - at
    acc = np.zeros(int(offsets[-1]))
    rel = np.arange(span)
    for a in range(0, tot, 100_000):
        s = slice(a, a + 100_000)
        idx = first[s, None] + rel
        ok = idx < lengths[owner[s], None]
        base, top = int(offsets[owner[s][0]]), int(offsets[owner[s][-1] + 1])
        val = charge[s, None] * table[phase[s, None] + rel * fine]
        acc[base:top] += np.bincount((offsets[owner[s], None] + idx)[ok] - base, weights=val[ok],
                                     minlength=top - base)
    wave = (acc + wl.sigma_eps * rng.standard_normal(len(acc))).astype(np.float32)
    return wl, wave, offsets, lam, synth.kmax_for(lam)


def _row(case):
    """The row length of the PE lists: the cap of the brightest waveform of the case's range."""
    return int(synth.kmax_for(np.array([case["lam_hi"]]))[0])


def _settings(case, wl, seed):
    n_steps = case["n_steps"]
    return dict(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay, t0_min=wl.t0_min,
                t0_max=wl.t0_max, sigma_eps=wl.sigma_eps, mu_q=wl.mu_q, sigma_q=wl.sigma_q, n_steps=n_steps,
                n_chains=case["n_chains"], burn_in=n_steps // 2, seed=seed,
                precision=fsmp.FSMP_FP32_REFRESH if case["form"] == "fp32" else fsmp.FSMP_FP64)


def prepare(case, seed):
    wl, wave, offsets, lam, kmax = _inputs(case, seed)
    kw = _settings(case, wl, seed)
    if case["kind"] == "event":
        return {"case": case, "server": fsmp.Server(kw), "wave": wave, "offsets": offsets, "lam": lam, "kmax": kmax}
    if case["records"]:
        kw.update(record_flags=fsmp.FSMP_REC_TRACE | fsmp.FSMP_REC_CHARGE, thin=25)
    if case["form"] == "mix":
        kw.update(mix=MIX)
    if case["form"] == "fp32":
        kw.update(refresh_M=64)
    state = {"case": case, "sampler": fsmp.Sampler(k_max=_row(case), **kw), "wave": torch.from_numpy(wave).cuda(),
             "offsets": offsets, "lam": lam, "kmax": kmax, "n_steps": None, "start": {}}
    smp = state["sampler"]
    if case["kind"] == "lucy":
        return state
    if case["wide"]:
        for cap in (32, 48, 96, 128, 160, 192):
            smp.set_design(cap, fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE)
    if case["adaptive"]:
        state["n_steps"] = smp.autotune_steps(state["wave"], offsets, lam, kmax=kmax, pilot_steps=100,
                                              min_steps=min(500, case["n_steps"]), max_steps=case["n_steps"])
    if case["records"]:
        z, g_range, t0 = smp.start_from(smp.lucy(state["wave"], offsets, kmax=kmax, n_iter=200), case["n_chains"])
        state["start"] = {"z_init": z, "g_range": g_range, "t0_init": t0, "occupancy": True}
    occ = smp.cfg.grid_sub * int(offsets[-1]) if case["records"] else 0
    state["out"] = smp.alloc_samples(case["n_wave"], _row(case), occ_len=occ)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "event":
        srv = state["server"]
        srv.submit(EVENT_ID, state["wave"], state["offsets"], state["lam"], state["kmax"])
        while True:
            srv.progress(wait=True)
            res = srv.result(EVENT_ID)
            if res is not None:
                del res["latency"]
                return res
    smp = state["sampler"]
    if case["kind"] == "lucy":
        res = smp.lucy(state["wave"], state["offsets"], kmax=state["kmax"], kz=_row(case), n_iter=case["n_steps"],
                       qhat=True)
        del res["kz"]
        return res
    out = smp.sample(state["wave"], state["offsets"], state["lam"], kmax=state["kmax"], n_steps=state["n_steps"],
                     out=state["out"], kz=_row(case), **state["start"])
    more = {"diagnostics": True, "lam": state["lam"]} if case["summary"] else {}
    if case["records"]:
        more["offsets"] = state["offsets"]
    post = smp.posterior(case["n_wave"], out, **more)
    return {"chains": {k: v for k, v in out.items() if k != "kz" and v is not None},
            "posterior": {k: v for k, v in post.items() if v is not None}}


# ------------------------------------------------------------------ work
def work(case):
    """Bytes: the samples in, the chains' and waveforms' results out.  Flops of the chains: per
    sweep the products of a proposal with the K x K inverse (three of four moves need one) and
    about 200 for the light curve's integral, the random values and the logs; per waveform the
    matched filter.  Flops of the deconvolution: the two sums of each iteration."""
    wl = synth.PRESETS[case["preset"]]
    n, C = case["n_wave"], case["n_chains"]
    lo, hi = case["lam_lo"], case["lam_hi"]
    if wl.lam_dist == "loguniform":
        m1 = (hi - lo) / math.log(hi / lo)
        m2 = (hi * hi - lo * lo) / (2.0 * math.log(hi / lo))
    elif wl.lam_dist == "mixture":
        m1 = 0.7 * 0.5 + 0.3 * 0.5 * (1.0 + hi)
        m2 = 0.7 / 3.0 + 0.3 * (hi * hi + hi + 1.0) / 3.0
    else:
        m1, m2 = 0.5 * (lo + hi), (hi * hi + hi * lo + lo * lo) / 3.0
    support = 64 if case["preset"] == "serving" else 96
    length = 0.5 * (case["length_lo"] + case["length_hi"])
    if case["length_lo"] != case["length_hi"] and (case["adaptive"] or case["kind"] == "lucy"):
        lens = [case["length_lo"] << k for k in range(12) if case["length_lo"] << k <= case["length_hi"]]
        length = sum(lens) / len(lens)
    if case["kind"] == "lucy":
        flops = 2.0 * n * case["n_steps"] * support * (2.0 * length + support)
        return {"bytes": n * (4.0 * length + 8.0 * (length + support) + 4.0 * m1 + 40.0), "flops": flops}
    sweeps = 0.25 * case["n_steps"] if case["adaptive"] else case["n_steps"]
    flops = n * C * sweeps * (1.5 * (m2 + m1) + 200.0) + n * 8.0 * length * support
    rows = 16.0 * m1 + 200.0
    if case["records"]:
        rows += (case["n_steps"] // 50) * (12.0 * m1 + 24.0)
    return {"bytes": n * (4.0 * length + C * rows + 150.0), "flops": flops}


# ------------------------------------------------------------------ values in 64 bits
def _ser_table(ser, sub):
    """V(m / sub), the ex-Gaussian over its maximum, cut where it stays below 1e-6, and its support in samples."""
    mu, sigma, tau = ser

    def pdf(t):
        x = torch.as_tensor(np.asarray(t, np.float64))
        a = (mu + sigma * sigma / tau - x) / (sigma * math.sqrt(2.0))
        # exp(-(t - mu)^2 / 2 sigma^2) erfcx(a) / 2 tau where erfcx does not overflow, the plain form elsewhere
        y = torch.where(a > 0, torch.exp(-0.5 * ((x - mu) / sigma) ** 2) * torch.special.erfcx(a.clamp(min=0)),
                        torch.exp(sigma * sigma / (2 * tau * tau) - (x - mu) / tau) * torch.special.erfc(a.clamp(max=0)))
        return (y / (2 * tau)).numpy()

    lo, hi = 0.0, mu + 5 * tau
    for _ in range(40):
        t = np.linspace(lo, hi, 101)
        k = int(np.argmax(pdf(t)))
        lo, hi = t[max(k - 1, 0)], t[min(k + 1, 100)]
    peak = float(pdf([0.5 * (lo + hi)])[0])
    support = 16
    while support < 512 and pdf(np.arange(support * sub, 4096.0) / sub).max() / peak >= 1e-6:
        support += 16
    return pdf(np.arange(support * sub) / sub) / peak, support


def _exact_lucy(case, seed):
    wl, wave, offsets, lam, kmax = _inputs(case, seed)
    sub, threshold, margin = 4, 0.1, 4
    table, LV = _ser_table(wl.ser, sub)
    V = table[::sub]
    n, kz = len(lam), _row(case)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    res = {"z": np.full((n, kz), -1, np.int32), "n_pe": np.zeros(n, np.int32), "g_range": np.zeros((n, 2), np.int32),
           "t0": np.zeros(n), "lambda": np.zeros(n), "cut": np.zeros((n, 2), np.int32),
           "qhat": np.zeros(int(offsets[-1]) + n * (LV - 1))}
    lengths = np.diff(offsets)
    for L in np.unique(lengths):
        L, idx = int(L), np.nonzero(lengths == L)[0]
        T = np.zeros((L + LV - 1, L))  # sample t takes V(t - tau) of every tau = i - (LV - 1)
        for s in range(LV):
            T[np.arange(L) + LV - 1 - s, np.arange(L)] = V[s] / V.sum()
        T = torch.from_numpy(T).to(dev)
        Tt = T.t().contiguous()
        d = np.stack([wave[offsets[i]:offsets[i + 1]] for i in idx]).astype(np.float64).clip(min=0.0)
        d = torch.from_numpy(d).to(dev)
        u = (d.sum(1, keepdim=True) / (L + LV - 1)).expand(-1, L + LV - 1).clone()
        for _ in range(case["n_steps"]):
            wr = u @ T
            u = u * (torch.where(wr > 0, d / wr, torch.zeros_like(wr)) @ Tt)
        q = (u / V.sum()).cpu().numpy()
        for row, i in enumerate(idx):
            qi = q[row]
            res["qhat"][offsets[i] + i * (LV - 1):offsets[i + 1] + (i + 1) * (LV - 1)] = qi
            res["lambda"][i] = qi.sum()
            tau = np.nonzero(qi[LV - 1:] > threshold)[0]
            if len(tau) > kmax[i]:
                tau = np.sort(tau[np.lexsort((tau, -qi[LV - 1 + tau]))[:kmax[i]]])
            if len(tau) == 0:
                res["t0"][i], res["g_range"][i], res["cut"][i] = 0.5 * (wl.t0_min + wl.t0_max), (1, 0), (0, L - 1)
                continue
            t0 = min(max(tau[0] - 0.5 / sub, wl.t0_min), wl.t0_max)
            z = sub * tau[tau - t0 > 0]
            res["t0"][i], res["n_pe"][i], res["z"][i, :len(z)] = t0, len(z), z
            res["g_range"][i] = max(0, sub * (tau[0] - margin)), min(sub * L - 1, sub * (tau[-1] + margin))
            res["cut"][i] = max(0, tau[0] - margin), min(L - 1, tau[-1] + margin + LV)
    return res


def _philox(step, block, uid, key):
    """Philox4x32-10 of the counters (step, block, uid lo, uid hi), one row per uid."""
    m32 = np.uint64(0xFFFFFFFF)
    c = [np.full(uid.shape, step, np.uint64), np.full(uid.shape, block, np.uint64), uid & m32, uid >> np.uint64(32)]
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m32, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1),
             p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _exact_chains(case, seed):
    """Every chain in plain numpy, all chains a sweep at a time, the marginal law of every
    proposal from scratch (Cholesky-free: solve and log-determinant of the padded Gram matrix)."""
    wl, wave, offsets, lam_w, kmax_w = _inputs(case, seed)
    sub, J, sd = 4, 0.25, 1.0
    dt, n, C, S = 1.0 / sub, case["n_wave"], case["n_chains"], case["n_steps"]
    burn, NC, K = S // 2, case["n_wave"] * case["n_chains"], _row(case)
    table, LV = _ser_table(wl.ser, sub)
    M = sub * LV
    own = np.repeat(np.arange(n), C)
    uid = np.arange(NC, dtype=np.uint64)
    L, lam, kmax = np.diff(offsets)[own], lam_w[own], kmax_w[own]
    ghi = sub * L - 1
    # matched filter and overlaps; the overlap of columns lo, lo + d over the first m samples that both see
    mf = np.zeros((n, sub * int(L.max())))
    for i in range(n):
        w = wave[offsets[i]:offsets[i + 1]].astype(np.float64)
        wp = np.concatenate([w, np.zeros(LV + 1)])
        for p in range(sub):  # g = sub q + p reads samples from q (p = 0) or q + 1
            V = table[(-p) % sub::sub]
            win = np.lib.stride_tricks.sliding_window_view(wp[1 if p else 0:], len(V))[:len(w)]
            mf[i, p:sub * len(w):sub] = win @ V
    ov = np.zeros((sub, M + 1, LV + 2))
    for p in range(sub):
        for d in range(M):
            n0 = -(-(p + d) // sub)
            s = np.arange(n0, (p + M - 1) // sub + 1)
            ov[p, d, 1:len(s) + 1] = np.cumsum(table[sub * s - p] * table[sub * s - p - d])
            ov[p, d, len(s) + 1:] = ov[p, d, len(s)]

    def overlap(a, b):
        lo, hi = np.minimum(a, b), np.maximum(a, b)
        seen = np.clip(L.reshape((-1,) + (1,) * (a.ndim - 1)) + (-hi // sub), 0, LV + 1)
        return ov[lo % sub, np.minimum(hi - lo, M), seen]

    s2 = wl.sigma_eps ** 2
    rho = s2 / wl.sigma_q ** 2
    biexp = wl.phi_kind == synth.PHI_BIEXP
    t1, t2 = wl.tau_rise, wl.tau_decay
    t12 = t1 * t2 / (t1 + t2) if biexp else 1.0
    amp = (t1 + t2) / t2 ** 2 if biexp else 1.0 / t2

    def log_phi(x):
        with np.errstate(divide="ignore", invalid="ignore"):
            r = math.log(amp) - x / t2
            if biexp:
                r = r + np.log(-np.expm1(-x / t1))
            return np.where((x > 0) | ((x == 0) & (not biexp)), r, -np.inf)

    def start(t0):
        return np.maximum(np.ceil(t0 / dt), 0.0)

    def partial(t0, k):  # the light curve summed over the first k grid points at or after t0
        x = start(t0) * dt - t0
        s = np.exp(-x / t2) * np.expm1(-k * dt / t2) / math.expm1(-dt / t2)
        if biexp:
            s = s - np.exp(-x / t12) * np.expm1(-k * dt / t12) / math.expm1(-dt / t12)
        return amp * s

    def total(t0):
        return partial(t0, np.maximum(ghi + 1 - start(t0), 0))

    slot = np.arange(K)
    rows = np.arange(NC)

    def law(z, N, chains):
        """log p(w | z) up to a constant and the charge means, for the rows `chains`."""
        nonlocal L
        keep, L = L, L[chains]
        on = slot < N[:, None]
        zz = np.where(on, z, 0)
        G = overlap(zz[:, :, None], zz[:, None, :]) * (on[:, :, None] & on[:, None, :])
        L = keep
        G[:, slot, slot] += np.where(on, rho, 1.0)
        b = np.where(on, mf[own[chains, None], zz] + rho * wl.mu_q, 0.0)
        x = np.linalg.solve(G, b[:, :, None])[:, :, 0]
        logdet = np.linalg.slogdet(G)[1]
        nu = -0.5 * (-N * math.log(rho) + logdet + (N * rho * wl.mu_q ** 2 - (b * x).sum(1)) / s2)
        return nu, x

    z, N, t0 = np.zeros((NC, K), np.int64), np.zeros(NC, np.int64), np.full(NC, 0.5 * (wl.t0_min + wl.t0_max))
    nu, x = law(z, N, rows)
    acc, batch = np.zeros((NC, 12)), np.zeros((NC, 3))
    nhist, counts, status = np.zeros((NC, K + 1), np.int32), np.zeros((NC, 8), np.int32), np.zeros(NC, np.int32)
    n_rec = S - burn
    nb = int(math.sqrt(n_rec))
    lb = n_rec // nb

    def u01(r):
        return (r.astype(np.float64) + 0.5) * 2.0 ** -32

    for step in range(S):
        r = _philox(step, 0, uid, seed) + _philox(step, 1, uid, seed)
        rad, th = np.sqrt(-2.0 * np.log(u01(r[0]))), 2.0 * math.pi * u01(r[1])
        on = slot < N[:, None]
        # t0
        t0p = t0 + sd * rad * np.cos(th)
        counts[:, 0] += 1
        with np.errstate(invalid="ignore"):
            la = np.where(on, log_phi(z * dt - t0p[:, None]) - log_phi(z * dt - t0[:, None]), 0.0).sum(1)
            la -= lam * dt * (total(t0p) - total(t0))
            ok = (t0p >= wl.t0_min) & (t0p <= wl.t0_max) & (np.log(u01(r[2])) < la)
        t0 = np.where(ok, t0p, t0)
        counts[:, 1] += ok
        # one jump
        phi = total(t0)
        Lam = lam * dt * phi
        um = u01(r[3])
        move = np.where((N == 0) | (um < J), 1, np.where(um < 2 * J, 2, 3))
        counts[rows, 2 * move] += 1
        full = (move == 1) & (N >= kmax)
        status |= full.astype(np.int32)
        v = (r[5] << np.uint64(32)) | r[4]
        target = ((v >> np.uint64(11)).astype(np.float64) * 2.0 ** -53 + 2.0 ** -54) * phi
        lo, hi = np.zeros(NC), np.maximum(ghi - start(t0), 0.0)
        while (lo < hi).any():
            mid = np.floor(0.5 * (lo + hi))
            above = partial(t0, mid + 1) > target
            lo, hi = np.where(above | (lo >= hi), lo, mid + 1), np.where(above, mid, hi)
        j = ((r[4] * N.astype(np.uint64)) >> np.uint64(32)).astype(np.int64)
        zj = z[rows, j]
        shift = np.rint(rad * np.sin(th) * sd / dt).astype(np.int64)
        g = np.where(move == 1, (start(t0) + lo).astype(np.int64), zj + shift)
        with np.errstate(invalid="ignore"):
            lp = log_phi(g * dt - t0) - log_phi(zj * dt - t0)
        can = np.where(move == 1, ~full & (phi > 0) & (Lam > 0),
                       (move == 2) | ((g >= 0) & (g <= ghi) & (lp > -np.inf)))
        new, Nn = z.copy(), N + np.where(move == 1, 1, np.where(move == 2, -1, 0))
        put = np.where(move == 1, np.minimum(N, K - 1), j)
        new[rows, put] = np.where(move == 2, z[rows, np.maximum(N - 1, 0)], g)
        Nn = np.where(can, Nn, N)
        nu2, x2 = nu.copy(), x.copy()
        do = np.nonzero(can)[0]
        nu2[do], x2[do] = law(new[do], Nn[do], do)
        with np.errstate(divide="ignore", invalid="ignore"):
            la = np.where(move == 1, np.log(Lam) - np.log(N + 1.0) + np.where(N == 0, math.log(J), 0.0),
                          np.where(move == 2, np.log(np.maximum(N, 1)) - np.log(Lam) - np.where(N == 1, math.log(J), 0.0),
                                   lp))
            la = np.where((move == 3) & (shift == 0), lp, la + (nu2 - nu))
            ok = can & (np.log(u01(r[6])) < la)
        counts[rows, 2 * move + 1] += ok
        z, N = np.where(ok[:, None], new, z), np.where(ok, Nn, N)
        nu, x = np.where(ok, nu2, nu), np.where(ok[:, None], x2, x)
        if step >= burn:
            i = step - burn
            val = np.stack([N, np.where(slot < N[:, None], x, 0.0).sum(1), t0], 1)
            acc[:, 0:6:2] += val
            acc[:, 1:6:2] += val ** 2
            nhist[rows, N] += 1
            if i < nb * lb:
                batch += val
                if (i + 1) % lb == 0:
                    acc[:, 6::2] += batch
                    acc[:, 7::2] += batch ** 2
                    batch[:] = 0.0
    on = slot < N[:, None]
    a, h = acc.reshape(n, C, 12).sum(1), nhist.reshape(n, C, K + 1).sum(1)
    mean = a[:, 0:6:2] / (n_rec * C)
    bm = a[:, 6::2] / (nb * C * lb)
    bv = np.maximum((a[:, 7::2] / lb ** 2 - nb * C * bm ** 2) / (nb * C - 1), 0.0)
    cn = counts.reshape(n, C, 8).sum(1).astype(np.float64)
    post = {"mean": mean, "var": np.maximum(a[:, 1:6:2] / (n_rec * C) - mean ** 2, 0.0), "mcse": np.sqrt(bv / (nb * C)),
            "p_n": h / h.sum(1, keepdims=True),
            "accept": np.where(cn[:, ::2] > 0, cn[:, 1::2] / np.maximum(cn[:, ::2], 1), 0.0),
            "status": np.bitwise_or.reduce(status.reshape(n, C), 1)}
    chains = {"n_pe": N.astype(np.int32), "t0": t0, "z": np.where(on, z, -1).astype(np.int32),
              "charge": np.where(on, x, 0.0), "acc": acc, "nhist": nhist, "counts": counts, "status": status,
              "rec_steps": np.full(NC, n_rec, np.int32)}
    return {"chains": chains, "posterior": post}


def exact(case, seed):
    if case["kind"] == "lucy":
        return _exact_lucy(case, seed)
    if (case["kind"] == "sample" and case["form"] == "fp64" and not case["adaptive"] and not case["summary"]
            and case["lam_hi"] <= 8.0 and case["n_wave"] * case["n_steps"] <= 250_000):
        return _exact_chains(case, seed)
    return None
