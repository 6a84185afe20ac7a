"""Up to capacity 64 a chain is the same bits whichever kernels hold it (needs an MI355X): state,
records, charge draws and the log of every step, for the single charge law, the mixture law and from
start lists; the LDS chains of all capacities in one launch, in one each, and the narrow
device-memory groups."""
import numpy as np
import pytest

from paper_2403_03156_amd import fsmp, synth
from tests.fsmp_cases import to_host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
MIX = ([0.041, 0.516, 0.187, 0.195, 0.061], [0.92, 1.98, 3.01, 4.70, 6.79], [0.22, 0.48, 0.80, 1.30, 2.04])


@pytest.mark.parametrize("preset,form", [("batched", "plain"), ("batched", "mix"), ("batched", "start"),
                                         ("plain", "plain"), ("pileup", "start"), ("pileup", "mix")])
def test_every_kernel_gives_the_same_bits(preset, form):
    wl = synth.PRESETS[preset]
    lam = np.concatenate([np.linspace(0.2, 22.0, 60), [8.0, 14.0, 21.5]])
    b = synth.generate(wl, n_wave=len(lam), seed=12, lam=lam)
    km = synth.kmax_for(lam)
    km[-3:] = (9, 15, 22)  # lists at K_max
    assert set(km.tolist()) == {9, 15, 16, 22, 32, 48, 64}
    wave = torch.from_numpy(b["wave"]).cuda()
    kw = {}
    if form == "start":
        t0 = float(np.floor(wl.t0_min)) + 1.0
        lo, hi = int(4 * t0) + 1, 4 * int(np.diff(b["offsets"])[0]) - 1
        z = [np.unique(np.clip(np.rint(np.asarray(t) * 4), lo, hi).astype(int))[:k].tolist()
             for t, k in zip(b["times"], km)]
        kw = dict(z_init=[x for x in z for _ in range(2)], t0_init=np.full(len(km), t0))
    print(f"[case] same bits {preset} {form}", flush=True)
    out = []
    for design, timed in ((None, False), (fsmp.FSMP_DESIGN_GROUP_LDS, True), (fsmp.FSMP_DESIGN_GROUP_DEVMEM, False)):
        s = fsmp.Sampler(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay,
                         t0_min=wl.t0_min, t0_max=wl.t0_max, sigma_eps=wl.sigma_eps, mu_q=wl.mu_q,
                         sigma_q=wl.sigma_q, n_steps=400, n_chains=2, burn_in=100, seed=21, thin=50, k_max=64,
                         record_flags=fsmp.FSMP_REC_TRACE | fsmp.FSMP_REC_LOG | fsmp.FSMP_REC_CHARGE,
                         **({"mix": MIX} if form == "mix" else {}))
        s.set_timing(timed)  # (timed: a launch per capacity)
        if design is not None:
            s.set_design(0, design)
        out.append(to_host(s.sample(wave, b["offsets"], lam, kmax=km, kz=64, **kw)))
    for o in out:
        lg = o.pop("log").view(fsmp.LOGREC_DTYPE)
        o.update({"log " + f: lg[f] for f in ("move", "flags", "j", "g", "t0", "dnu", "log_alpha")})
    for k, v in out[0].items():
        if isinstance(v, np.ndarray):
            np.testing.assert_array_equal(out[1][k], v, err_msg=k)
            np.testing.assert_array_equal(out[2][k], v, err_msg=k)


@pytest.mark.parametrize("preset", ["batched", "plain"])
def test_mixed_precision_does_not_depend_on_the_number_of_chains(preset):
    # capacity 16 in 16-lane groups alone, in 4-lane groups among 9,000 chains, in the launch of
    # capacity 32; with rebuilds from the bounds and every 64 sweeps, and from start lists
    wl = synth.PRESETS[preset]
    n, r = 100, 90
    lam = np.linspace(0.1, 3.2, n)
    b = synth.generate(wl, n_wave=n, seed=2, lam=lam)
    km = np.full(n, 16, np.int32)
    km[:3] = (1, 5, 9)
    t0 = float(np.floor(wl.t0_min)) + 1.0
    L = int(np.diff(b["offsets"])[0])
    z = [np.unique(np.clip(np.rint(np.asarray(t) * 4), int(4 * t0) + 1, 4 * L - 1).astype(int))[:k].tolist()
         if i % 2 else [] for i, (t, k) in enumerate(zip(b["times"], km))]
    s = fsmp.Sampler(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay,
                     t0_min=wl.t0_min, t0_max=wl.t0_max, sigma_eps=wl.sigma_eps, mu_q=wl.mu_q, sigma_q=wl.sigma_q,
                     n_steps=200, burn_in=60, seed=3, thin=20, k_max=32,
                     record_flags=fsmp.FSMP_REC_TRACE | fsmp.FSMP_REC_LOG | fsmp.FSMP_REC_CHARGE,
                     precision=fsmp.FSMP_FP32_REFRESH, refresh_M=64)

    def run(rep, k, wide32=False):
        # wide32: a waveform of capacity 32 besides, so that both share a launch
        kk = np.tile(k, rep)
        wid = np.tile(np.arange(n, dtype=np.uint64), rep)
        if wide32:
            kk[0] = 32
        off = np.concatenate([[0], np.cumsum(np.full(n * rep, L, np.int64))])
        s.set_timing(True)
        out = s.sample(torch.from_numpy(np.tile(b["wave"], rep)).cuda(), off, np.tile(lam, rep), kmax=kk, kz=32,
                       wave_id=wid, z_init=z * rep, t0_init=np.full(n * rep, t0))
        lanes = {(t["kcap"], t["lanes"]) for t in s.last_timings() if t["kcap"] > 0}
        o = to_host(out)
        lg = o.pop("log").view(fsmp.LOGREC_DTYPE)
        o.update({"log " + f: lg[f] for f in ("move", "flags", "j", "g", "t0", "dnu", "log_alpha")})
        return lanes, {q: v[-n + 1:] for q, v in o.items() if isinstance(v, np.ndarray)}  # (the first one apart)

    print(f"[case] mixed precision few and many, {preset}", flush=True)
    few, many, joined = run(1, km), run(r, km), run(1, km, wide32=True)
    assert few[0] == {(16, 16)} and many[0] == {(16, 4)} and joined[0] == {(32, 16)}
    assert few[1]["n_pe"].max() > 3
    for k, v in few[1].items():
        np.testing.assert_array_equal(many[1][k], v, err_msg=k)
        np.testing.assert_array_equal(joined[1][k], v, err_msg=k)
