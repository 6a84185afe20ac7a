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
