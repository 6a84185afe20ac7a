"""Which kernels a context runs (needs an MI355X): the design a capacity is set to, or left to the
library, names the kernels that its launches report."""
import numpy as np
import pytest

from paper_2403_03156_amd import fsmp, synth
from tests.fsmp_cases import gpu_sampler, to_host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
KEYS = ("n_pe", "t0", "z", "charge", "acc", "nhist", "counts", "status")


def _launches(smp, wave, b, km, **kw):
    """capacity -> (kernel name, lanes per chain) of one call"""
    smp.set_timing(True)
    smp.sample(wave, b["offsets"], b["lam"], kmax=km, **kw)
    t = {r["kcap"]: (r["name"], r["lanes"]) for r in smp.last_timings() if r["kcap"] > 0}
    smp.set_timing(False)
    return t


def test_automatic_is_a_design():
    wl = synth.PRESETS["batched"]
    b = synth.generate(wl, n_wave=24, seed=5, lam=np.linspace(0.5, 22.0, 24))
    km = synth.kmax_for(b["lam"])
    assert set(km.tolist()) == {16, 32, 48, 64}
    wave = torch.from_numpy(b["wave"]).cuda()
    print("[case] automatic design", flush=True)
    smp = gpu_sampler(wl, 60, 30, 1, 3)
    assert [smp.get_design(c) for c in synth.KCAPS] == [fsmp.FSMP_DESIGN_AUTO] * 8
    auto = _launches(smp, wave, b, km)
    ref = to_host(smp.sample(wave, b["offsets"], b["lam"], kmax=km))
    assert all(not name.startswith("chain_group_dm") for name, _ in auto.values())
    for cap, d in ((16, fsmp.FSMP_DESIGN_LANE), (0, fsmp.FSMP_DESIGN_GROUP_DEVMEM)):
        smp.set_design(cap, d)
    assert all(name.startswith("chain_group_dm") for name, _ in _launches(smp, wave, b, km).values())
    saved = {c: fsmp.FSMP_DESIGN_AUTO for c in synth.KCAPS}  # a saved plan of a fresh context
    for cap, d in saved.items():
        smp.set_design(cap, d)
    assert {c: smp.get_design(c) for c in synth.KCAPS} == saved
    assert _launches(smp, wave, b, km) == auto
    out = to_host(smp.sample(wave, b["offsets"], b["lam"], kmax=km))
    for k in KEYS:
        np.testing.assert_array_equal(out[k], ref[k], err_msg=k)


def test_automatic_where_there_is_no_choice():
    # the mixed-precision form has other kernels at capacities 16 and 32 only
    wl = synth.PRESETS["plain"]
    smp = fsmp.Sampler(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay,
                       t0_min=wl.t0_min, t0_max=wl.t0_max, n_steps=10, burn_in=5, seed=1,
                       precision=fsmp.FSMP_FP32_REFRESH)
    assert [smp.get_design(c) for c in synth.KCAPS] == [fsmp.FSMP_DESIGN_AUTO] * 2 + [fsmp.FSMP_DESIGN_GROUP_DEVMEM] * 6


# the five-Gaussian charge law of MCP-PMTs
MIX = ([0.041, 0.516, 0.187, 0.195, 0.061], [0.92, 1.98, 3.01, 4.70, 6.79], [0.22, 0.48, 0.80, 1.30, 2.04])


@pytest.mark.parametrize("form", ["mix", "fp32"])
def test_autotuner_tries_the_automatic_choice(form):
    # mixture law: the LDS chains are the library's choice only, no design a caller can name.  Mixed
    # precision: the launch that capacities 16 and 32 share exists where neither is set.  (Times
    # differ between runs: what a capacity may end with is checked, and that the kernels agree.)
    wl = synth.PRESETS["batched"]
    b = synth.generate(wl, n_wave=600, seed=9, lam=np.linspace(0.2, 8.0, 600))
    km = synth.kmax_for(b["lam"])
    assert set(km.tolist()) == {16, 32}
    wave = torch.from_numpy(b["wave"]).cuda()
    kw = {"mix": MIX} if form == "mix" else {"precision": fsmp.FSMP_FP32_REFRESH, "refresh_M": 64}
    smp = fsmp.Sampler(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay,
                       t0_min=wl.t0_min, t0_max=wl.t0_max, n_steps=400, burn_in=200, seed=2, **kw)
    print(f"[case] autotune {form}", flush=True)
    fresh = _launches(smp, wave, b, km)
    designs = smp.autotune(wave, b["offsets"], b["lam"], kmax=km, trial_steps=200)
    print(f"[autotune] {designs}", flush=True)
    tuned = _launches(smp, wave, b, km)
    # 600 chains are a twentieth of what the kernels for few chains are the faster ones for
    # (3.2 against 8-13 us a sweep; 1.1 against 1.4 and 1.4 against 2.7 ms for 4,000 chains)
    assert designs[16] == designs[32] == fsmp.FSMP_DESIGN_AUTO
    assert tuned == fresh
    if form == "mix":
        assert all(not name.startswith("chain_group_dm") for name, _ in tuned.values())
    else:
        assert set(tuned) == {32}  # one launch for both
    assert all(designs[c] == smp.get_design(c) for c in synth.KCAPS)
