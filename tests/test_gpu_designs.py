"""Which kernels a context runs (needs an MI355X): the design a capacity is set to, or left to the
library, names the kernels that its launches report."""
import numpy as np
import pytest

import oracle
from paper_2403_03156_amd import fsmp, synth
from tests.fsmp_cases import check_partings, compare_chains, gpu_sampler, oracle_params, to_host

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


def _mixed(wl, lam, seed=7):
    b = synth.generate(wl, n_wave=len(lam), seed=seed, lam=np.asarray(lam, float))
    return b, synth.kmax_for(b["lam"]), torch.from_numpy(b["wave"]).cuda()


PINNED = {fsmp.FSMP_DESIGN_GROUP_LDS: ("chain_group_k", {96: 128, 128: 128, 160: 192}),
          fsmp.FSMP_DESIGN_GROUP_DEVMEM: ("chain_group_dm_k", {96: 16, 128: 32, 160: 32}),
          fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE_ONLY: ("chain_group_dm_k", {96: 64, 128: 64, 160: 64})}


@pytest.mark.parametrize("design", list(PINNED))
@pytest.mark.parametrize("start", [False, True])
def test_pinned_kernels_against_the_oracle(design, start):
    # every kernel of capacities 96 to 160, whatever the number of chains: birth by birth from no
    # PEs, and from start lists
    wl = synth.PRESETS["pileup"]
    lam = [45.0, 50.0, 58.0, 62.0, 75.0, 85.0, 92.0, 100.0]
    b, km, wave = _mixed(wl, lam)
    assert set(km.tolist()) == {96, 128, 160}
    n_steps, burn, seed, kz = 200, 80, 11, 160
    print(f"[case] pinned {design} start lists {start}", flush=True)
    kw, okw = {}, {}
    if start:
        z = [np.unique(np.clip(np.rint(np.asarray(t) * 4), 4 * 101, 4 * 1024 - 1).astype(int))[:k - 2].tolist()
             for t, k in zip(b["times"], km)]
        kw = dict(z_init=z, t0_init=np.full(len(km), 100.0))
        okw = dict(z_init=z, t0_init=np.full(len(km), 100.0))

    def sampler(flags):
        s = gpu_sampler(wl, n_steps, burn, 1, seed, k_max=kz, record_flags=flags)
        s.set_design(0, fsmp.FSMP_DESIGN_GROUP_DEVMEM)
        for cap in (96, 128, 160):
            s.set_design(cap, design)
        return s

    smp = sampler(0)
    name, lanes = PINNED[design]
    t = _launches(smp, wave, b, km, kz=kz, **kw)
    assert {c: v[1] for c, v in t.items()} == lanes and all(v[0].startswith(name) for v in t.values()), t
    g = to_host(smp.sample(wave, b["offsets"], b["lam"], kmax=km, kz=kz, **kw))
    p = oracle_params(wl)
    o = oracle.run(p, b["wave"], b["offsets"], b["lam"], 1, n_steps, burn, seed, kz, kmax=km, **okw)
    parted = compare_chains(g, o)
    assert (g["n_pe"] > 10).all()
    if start:
        assert len(parted) == 0, parted
    else:
        check_partings(parted, p, b, b["lam"], km, 1, n_steps, burn, seed, kz, sampler)


def test_wide_groups_where_they_do_not_exist():
    wl = synth.PRESETS["plain"]
    smp = gpu_sampler(wl, 10, 5, 1, 1)
    for cap in (16, 32, 48, 64, 192):
        with pytest.raises(RuntimeError):
            smp.set_design(cap, fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE_ONLY)
    smp.set_design(0, fsmp.FSMP_DESIGN_GROUP_DEVMEM)
    smp.set_design(0, fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE_ONLY)
    assert [smp.get_design(c) for c in synth.KCAPS] == [2] * 4 + [7] * 3 + [2]


def test_replays_with_the_pinned_wide_groups():
    # the wide design and the pinned one replay the same kernels
    wl = synth.PRESETS["pileup"]
    b, km, wave = _mixed(wl, [50.0, 70.0, 95.0])
    p = oracle_params(wl)
    o = oracle.run(p, b["wave"], b["offsets"], b["lam"], 1, 60, 30, 4, 160, kmax=km, log=True)
    out = []
    for d in (fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE, fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE_ONLY):
        s = gpu_sampler(wl, 60, 30, 1, 4, k_max=160)
        s.set_design(0, d)
        dnu, la, _ = s.replay(wave, b["offsets"], b["lam"], np.asarray(o.log), kmax=km, kz=160)
        out.append((dnu.cpu().numpy(), la.cpu().numpy()))
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])


def test_mixture_in_the_device_memory_groups():
    wl = synth.PRESETS["batched"]
    b, km, wave = _mixed(wl, np.concatenate([np.linspace(0.3, 22.0, 24), [40.0, 60.0]]))
    assert set(km.tolist()) >= {16, 32, 48, 64, 96}
    n_steps, burn, seed, kz = 200, 100, 5, int(km.max())
    print("[case] mixture, device-memory groups", flush=True)
    smp = fsmp.Sampler(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay,
                       t0_min=wl.t0_min, t0_max=wl.t0_max, sigma_eps=wl.sigma_eps, n_steps=n_steps, burn_in=burn,
                       seed=seed, k_max=kz, mix=MIX)
    smp.set_design(0, fsmp.FSMP_DESIGN_GROUP_DEVMEM)
    assert all(v[0].startswith("chain_group_dm") for v in _launches(smp, wave, b, km, kz=kz).values())
    g = to_host(smp.sample(wave, b["offsets"], b["lam"], kmax=km, kz=kz))
    p = oracle_params(wl)
    p.n_mix = len(MIX[0])
    for i in range(p.n_mix):
        p.mix_w[i], p.mix_mu[i], p.mix_sigma[i] = MIX[0][i], MIX[1][i], MIX[2][i]
    o = oracle.run(p, b["wave"], b["offsets"], b["lam"], 1, n_steps, burn, seed, kz, kmax=km)
    parted = compare_chains(g, o)
    assert len(parted) == 0, parted
    np.testing.assert_array_equal(g["comp"], o.e)


def test_mixed_precision_in_the_narrow_groups():
    wl = synth.PRESETS["batched"]
    b, km, wave = _mixed(wl, np.linspace(0.3, 9.0, 60))
    assert set(km.tolist()) == {16, 32}
    n_steps, burn, seed, kz = 300, 150, 31, 32
    print("[case] mixed precision, narrow groups", flush=True)

    def sampler(flags):
        s = fsmp.Sampler(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay,
                         t0_min=wl.t0_min, t0_max=wl.t0_max, sigma_eps=wl.sigma_eps, mu_q=wl.mu_q,
                         sigma_q=wl.sigma_q, n_steps=n_steps, burn_in=burn, seed=seed, record_flags=flags, k_max=kz,
                         precision=fsmp.FSMP_FP32_REFRESH, refresh_M=64)
        for cap in (16, 32):
            s.set_design(cap, fsmp.FSMP_DESIGN_GROUP_DEVMEM)
        return s

    smp = sampler(0)
    assert {v[1] for v in _launches(smp, wave, b, km, kz=kz).values()} == {4}  # lanes per chain
    g = to_host(smp.sample(wave, b["offsets"], b["lam"], kmax=km, kz=kz))
    p = oracle_params(wl)
    o = oracle.run(p, b["wave"], b["offsets"], b["lam"], 1, n_steps, burn, seed, kz, kmax=km)
    parted = compare_chains(g, o, tol=1e-7)
    check_partings(parted, p, b, b["lam"], km, 1, n_steps, burn, seed, kz, sampler)


def test_long_responses_at_any_number_of_chains():
    # a response whose overlap table takes the LDS of the device-memory groups: accepted for few chains
    # and for more than the LDS kernels are otherwise chosen for, with the same results
    wl = synth.Workload("long", 8, (600,), "uniform", 0.5, 6.0, ser=(8.0, 1.5, 45.0))
    b = synth.generate(wl, n_wave=8, seed=3)
    km = np.array([16, 32, 48, 64] * 2, np.int32)
    r = 1800  # 3,600 chains per capacity: past the 3,500 of capacity 64
    s = gpu_sampler(wl, 20, 10, 1, 2, sub=8, support=512)
    with pytest.raises(RuntimeError):
        s.set_design(64, fsmp.FSMP_DESIGN_GROUP_DEVMEM)
    print("[case] long response", flush=True)
    few = to_host(s.sample(torch.from_numpy(b["wave"]).cuda(), b["offsets"], b["lam"], kmax=km, kz=64))
    off = np.arange(8 * r + 1, dtype=np.int64) * 600
    many = to_host(s.sample(torch.from_numpy(np.tile(b["wave"], r)).cuda(), off, np.tile(b["lam"], r),
                            kmax=np.tile(km, r), kz=64, wave_id=np.tile(np.arange(8, dtype=np.uint64), r)))
    for k in KEYS:
        np.testing.assert_array_equal(many[k][-8:], few[k], err_msg=k)
    p = oracle_params(wl, sub=8, support=512)
    o = oracle.run(p, b["wave"], b["offsets"], b["lam"], 1, 20, 10, 2, 64, kmax=km)
    assert len(compare_chains(few, o)) == 0


def _kernels(smp, cap, n, lam, lists=0):
    """the kernel name and the outputs of n chains of one capacity"""
    wl = synth.PRESETS["batched"]
    m = 40
    b = synth.generate(wl, n_wave=m, seed=6, lam=np.full(m, 20.0), lengths=np.full(m, 300))
    r = n // m
    kw = {}
    if lists:
        z = [np.arange(4 * 80, 4 * 80 + 3 * lists, 3).tolist()] * (m * r)
        kw.update(z_init=z, t0_init=np.full(m * r, 75.0))
    km, la = np.full(m * r, cap, np.int32), np.full(m * r, float(lam))
    smp.set_timing(True)
    out = smp.sample(torch.from_numpy(np.tile(b["wave"], r)).cuda(), np.arange(m * r + 1, dtype=np.int64) * 300, la,
                     kmax=km, kz=cap, **kw)
    t = [x["name"] for x in smp.last_timings() if x["kcap"] == cap]
    return t[0], to_host(out), b, m


# capacity, chains, intensity, sweeps, length of the start lists: the kernels of lists that stay short
# against those of lists near the capacity.  Both sides as measured, microseconds a sweep LDS / narrow.
@pytest.mark.parametrize("cap,n,lam,steps,lists,lds", [
    (192, 4000, 2.0, 200, 0, False),    # K_max far above the intensity: 65 / 12
    (192, 4000, 130.0, 20, 120, True),  # 145 / 200
    (160, 2000, 90.0, 100, 0, False),   # a short run from no PEs: 33 / 7
    (160, 2000, 120.0, 20, 110, True),  # 66 / 99
    (160, 320, 90.0, 100, 0, True),
    (128, 4000, 80.0, 20, 75, True),    # 60 / 100
    (128, 2000, 5.0, 200, 0, False),    # 17 / 7
    (96, 3000, 4.0, 200, 0, False),     # 17 / 9
    (96, 5000, 60.0, 2000, 0, True),
    (64, 3400, 4.0, 200, 0, False),     # 14 / 8
    (48, 5000, 2.0, 200, 0, False),     # 14 / 9
    (32, 10000, 1.0, 200, 0, False),
    (32, 10000, 8.0, 200, 0, True),
])
def test_routes_follow_the_length_of_the_lists(cap, n, lam, steps, lists, lds):
    smp = gpu_sampler(synth.PRESETS["batched"], steps, steps // 2, 1, 4, k_max=cap)
    print(f"[case] route {cap} {n} {lam} {steps} {lists}", flush=True)
    name, g, b, m = _kernels(smp, cap, n, lam, lists)
    assert name.startswith("chain_group_dm") == (not lds), name
    if lists == 0 and steps <= 200:
        p = oracle_params(synth.PRESETS["batched"])
        o = oracle.run(p, b["wave"], b["offsets"], np.full(m, lam), 1, steps, steps // 2, 4, cap,
                       kmax=np.full(m, cap, np.int32))
        part = {k: (v[:m] if isinstance(v, np.ndarray) else v) for k, v in g.items()}
        assert len(compare_chains(part, o)) == 0


def test_workspace_follows_the_route():
    # the predicted workspace is that of the kernels that run: K^2 per chain in LDS, 2 K^2 beside it
    wl = synth.PRESETS["batched"]
    for lam, words in ((2.0, 2), (190.0, 1)):
        smp = gpu_sampler(wl, 4000, 10, 1, 4, k_max=192)
        off = np.arange(4001, dtype=np.int64) * 300
        big = smp.workspace_bytes(off, np.full(4000, lam), kmax=np.full(4000, 192, np.int32))
        assert abs(big - 4000 * words * 192 * 192 * 8) < 100e6
