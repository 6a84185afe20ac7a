"""The LDS chains (G^-1 in LDS) at the edges of their capacities, light curves and routes (needs
an MI355X).  Against the oracle: PE lists, histograms and counts equal, t0, accumulators and
charges to 1e-9 (the bound of the FP64 form).  Against the narrow device-memory groups: bit for
bit up to capacity 64, where both take sums, products and edits in the same order and rounding,
so that a chain's outputs do not depend on which of the two the number of chains selects."""
import numpy as np
import pytest

import oracle
from paper_2403_03156_amd import fsmp, synth
from tests.fsmp_cases import check_partings, compare_chains, gpu_sampler, oracle_params, to_host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
KEYS = ("n_pe", "t0", "z", "charge", "acc", "nhist", "counts", "status")


def _against_oracle(wl, b, km, n_steps, burn, seed, sub=4, g_range=None, t0_sd=1.0):
    kz = int(km.max())
    smp = lambda flags: gpu_sampler(wl, n_steps, burn, 1, seed, k_max=kz, record_flags=flags, sub=sub, t0_sd=t0_sd)
    out = smp(0).sample(torch.from_numpy(b["wave"]).cuda(), b["offsets"], b["lam"], kmax=km, kz=kz, g_range=g_range)
    torch.cuda.synchronize()
    p = oracle_params(wl, sub=sub, t0_sd=t0_sd)
    o = oracle.run(p, b["wave"], b["offsets"], b["lam"], 1, n_steps, burn, seed, kz, kmax=km, g_range=g_range)
    g = to_host(out)
    parted = compare_chains(g, o)
    if g_range is None:
        check_partings(parted, p, b, b["lam"], km, 1, n_steps, burn, seed, kz, smp)
    else:
        assert len(parted) == 0, parted
    return g


@pytest.mark.parametrize("caps", [(1, 15, 16), (17, 31, 32), (33, 47, 48), (49, 64), (65, 95, 96), (97, 128),
                                  (129, 160), (161, 191, 192)])
def test_capacity_edges(caps):
    # lists that reach K_max (PEs rejected there) at the first, last and inner sizes of a capacity
    wl = synth.PRESETS["pileup"]
    km = np.repeat(np.array(caps, np.int32), 3)
    lam = np.where(km < 64, km * 1.2 + 1.0, 110.0)
    b = synth.generate(wl, n_wave=len(km), seed=7, lam=lam)
    print(f"[case] capacity edges {caps}", flush=True)
    g = _against_oracle(wl, b, km, 400, 200, 5)
    if max(caps) <= 64:
        assert (g["status"] & 1).any()


@pytest.mark.parametrize("rise,decay,sub,length", [
    (2.0, 25.0, 4, 130),   # windows that end inside the response: the table of partial overlap sums
    (0.3, 10.0, 1, 256),   # dt / tau above 1/4: the library's exponentials
    (20.0, 25.0, 16, 300),  # a rise over more grid points than the table holds
    (2.0, 25.0, 3, 256),   # a grid step that is no power of two
])
def test_light_curves(rise, decay, sub, length):
    wl = synth.Workload("lc", 20, (length,), "uniform", 0.5, 12.0, phi_kind=synth.PHI_BIEXP, tau_rise=rise,
                        tau_decay=decay)
    b = synth.generate(wl, n_wave=20, seed=3)
    print(f"[case] light curve rise {rise} decay {decay} sub {sub} length {length}", flush=True)
    _against_oracle(wl, b, synth.kmax_for(b["lam"]), 300, 150, 9, sub=sub)


def test_solution_spaces():
    # T that starts after every t0, one that ends before some, a single point, and none
    wl = synth.PRESETS["batched"]
    b = synth.generate(wl, n_wave=16, seed=4, lam=np.full(16, 6.0))
    gr = np.array([[420, 4 * 1024 - 1], [0, 330], [400, 400], [1, 0]] * 4, np.int32)
    print("[case] solution spaces", flush=True)
    _against_oracle(wl, b, synth.kmax_for(b["lam"]), 300, 150, 9, g_range=gr)


@pytest.mark.parametrize("preset", ["plain", "batched", "pileup"])
def test_same_bits_as_the_device_memory_groups(preset):
    wl = synth.PRESETS[preset]
    lam = np.linspace(0.2, 22.0, 48)
    b = synth.generate(wl, n_wave=48, seed=12, lam=lam)
    km = synth.kmax_for(lam)
    assert set(km.tolist()) == {16, 32, 48, 64}
    wave = torch.from_numpy(b["wave"]).cuda()
    out = []
    for design, timed in ((None, False), (None, True), (fsmp.FSMP_DESIGN_GROUP_DEVMEM, False)):
        s = gpu_sampler(wl, 500, 250, 2, 21)  # one launch for all capacities; one each; device memory
        s.set_timing(timed)
        if design is not None:
            s.set_design(0, design)
        out.append(to_host(s.sample(wave, b["offsets"], lam, kmax=km, kz=64)))
    for k in KEYS:
        np.testing.assert_array_equal(out[0][k], out[1][k], err_msg=k)
        np.testing.assert_array_equal(out[0][k], out[2][k], err_msg=k)


def test_a_chain_does_not_depend_on_the_number_of_chains():
    # capacity 16 in LDS alone, in the device-memory groups among 15,000
    wl = synth.PRESETS["plain"]
    b = synth.generate(wl, n_wave=100, seed=2, lam=np.linspace(0.1, 2.0, 100))
    km = np.full(100, 16, np.int32)
    s = gpu_sampler(wl, 120, 60, 1, 3)
    few = to_host(s.sample(torch.from_numpy(b["wave"]).cuda(), b["offsets"], b["lam"], kmax=km, kz=16))
    r = 150
    off = np.concatenate([b["offsets"], b["offsets"][-1] * np.arange(1, r)[:, None] + b["offsets"][1:][None]], axis=None)
    many = to_host(s.sample(torch.from_numpy(np.tile(b["wave"], r)).cuda(), off, np.tile(b["lam"], r),
                            kmax=np.tile(km, r), kz=16, wave_id=np.tile(np.arange(100, dtype=np.uint64), r)))
    for k in KEYS:
        np.testing.assert_array_equal(many[k][-100:], few[k], err_msg=k)


def test_mixed_precision_capacities_joined():
    # capacities 16 and 32 in one launch (no design set) and in one each (the wide groups set)
    wl = synth.PRESETS["batched"]
    b = synth.generate(wl, n_wave=40, seed=6, lam=np.linspace(0.2, 8.0, 40))
    km = synth.kmax_for(b["lam"])
    assert set(km.tolist()) == {16, 32}
    wave = torch.from_numpy(b["wave"]).cuda()
    out = []
    for wide in (False, True):
        s = fsmp.Sampler(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay,
                         t0_min=wl.t0_min, t0_max=wl.t0_max, n_steps=200, burn_in=100, seed=4,
                         precision=fsmp.FSMP_FP32_REFRESH, refresh_M=64)
        if wide:
            s.set_design(16, fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE)
            s.set_design(32, fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE)
        out.append(to_host(s.sample(wave, b["offsets"], b["lam"], kmax=km, kz=32)))
    for k in KEYS:
        np.testing.assert_array_equal(out[0][k], out[1][k], err_msg=k)


def test_lambda_estimate_of_long_rows():
    # histogram rows of more than 2,048 entries are read from device memory: the same estimates
    wl = synth.PRESETS["batched"]
    b = synth.generate(wl, n_wave=24, seed=8)
    km = synth.kmax_for(b["lam"])
    wave = torch.from_numpy(b["wave"]).cuda()
    est = []
    for kz in (64, 2100):
        s = gpu_sampler(wl, 200, 100, 2, 5)
        out = s.sample(wave, b["offsets"], b["lam"], kmax=km, kz=kz)
        post = s.posterior(24, out, diagnostics=True, lam=b["lam"])
        est.append({k: post[k].cpu().numpy() for k in ("lambda_hat", "mean", "rhat")})
    for k in est[0]:
        np.testing.assert_array_equal(est[0][k], est[1][k], err_msg=k)


def test_deconvolution_by_length_class():
    # more windows than run at once: one launch per length class; against the windows alone (one
    # launch, other workgroup sizes: the start's total is summed in another order, 1e-9)
    wl = synth.PRESETS["uneven"]
    rng = np.random.default_rng(1)
    lengths = np.concatenate([[1, 63, 64, 65, 128, 129, 2048], rng.integers(60, 1200, 1100)])
    b = synth.generate(wl, n_wave=len(lengths), seed=5, lam=rng.uniform(0.5, 8.0, len(lengths)), lengths=lengths)
    km = synth.kmax_for(b["lam"])
    s = gpu_sampler(wl, 100, 50, 1, 1)
    wave = torch.from_numpy(b["wave"]).cuda()
    lv = s.support_samples()
    a = {k: v.cpu().numpy() if v is not None and k != "kz" else v
         for k, v in s.lucy(wave, b["offsets"], kmax=km, n_iter=30, qhat=True).items()}
    n = 12
    off = b["offsets"][:n + 1]
    f = {k: v.cpu().numpy() if v is not None and k != "kz" else v
         for k, v in s.lucy(wave[:int(off[-1])].contiguous(), off, kmax=km[:n], kz=a["kz"], n_iter=30, qhat=True).items()}
    for k in ("z", "n_pe", "g_range", "cut"):
        np.testing.assert_array_equal(a[k][:n], f[k], err_msg=k)
    m = int(off[-1]) + n * (lv - 1)
    np.testing.assert_allclose(a["qhat"][:m], f["qhat"], rtol=1e-9, atol=1e-15)
    np.testing.assert_allclose(a["lambda"][:n], f["lambda"], rtol=1e-9)
    np.testing.assert_array_equal(a["t0"][:n], f["t0"])
