"""Serving bright channels (needs an MI355X): an event's results are the same bits alone and in a
micro-batch of more chains than the kernels for few chains are chosen for."""
import numpy as np
import pytest

from paper_2403_03156_amd import fsmp, synth
from tests.test_gpu_serving import _serve

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["single", "mix"])
def test_bright_event_alone_equals_mixed(form):
    wl = synth.PRESETS["serving"]
    kw = dict(ser=wl.ser, phi_kind=wl.phi_kind, tau_rise=wl.tau_rise, tau_decay=wl.tau_decay, t0_min=wl.t0_min,
              t0_max=wl.t0_max, sigma_eps=wl.sigma_eps, mu_q=wl.mu_q, sigma_q=wl.sigma_q, n_steps=160, n_chains=1,
              seed=3)
    if form == "mix":
        kw["mix"] = ([0.3, 0.7], [0.6, 1.2], [0.2, 0.3])
    small = synth.generate(wl, n_wave=30, seed=4, lam=np.full(30, 60.0), lengths=np.full(30, 256))
    km = np.where(np.arange(30) % 2, 160, 128).astype(np.int32)
    m, r = 100, 65  # 6,500 channels more of capacity 160
    base = synth.generate(wl, n_wave=m, seed=5, lam=np.full(m, 60.0), lengths=np.full(m, 256))
    big = {"wave": np.tile(base["wave"], r), "lam": np.tile(base["lam"], r),
           "offsets": np.arange(m * r + 1, dtype=np.int64) * 256}
    big_km = np.full(m * r, 160, np.int32)
    print(f"[case] bright event {form}", flush=True)
    srv = fsmp.Server(kw, n_streams=1, max_batch_wave=1 << 20)
    alone = _serve(srv, [(7, small, km)])[7]
    mixed = _serve(srv, [(7, small, km), (9, big, big_km)])[7]
    srv.close()
    assert (alone["mean"][:, 0] > 3).all()
    for k in ("mean", "mcse", "status"):
        np.testing.assert_array_equal(alone[k], mixed[k], err_msg=k)
