"""Sampling in the wide device-memory groups (capacities 96 to 160, a wavefront per chain), on the CPU
under AddressSanitizer against the oracle."""
import numpy as np

import oracle
from paper_2403_03156_amd import fsmp, synth
from tests.fsmp_cases import compare_chains, oracle_params
from tests.test_cpu_emu import _run_emu


def test_wide_groups_on_the_cpu_under_asan(tmp_path):
    wl = synth.PRESETS["pileup"]
    km = np.array([96, 128, 160], np.int32)
    b = synth.generate(wl, n_wave=3, seed=31, lam=km * 0.6, lengths=np.array([300, 160, 512]))
    n_steps, burn, seed = 70, 30, 3
    d = fsmp.FSMP_DESIGN_GROUP_DEVMEM_WIDE_ONLY
    g = _run_emu(str(tmp_path), wl, b["wave"], b["offsets"], b["lam"], km, n_steps, burn, 1, seed,
                 [-1] * 4 + [d] * 3 + [-1], record_flags=fsmp.FSMP_REC_LOG)
    o = oracle.run(oracle_params(wl), b["wave"], b["offsets"], b["lam"], 1, n_steps, burn, seed, int(km.max()),
                   kmax=km, log=True)
    parted = compare_chains(g, o)
    assert len(parted) == 0, parted
    assert (g["n_pe"] > 5).all()
    for f in ("move", "flags", "j", "g"):
        np.testing.assert_array_equal(g["log"][f], o.log[f])
