"""The LDS chains above capacity 64 (a workgroup of two or three wavefronts per chain, the matrix by
wrapped diagonals) and the mixture law's, on the CPU under AddressSanitizer against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2403_03156_amd import synth
from tests.fsmp_cases import compare_chains, oracle_params
from tests.test_cpu_emu import MIX, _run_emu


@pytest.mark.parametrize("caps,mix", [((96, 128), None), ((160, 192), None), ((16, 32), MIX), ((48, 96), MIX)])
def test_lds_chains_on_the_cpu_under_asan(tmp_path, caps, mix):
    wl = synth.PRESETS["pileup"]
    km = np.array(caps, np.int32)
    b = synth.generate(wl, n_wave=2, seed=31, lam=np.minimum(km * 0.8, 100.0), lengths=np.array([300, 160]))
    n_steps, burn, seed = 60, 30, 3
    g = _run_emu(str(tmp_path), wl, b["wave"], b["offsets"], b["lam"], km, n_steps, burn, 1, seed, [-1] * 8, mix=mix)
    p = oracle_params(wl)
    if mix is not None:
        p.n_mix = len(mix[0])
        for i in range(p.n_mix):
            p.mix_w[i], p.mix_mu[i], p.mix_sigma[i] = mix[0][i], mix[1][i], mix[2][i]
    o = oracle.run(p, b["wave"], b["offsets"], b["lam"], 1, n_steps, burn, seed, int(km.max()), kmax=km)
    parted = compare_chains(g, o)
    assert len(parted) == 0, parted
