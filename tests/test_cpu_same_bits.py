"""The kernels that hold the same chains write the same arithmetic: on the CPU, where nothing fuses a
product into a sum that the source does not fuse, the LDS chains and the narrow device-memory groups
of capacities 16 to 64 give the same bits."""
import numpy as np
import pytest

from paper_2403_03156_amd import fsmp, synth
from tests.test_cpu_emu import MIX, _run_emu

KEYS = ("n_pe", "t0", "z", "charge", "acc", "nhist", "counts", "status", "trace", "zdraw", "qdraw")


@pytest.mark.parametrize("mix,n_steps", [(None, 140), (MIX, 60)])  # (G^-1 is rebuilt after 128 sweeps)
def test_lds_and_device_memory_groups_agree_bit_for_bit(tmp_path, mix, n_steps):
    wl = synth.PRESETS["batched"]
    lam = np.array([3.0, 9.0, 13.0, 20.0])
    b = synth.generate(wl, n_wave=len(lam), seed=14, lam=lam, lengths=np.array([300] * 4))
    km = np.array([16, 32, 48, 64], np.int32)
    flags = fsmp.FSMP_REC_LOG | fsmp.FSMP_REC_TRACE | fsmp.FSMP_REC_CHARGE
    out = []
    for name, design in (("lds", fsmp.FSMP_DESIGN_GROUP_LDS), ("dm", fsmp.FSMP_DESIGN_GROUP_DEVMEM)):
        d = tmp_path / name
        d.mkdir()
        out.append(_run_emu(str(d), wl, b["wave"], b["offsets"], b["lam"], km, n_steps, 20, 1, 8, [design] * 8,
                            record_flags=flags, thin=25, mix=mix))
    assert (out[0]["n_pe"][2:] > 5).all()
    for k in KEYS:
        np.testing.assert_array_equal(out[0][k], out[1][k], err_msg=k)


def test_the_records_of_every_step_agree_bit_for_bit(tmp_path):
    wl = synth.PRESETS["pileup"]
    lam = np.array([0.8, 9.0, 14.0, 21.0])
    b = synth.generate(wl, n_wave=len(lam), seed=15, lam=lam, lengths=np.array([300] * 4))
    km = np.array([16, 32, 48, 64], np.int32)
    log = []
    for name, design in (("lds", fsmp.FSMP_DESIGN_GROUP_LDS), ("dm", fsmp.FSMP_DESIGN_GROUP_DEVMEM)):
        d = tmp_path / name
        d.mkdir()
        log.append(_run_emu(str(d), wl, b["wave"], b["offsets"], b["lam"], km, 60, 20, 1, 9, [design] * 8,
                            record_flags=fsmp.FSMP_REC_LOG)["log"])
    for f in ("move", "flags", "j", "g", "t0", "dnu", "log_alpha"):
        np.testing.assert_array_equal(log[0][f], log[1][f], err_msg=f)
