"""The NUFFT spread's two forms (element terms staged for a workgroup, or a lane's own) on both
sides of the rule that chooses, against the FP64 oracle: elements around a quarter of the
workgroup's lanes, waves with idle lanes and workgroups with idle waves, runs longer than a batch,
and the delay within the chirp. Tolerance: the relative RMS bar of the FP32 sum, 1e-4."""
import numpy as np
import pytest

import oracle
import scenes
from scenes import RadarArray

pytestmark = pytest.mark.gpu

NUFFT = 3


@pytest.mark.parametrize("P,Q,intra", [
    (4, 12, False),   # 16 elements of 64 lanes: staged
    (1, 16, False),   # 17, and 16 channels: own terms, 48 idle lanes
    (1, 16, True),
    (3, 30, True),    # 33 of 128 lanes, the second wave part idle
    (64, 1, True),    # the most elements of one wave
    (2, 64, False),
    (64, 5, False),   # 69 of 256 lanes, five waves: three idle ones in the second workgroup
    (64, 5, True),
])
def test_forms_against_oracle(P, Q, intra):
    from paper_2208_10939_amd.pipeline import Simulator
    print(f"case spread form P={P} Q={Q} intra={intra}", flush=True)
    cfg = scenes.small_single(n_samples=64, n_chirps=1, n_tris=4000)
    sc, wf = cfg.scenes[0], cfg.waveform
    c = cfg.array.tx.mean(0)
    arr = RadarArray(tx=c + [[0.002 * (k % 8), 0.0, 0.002 * (k // 8)] for k in range(P)],
                     rx=c + [[0.002 * (k % 8), 0.0, -0.002 * (k // 8)] for k in range(Q)])
    sim = Simulator([sc], wf, arr)
    omask, _ = oracle.visibility(sc, arr, wf)
    H = sim.synthesize(mask=sim.mask_from_numpy([omask]), mask_mode=1, kernel=NUFFT,
                       intra_chirp=intra).cpu().numpy()[0]
    ch = np.unique(np.linspace(0, P * Q - 1, 24).astype(int))
    Ho = oracle.synthesize(sc, wf, arr, mask=omask, channels=ch, intra_chirp=intra)
    err = float(np.sqrt(np.sum(np.abs(H[ch] - Ho) ** 2) / np.sum(np.abs(Ho) ** 2)))
    print(f"  rel_rms={err:.3e}", flush=True)
    assert err <= 1e-4
