"""The NUFFT spread's element terms (a lane per record and Tx or Rx element) and block selection
at their edges, against the FP64 oracle (Sections 2.2 and 3.2, eqs. (7)-(13)): element counts
that change how many records are staged together, channel counts around 64 and beyond four
waves, apertures that ask for longer blocks, and the delay within the chirp. Tolerance: the
relative RMS bar of the FP32 sum, 1e-4."""
import numpy as np
import pytest

import oracle
import scenes
from scenes import RadarArray

pytestmark = pytest.mark.gpu

NUFFT = 3


def rel_rms(a, b):
    return float(np.sqrt(np.sum(np.abs(a - b) ** 2) / np.sum(np.abs(b) ** 2)))


def _array(arr, P, Q, scale):
    tx, rx = np.array(arr.tx), np.array(arr.rx)
    c = 0.5 * (tx.mean(0) + rx.mean(0))

    def take(e, n):  # n elements: the array's rows repeated 4 mm apart
        return np.concatenate([e + [0, 0, 0.004 * k] for k in range(-(-n // len(e)))])[:n]

    return RadarArray(tx=c + scale * (take(tx, P) - c), rx=c + scale * (take(rx, Q) - c))


@pytest.mark.parametrize("n_tris,M,P,Q,scale,intra", [
    (1500, 256, 12, 16, 1.0, False),  # 28 elements, blocks of 14 cells
    (1500, 256, 12, 16, 2.5, False),  # 16 cells
    (300, 256, 12, 16, 5.0, True),    # 20 cells, sources up to 4.8 cells apart
    (600, 64, 40, 30, 0.5, False),    # 70 elements, 1200 channels: five planes of waves
    (600, 64, 40, 30, 0.5, True),
    (600, 64, 64, 1, 0.3, False),     # 65 elements
    (600, 96, 5, 13, 1.0, True),      # 65 channels: a wave with one
    (600, 96, 1, 1, 1.0, False),
])
def test_spread_against_oracle(n_tris, M, P, Q, scale, intra):
    from paper_2208_10939_amd.pipeline import Simulator
    print(f"case spread n_tris={n_tris} M={M} P={P} Q={Q} x{scale} intra={intra}", flush=True)
    cfg = scenes.small_single(n_samples=M, n_chirps=1, n_tris=n_tris)
    sc, wf = cfg.scenes[0], cfg.waveform
    arr = _array(cfg.array, P, Q, scale)
    sim = Simulator([sc], wf, arr)
    omask, _ = oracle.visibility(sc, arr, wf)
    H = sim.synthesize(mask=sim.mask_from_numpy([omask]), mask_mode=1, kernel=NUFFT,
                       intra_chirp=intra).cpu().numpy()[0]
    ch = np.unique(np.linspace(0, P * Q - 1, 40).astype(int))
    Ho = oracle.synthesize(sc, wf, arr, mask=omask, channels=ch, intra_chirp=intra)
    err = rel_rms(H[ch], Ho)
    print(f"  rel_rms={err:.3e}", flush=True)
    assert err <= 1e-4
