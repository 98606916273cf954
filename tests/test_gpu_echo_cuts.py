"""The facet sum's cut forms (one block of samples a workgroup, a chunk of it a thread), which
plain launches with CUs to spare take, against the whole form, which the persistent launch
takes: the same terms in the same order, so the same bits. Channel counts around the widths of
the cuts, sample counts that end inside a chunk, a block and a tile, both cuts, both types."""
import numpy as np
import pytest

import scenes
from scenes import RadarArray

pytestmark = pytest.mark.gpu

VECTOR = 1


@pytest.mark.parametrize("M,N,P,Q,fp64,intra", [
    (256, 4, 12, 16, False, False),  # 64 channels, 16 samples a thread
    (17, 1, 12, 16, False, True),
    (130, 3, 5, 13, False, False),   # 65 channels: 33 and 32
    (96, 5, 1, 3, False, False),
    (200, 30, 12, 16, False, True),  # 192 channels, 32 samples a thread
    (70, 40, 14, 16, False, False),  # 224 channels: 112 and 112
    (96, 60, 12, 16, False, False),  # not cut
    (100, 8, 1, 4, True, False),     # FP64: 64 channels, 8 samples a thread
    (25, 3, 5, 13, True, False),
    (90, 24, 12, 16, True, False),   # 192 channels
])
def test_cut_forms_same_bits(M, N, P, Q, fp64, intra):
    from paper_2208_10939_amd.pipeline import Simulator
    print(f"case cuts M={M} N={N} P={P} Q={Q} fp64={fp64} intra={intra}", flush=True)
    cfg = scenes.small_single(n_samples=M, n_chirps=N, n_tris=400)
    tx, rx = np.array(cfg.array.tx), np.array(cfg.array.rx)
    arr = RadarArray(tx=np.resize(tx, (P, 3)) + [[0, 0, 0.004 * k] for k in range(P)],
                     rx=np.resize(rx, (Q, 3)) + [[0, 0, 0.004 * k] for k in range(Q)])
    sim = Simulator(cfg.scenes[:1], cfg.waveform, arr)
    kw = dict(precision=int(fp64), intra_chirp=intra, kernel=0 if fp64 else VECTOR)
    cut = sim.synthesize(**kw).cpu().numpy()
    whole = sim.synthesize(persistent=True, **kw).cpu().numpy()
    assert np.abs(whole).max() > 0
    assert np.array_equal(cut, whole)
