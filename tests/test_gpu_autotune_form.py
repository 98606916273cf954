"""The autotuner and the cut form of the facet sum's default tiles, which calls with idle CUs take
when no tile is asked for: such a call is not slower after tuning than before it, and the time that
the tuner writes is that of the kernel a tuned call launches. 4 x 8 channels, 4 chirps, 256 samples:
on the vector units the cut form takes some 0.29 ms, the next best tiles 0.42, so the bars (1.2 of
the time, and a quarter of it) lie well apart from either."""
import json

import numpy as np
import pytest

import scenes
from scenes import RadarArray

pytestmark = pytest.mark.gpu

AUTO, VECTOR = 0, 1


def test_tuned_call_is_not_slower(tmp_path):
    from paper_2208_10939_amd.pipeline import Simulator
    cfg = scenes.small_single(n_samples=256, n_chirps=4, n_tris=1500)
    arr = RadarArray(tx=np.array(cfg.array.tx[:4]), rx=np.array(cfg.array.rx[:8]))
    sim = Simulator(cfg.scenes, cfg.waveform, arr)

    def facet_sum_ms(kernel):
        times = []
        for _ in range(6):
            H = sim.synthesize(kernel=kernel, timing=True)
            sim.ctx.sync()
            times.append(sim.ctx.last_timings()["facet_sum"])
        return min(times), H.cpu().numpy()

    before, want = facet_sum_ms(VECTOR)
    for tuning in (1, 2):  # the second with an earlier choice in place
        sim.ctx.autotune(sim.scene_ids, str(tmp_path / "tuned"))
        line = json.loads((tmp_path / "tuned").read_text().splitlines()[-1])
        after, got = facet_sum_ms(VECTOR)
        auto, _ = facet_sum_ms(AUTO)
        print(f"  tuning {tuning}: vector {before:.3f} -> {after:.3f} ms, auto {auto:.3f}, "
              f"stored {line}", flush=True)
        assert after <= 1.2 * before
        assert abs(line["facet_sum_ms"] - auto) <= 0.25 * auto
        assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
