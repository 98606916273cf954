"""Scenes of more instances than fit one word (32) or both words (64) of the instance filters that
visibility and the connection search keep: 40 and 70 boxes in rows, the later ones nearer to the
radar, so that boxes from index 32 and from index 64 on block the ones behind them and take their
reflections. Masks and connections of the first and last chirp against the FP64 oracle; they may
differ only where the oracle calls a decision ambiguous."""
import numpy as np
import pytest

import oracle
import scenes
from oracle import dbounce
from scenes import Instance, Scene

pytestmark = pytest.mark.gpu


def _boxes(n):
    rng = np.random.default_rng(n)
    box = scenes.box_mesh([-0.6, -0.5, 0.0], [0.6, 0.5, 1.4], (2, 2, 2))
    return Scene([box], [Instance(0, scenes.yaw_matrix(rng.uniform(-0.6, 0.6)),
                                  np.array([-5.0 + 2.2 * (k % 6) + rng.uniform(-0.3, 0.3),
                                            44.0 - 2.6 * (k // 6) + rng.uniform(-0.3, 0.3), 0.0]),
                                  np.array([0.2 * rng.standard_normal(), rng.uniform(-8, 8), 0.0]))
                         for k in range(n)])


@pytest.mark.parametrize("n,N", [(40, 66), (70, 66), (70, 5)])
def test_masks_against_oracle(n, N):
    from paper_2208_10939_amd.pipeline import Simulator
    print(f"case masks of {n} instances N={N}", flush=True)
    cfg = scenes.small_single(n_samples=16, n_chirps=N, n_tris=300)
    sc, wf, arr = _boxes(n), cfg.waveform, cfg.array
    sim = Simulator([sc], wf, arr)
    mask = sim.mask_buffer()
    sim.synthesize(mask=mask, kernel=3)
    chirps = np.array([0, N - 1])
    om, amb = oracle.visibility(sc, arr, wf, chirps=chirps)
    per = sc.n_tris // n
    for first in (k for k in (32, 64) if k < n):  # without these instances more would be lit
        less, _ = oracle.visibility(Scene(sc.meshes, sc.instances[:first]), arr, wf, chirps=chirps)
        assert (less & ~om[:, :first * per]).any()
    bad = (sim.masks_numpy(mask)[0][chirps] != om) & ~amb
    assert not bad.any(), f"{bad.sum()} unambiguous mask mismatches"


@pytest.mark.parametrize("n,N", [(40, 3), (70, 5)])
def test_connections_against_oracle(n, N):
    from paper_2208_10939_amd.pipeline import Simulator
    print(f"case connections of {n} instances N={N}", flush=True)
    cfg = scenes.small_single(n_samples=16, n_chirps=N, n_tris=300)
    sc, wf, arr = _boxes(n), cfg.waveform, cfg.array
    sim = Simulator([sc], wf, arr)
    sim.set_double_bounce(True, -1.0)
    mask = sim.mask_buffer()
    sim.synthesize(mask=mask)
    chirps = np.array([0, N - 1])
    pairs = dbounce.double_bounce_pairs(sc, arr, wf, chirps=chirps)
    want = dbounce.connection_table(pairs, sc.n_tris)
    amb = np.zeros_like(want, bool)
    for i, ends in enumerate(pairs):
        for k in (0, 1):
            amb[k, i, ends[k]["amb_facets"]] = True
    b = want[want >= 0] // (sc.n_tris // n)
    assert (b >= 32).any() and (n <= 64 or (b >= 64).any())
    bad = (sim.connections_numpy(mask)[0][:, chirps] != want) & ~amb
    assert not bad.any(), f"{bad.sum()} unambiguous connection mismatches"
