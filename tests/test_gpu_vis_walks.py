"""Visibility where each lane walks a BVH for itself (few chirps of many facets) against where a
wave walks it together: a chirp's decisions do not depend on how many chirps the call has, so the
masks of a call on the near side of the rule equal, bit for bit, those of the same chirps in a call
of 12 (tests of both against the oracle: test_gpu_vis_packets.py); one case of own walks is
compared with the FP64 oracle on sampled facets here."""
import numpy as np
import pytest

import oracle
import scenes
from scenes import Instance, Scene

pytestmark = pytest.mark.gpu


def _scene(n_tris, n_inst):
    car = scenes.vehicle_mesh("car", n_tris)
    return Scene([car], [Instance(0, scenes.yaw_matrix(1.5 - 0.4 * k),
                                  np.array([3.0 - 2.5 * k, 14.0 + 3.0 * k, 0.0]),
                                  np.array([0.3, -6.0 + 9.0 * k, 0.0])) for k in range(n_inst)])


def _masks(sc, N, ground):
    from paper_2208_10939_amd.pipeline import Simulator
    cfg = scenes.small_single(n_samples=16, n_chirps=N, n_tris=300)
    sim = Simulator([sc], cfg.waveform, cfg.array)
    if ground:
        sim.set_ground(True, -0.5, -0.7)
    mask = sim.mask_buffer()
    mask.fill_(-1)
    sim.synthesize(mask=mask, kernel=3)
    return mask.cpu().numpy().reshape(4 if ground else 1, N, sim.mask_words[0]), cfg


@pytest.mark.parametrize("n_tris,n_inst,N,ground", [
    (176_000, 3, 1, False),  # one chirp, just above half a million facets
    (125_000, 1, 1, True),   # one facet a lane
    (62_000, 1, 2, True),
    (31_000, 1, 4, True),    # 4 chirps a group, just above the rule
    (20_500, 3, 3, True),    # 4 a group, one of them idle
])
def test_own_walks_decide_alike(n_tris, n_inst, N, ground):
    print(f"case walks n_tris={n_tris} x{n_inst} N={N} ground={ground}", flush=True)
    sc = _scene(n_tris, n_inst)
    few, cfg = _masks(sc, N, ground)
    many, _ = _masks(sc, 12, ground)
    assert few.any()
    assert np.array_equal(few, many[:, :N])
    if not ground:
        facets = np.unique(np.random.default_rng(2).integers(0, sc.n_tris, 80))
        om, amb = oracle.visibility(sc, cfg.array, cfg.waveform, chirps=np.array([0]), facets=facets)
        bits = np.unpackbits(few[0].view(np.uint8), axis=-1, bitorder="little")[:, facets]
        assert not ((bits.astype(bool) != om) & ~amb).any()
