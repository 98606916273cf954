"""Visibility by waves that walk a BVH together, over the launch shapes (chirps a group, facets a
workgroup, threads) that sizes choose, against the FP64 oracle on sampled chirps and facets:
facet counts off the bytes and words of the mask, chirp counts around a wave, several instances,
the ground's four path types. Bits may differ only where the oracle calls them ambiguous; the
padding bits of a mask that held ones come out zero."""
import numpy as np
import pytest

import oracle
import scenes
from oracle import bounce
from scenes import Instance, Scene

pytestmark = pytest.mark.gpu


def _scene(n_tris, n_inst):
    car = scenes.vehicle_mesh("car", n_tris)
    return Scene([car], [Instance(0, scenes.yaw_matrix(1.5 - 0.4 * k),
                                  np.array([3.0 - 2.5 * k, 14.0 + 3.0 * k, 0.0]),
                                  np.array([0.3, -6.0 + 9.0 * k, 0.0])) for k in range(n_inst)])


@pytest.mark.parametrize("n_tris,n_inst,N,ground", [
    (300, 1, 1, False),       # one facet a wave, 8 a workgroup of 512
    (700, 3, 33, False),
    (700, 2, 65, True),
    (9500, 2, 4, False),      # 32 chirps a group
    (9500, 1, 70, False),     # 64 chirps a group, 8 facets a workgroup
    (9500, 1, 5, True),
    (50_000, 3, 4, False),    # 32 chirps, 8 facets: just too few facets for packed waves
    (50_000, 3, 40, False),   # 64 chirps, 16 facets
    (100_000, 3, 4, False),   # 4 chirps a group, 16 facets a wave, 64 a workgroup
    (100_000, 3, 70, False),  # 64 chirps, 32 facets
    (180_000, 3, 3, True),    # 4 chirps, four types
])
def test_masks_against_oracle(n_tris, n_inst, N, ground):
    from paper_2208_10939_amd.pipeline import Simulator
    print(f"case vis n_tris={n_tris} x{n_inst} N={N} ground={ground}", flush=True)
    cfg = scenes.small_single(n_samples=16, n_chirps=N, n_tris=300)
    wf, arr, sc = cfg.waveform, cfg.array, _scene(n_tris, n_inst)
    sim = Simulator([sc], wf, arr)
    if ground:
        sim.set_ground(True, -0.5, -0.7)
    mask = sim.mask_buffer()
    mask.fill_(-1)
    sim.synthesize(mask=mask, kernel=3)
    F, words, types = sim.n_facets[0], sim.mask_words[0], 4 if ground else 1
    bits = np.unpackbits(mask.cpu().numpy().view(np.uint8).reshape(types, N, 4 * words), axis=-1,
                         bitorder="little")
    assert not bits[..., F:].any()
    chirps = np.unique([0, N // 2, N - 1])
    rng = np.random.default_rng(1)
    facets = np.unique(np.concatenate([np.arange(min(F, 40)), np.arange(max(0, F - 40), F),
                                       rng.integers(0, F, 60)]))
    if ground and F < 4000:
        om, amb = bounce.visibility_bounce(sc, arr, wf, -0.5, chirps=chirps)
        om, amb = om[..., facets], amb[..., facets]
    else:  # type 0, both ends direct, is the single path
        om, amb = oracle.visibility(sc, arr, wf, chirps=chirps, facets=facets)
        om, amb, bits = om[None], amb[None], bits[:1]
    bad = (bits[:, chirps][..., facets].astype(bool) != om) & ~amb
    assert not bad.any(), f"{bad.sum()} unambiguous mask mismatches"
