"""The register-pass transforms and the detection list at their edges (Section 3.3): every pair
of stages a length 2^a 3^b can be made of, column tiles that the map does not fill, maps whose
cells do not start on 16 bytes, and more detections than points.

Tolerance of the transforms: FP32 rounding of at most 12 stages, a few parts in 1e7 of the
map's RMS (1e-6); FP64 1e-14."""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sim(N, M, P=1, Q=3):
    from paper_2208_10939_amd.pipeline import Simulator
    wf = SimpleNamespace(f0=77e9, slope=12.5e12, fs=5.12e6, chirp_period=M / 5.12e6 + 1e-5,
                         n_samples=M, n_chirps=N)
    h = 0.5 * 299_792_458.0 / (wf.f0 + 0.5 * M * wf.slope / wf.fs)
    at = np.array([0.0, 0.0, 6.0])
    tx = at + np.array([[16 * h * i, 0, 0] for i in range(P)])
    rx = at + np.array([[h * i, 0, 0] for i in range(Q)])
    return Simulator([], wf, SimpleNamespace(tx=tx, rx=rx))


# (4,4) (4,2) (4,3) (4) (2,3) (2) (3,3) (3) as first, middle and last pass
@pytest.mark.parametrize("N,M", [(2, 3), (4, 6), (8, 9), (12, 16), (18, 27), (24, 32), (48, 54),
                                 (64, 81), (96, 128), (144, 256), (162, 243), (192, 384),
                                 (288, 512), (36, 1024), (1024, 36), (2187, 4), (6, 2592)])
@pytest.mark.parametrize("precision", [0, 1])
def test_transforms_against_numpy(N, M, precision):
    import torch
    print(f"case transforms N={N} M={M} precision={precision}", flush=True)
    sim = _sim(N, M)
    rng = np.random.default_rng(N * 5000 + M)
    H = rng.standard_normal((2, 3, N, M)) + 1j * rng.standard_normal((2, 3, N, M))
    H = H.astype(np.complex128 if precision else np.complex64)
    rdm, y = sim.form_rdm(torch.from_numpy(H).cuda(), precision=precision, want_y=True)
    want = np.fft.fft(np.fft.fft(np.conj(H.astype(np.complex128)), axis=-1), axis=-2)
    want = np.roll(want, N // 2, axis=-2)
    tol = 1e-14 if precision else 1e-6
    rms = np.sqrt(np.mean(np.abs(want) ** 2))
    assert np.sqrt(np.mean(np.abs(y.cpu().numpy() - want) ** 2)) <= tol * rms
    power = np.abs(want) ** 2
    assert np.sqrt(np.mean((rdm.cpu().numpy() - power) ** 2)) <= 4 * tol * np.sqrt(np.mean(power ** 2))


@pytest.mark.parametrize("N,M,cubes,max_points", [(81, 81, 3, 300), (64, 48, 2, 4000),
                                                  (256, 512, 1, 500), (24, 27, 2, 1)])
def test_detection_list_follows_the_map(N, M, cubes, max_points):
    import torch
    print(f"case detection list N={N} M={M} cubes={cubes} max_points={max_points}", flush=True)
    sim = _sim(N, M, 1, 4)
    g = torch.Generator("cuda").manual_seed(N * M)
    y = torch.randn((cubes, 4, N, M), dtype=torch.complex64, device="cuda", generator=g)
    rdm = y.real ** 2 + y.imag ** 2
    pts, cnt, det, _ = sim.detect(rdm, y, max_points=max_points, guard=(1, 1), train=(2, 2),
                                  scale=1.4, want_maps=True)
    for c, rec in enumerate(sim.points_numpy(pts, cnt)):
        cells = np.argwhere(det[c].cpu().numpy())
        assert int(cnt[c]) == len(cells) > 0
        assert np.array_equal(np.stack([rec["row"], rec["bin"]], 1), cells[:max_points])
