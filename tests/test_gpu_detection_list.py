"""The detection list on both sides of the count that sets the cells a thread takes, with steps that
end on their last cell and ones that do not, and every cell detected: row-major, first max_points."""
import numpy as np
import pytest

from test_gpu_cube_edges import _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,cubes,max_points,scale", [
    (16, 32, 40, 64, 0.01),    # every cell, more than the points
    (128, 128, 2, 2000, 1.2),  # 16384 cells: one step of 16 a thread
    (128, 256, 1, 900, 1.2),   # 32768: two
    (81, 432, 3, 700, 1.2),    # 34992: 64 a thread, the last threads' cells past the end
])
def test_list(N, M, cubes, max_points, scale):
    import torch
    print(f"case list N={N} M={M} cubes={cubes} max_points={max_points}", flush=True)
    sim = _sim(N, M, 1, 4)
    g = torch.Generator("cuda").manual_seed(N + M)
    y = torch.randn((cubes, 4, N, M), dtype=torch.complex64, device="cuda", generator=g)
    rdm = y.real ** 2 + y.imag ** 2
    pts, cnt, det, _ = sim.detect(rdm, y, max_points=max_points, guard=(1, 1), train=(2, 2),
                                  scale=scale, want_maps=True)
    for c, rec in enumerate(sim.points_numpy(pts, cnt)):
        cells = np.argwhere(det[c].cpu().numpy())
        assert int(cnt[c]) == len(cells) > max_points
        assert np.array_equal(np.stack([rec["row"], rec["bin"]], 1), cells[:max_points])
