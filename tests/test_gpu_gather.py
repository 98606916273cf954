"""The NUFFT adjoint's element terms (in LDS per element, a Tx element's kept for its Rx channels)
at element counts where they can go wrong, against the vector-unit adjoint on the same gradient
input. Tolerance: 1e-4 relative L2, that of the FP32 sums in different orders."""
import numpy as np
import pytest

import scenes
from scenes import RadarArray

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,Q,M", [(1, 1, 96), (64, 1, 64), (1, 64, 64), (5, 13, 96),
                                   (64, 64, 32), (12, 16, 256)])
def test_gather_equals_vector_adjoint(P, Q, M):
    import torch
    from paper_2208_10939_amd.pipeline import Simulator
    print(f"case gather P={P} Q={Q} M={M}", flush=True)
    cfg = scenes.small_single(n_samples=M, n_chirps=2, n_tris=300)
    sc, wf = cfg.scenes[0], cfg.waveform
    tx, rx = np.array(cfg.array.tx), np.array(cfg.array.rx)
    arr = RadarArray(tx=np.resize(tx, (P, 3)) + [[0, 0, 0.001 * k] for k in range(P)],
                     rx=np.resize(rx, (Q, 3)) + [[0, 0, 0.001 * k] for k in range(Q)])
    sim = Simulator([sc], wf, arr)
    mask = sim.mask_buffer()
    echo = sim.synthesize(mask=mask, kernel=1)
    rng = np.random.default_rng(P * 100 + Q)
    g = rng.normal(size=echo.shape) + 1j * rng.normal(size=echo.shape)
    ge = torch.from_numpy(g.astype(np.complex64)).cuda()
    out = {}
    for kernel in (1, 3):
        gv = [torch.zeros((m.verts.shape[0], 3), dtype=torch.float32, device="cuda")
              for m in sc.meshes]
        gvel = torch.zeros((len(sc.instances), 3), dtype=torch.float64, device="cuda")
        sim.ctx.set_backward_kernel(kernel)
        sim.ctx.backward(sim.scene_ids[0], ge, mask, gv, gvel)
        out[kernel] = (np.concatenate([x.cpu().numpy().ravel() for x in gv]).astype(np.float64),
                       gvel.cpu().numpy().ravel())
    for a, b in zip(out[3], out[1]):
        assert np.linalg.norm(b) > 0
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        print(f"  rel_l2={err:.2e}", flush=True)
        assert err <= 1e-4
