"""RadarRDM's backward loads its forward's geometry again where any vertices or motion were set
after the forward loaded its own, also while the forward was still running (another thread's
forward on the same simulator: the library's calls release the interpreter lock). The library is
replaced by one that records what is set; no GPU."""
from types import SimpleNamespace

import pytest
import torch

from paper_2208_10939_amd.autograd import RadarRDM


class _Library:
    """A context of one scene with one mesh and one instance; `during` runs in the forward's
    range-Doppler call."""

    def __init__(self):
        self.geometry_changes = 0
        self.scene_meshes = {0: [0]}
        self.verts = self.motion = self.used = None
        self.during = lambda: None

    def update_mesh(self, mesh, verts):
        self.geometry_changes += 1
        self.verts = verts.copy()

    def set_instance_motion(self, scene, inst, pos0, vel):
        self.geometry_changes += 1
        self.motion = vel.copy()

    def set_backward_intra_chirp(self, enable):
        pass

    def rdm_backward(self, g, y, grad_echo):
        grad_echo.zero_()

    def backward(self, scene, grad_echo, mask, grad_verts, grad_vel):
        self.used = (self.verts, self.motion)


def _simulator():
    lib = _Library()

    def form_rdm(echo, want_y):
        lib.during()
        return torch.ones(1, 1, 2, 2), echo

    return SimpleNamespace(ctx=lib, scene_ids=[0], inst_pos0=[[0.0]], intra_chirp=False,
                           mask_buffer=lambda which: torch.zeros(1, dtype=torch.int32),
                           synthesize=lambda *a, **k: torch.zeros(1, 1, 2, 2, dtype=torch.complex64),
                           form_rdm=form_rdm)


@pytest.mark.parametrize("when", ["never", "during", "after"])
def test_backward_uses_forward_geometry(when, monkeypatch):
    monkeypatch.setattr(torch.cuda, "synchronize", lambda device=None: None)
    sim = _simulator()
    verts = torch.arange(9.0).reshape(3, 3).requires_grad_(True)
    vel = torch.ones(1, 3, dtype=torch.float64)

    def other():
        sim.ctx.update_mesh(0, -verts.detach().numpy())
        sim.ctx.set_instance_motion(0, 0, None, -vel[0].numpy())

    if when == "during":
        sim.ctx.during = other
    rdm = RadarRDM.apply(sim, 0, vel, verts)
    if when == "after":
        other()
    loads = sim.ctx.geometry_changes
    rdm.sum().backward()
    assert (sim.ctx.used[0] == verts.detach().numpy()).all()
    assert (sim.ctx.used[1] == vel[0].numpy()).all()
    assert (sim.ctx.geometry_changes == loads) == (when == "never")
