"""Row kernel of the x-pass against the oracle at the edges of its dispatch (needs an MI355X).

Grids from the smallest (one wavefront with rows per workgroup) past the change from
shared to per-wavefront point lists and from single rows to row pairs; bodies that
fill the lists, leave them empty, reach over the box's faces or overlap."""
import numpy as np
import pytest
import torch

import paper_1506_06513_amd as F
import workloads as W
from oracle import flusi_oracle as O

pytestmark = pytest.mark.gpu

L = 4.0


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.name}", flush=True)
    yield
    torch.cuda.synchronize()


def _body(kind, n):
    sphere = dict(body="sphere", smooth="cos", c_smth=1.0)
    insect = W.model_insect(n, L)
    return {
        "full": dict(sphere, x_cntr=(L / 2,) * 3, radius=L),             # every point in the lists
        "corner": dict(sphere, x_cntr=(0.0, 0.1, L), radius=0.3 * L, smooth="tanh"),
        "outside": dict(sphere, x_cntr=(-3 * L, 0.0, 0.0), radius=0.5),  # no point
        "insect": insect,
        "headed": dict(insect, head_x=(0.5, 0.0, 0.0), head_r=0.2, eye_x=(0.6, 0.1, 0.05), eye_r=0.1),
        "rect": dict(insect, wing_shape="rectangle", rect_a=0.1, rect_tip=1.0, rect_b=0.1, rect_B=0.4,
                     psi=0.3, gamma=0.2, psi_dot=0.5),
        "fourier": dict(insect, wing_shape="fourier", wing_fa=(0.7, 0.1, 0.02), wing_fb=(0.0, 0.05, 0.0),
                        wing_c=(0.05, 0.5), wings=True, body="none"),
    }[kind]


CASES = [
    # n, nx, dtype, body, sponge, wall, x_pass
    (16, 16, "f64", "full", False, False, 0), (16, 16, "f32", "insect", True, False, 1),
    (24, 24, "f32", "full", False, True, 0), (24, 24, "f64", "headed", False, False, 2),
    (32, 32, "f64", "corner", True, False, 0), (32, 32, "f32", "rect", False, False, 1),
    (32, 48, "f32", "insect", False, True, 0), (32, 64, "f64", "fourier", False, False, 0),
    (48, 48, "f64", "insect", True, True, 2), (48, 48, "f32", "headed", False, False, 0),
    (64, 64, "f32", "full", False, False, 0), (64, 64, "f64", "rect", False, True, 1),
    (96, 96, "f64", "insect", True, False, 0), (96, 96, "f32", "fourier", False, False, 2),
    (128, 128, "f32", "corner", False, False, 0), (128, 128, "f64", "outside", False, False, 0),
    (128, 192, "f32", "headed", True, False, 0), (128, 192, "f64", "full", False, False, 0),
    (192, 192, "f32", "insect", False, False, 1),
]


@pytest.mark.parametrize("n,nx,dtype,body,sponge,wall,x_pass", CASES)
def test_steps_match_the_oracle(n, nx, dtype, body, sponge, wall, x_pass):
    nu, eta, steps = 1 / 150.0, 5e-4, 3
    ins = _body(body, n)
    opt = {}
    P = F.Plan(n, L, nu, eta, dtype, nx=nx)
    if sponge:
        P.set_sponge(0.1, (0.5, 0.0, 0.0))
        opt.update(c_sp=0.1, sponge=(0.5, 0.0, 0.0))
    if wall:
        P.set_walls((0.0, 0.0, 0.4), (0.2, 0.0, 0.0))
        opt.update(wall=(0.0, 0.0, 0.4), u_wall=(0.2, 0.0, 0.0))
    P.set_schedule({"x_pass": x_pass})
    u0 = W.inflow_noise(n, L, seed=4, rms=5e-2, kmax=min(6.0, n / 4), nx=nx)
    p = O.Params(n, L, nu, eta, **(dict(nx=nx, Lx=L * nx / n) if nx != n else {}), **opt)
    ost, oh = O.run(p, u0, steps, O.StepControl(cfl=0.1), O.Insect.from_dict(ins))
    st = P.new_state(torch.from_numpy(u0))
    h = P.step(st, steps, ins, cfl=0.1, history=True).cpu().numpy()
    u, ou = P.velocity(st).double().cpu().numpy(), O.velocity(p, ost)
    assert np.linalg.norm(u - ou) <= (1e-11 if dtype == "f64" else 2e-5) * np.linalg.norm(ou)
    f = np.array([np.concatenate([np.concatenate([d["F"][c], d["M"][c]]) for c in range(3)]) for d in oh])
    assert np.max(np.abs(h[:, 4:22] - f)) <= (1e-9 if dtype == "f64" else 1e-3) * np.max(np.abs(f))
    if body == "outside":
        assert np.all(h[:, 4:22] == 0.0)
