"""z-pass with the columns in registers (192 to 512 points) against the oracle (needs an MI355X).

Every tile variant and both launch forms, in FP32 and FP64, on the grids at the ends of
its plans: 192 (first of its range), 256 and 384 (row plans of 8 and 12 values per
lane); steps with and without a previous right-hand side."""
import functools

import numpy as np
import pytest
import torch

import paper_1506_06513_amd as F
import workloads as W
from oracle import flusi_oracle as O

pytestmark = pytest.mark.gpu

L, NU, DT = 4.0, 0.01, 1e-3


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.name}", flush=True)
    yield
    torch.cuda.synchronize()


@functools.lru_cache(maxsize=1)
def _case(n):
    steps = 2 if n < 384 else 1
    u0 = W.inflow_noise(n, L, seed=9, rms=0.3, kmax=n / 4, mean=(0.5, 0.2, -0.1))
    p = O.Params(n, L, NU, 1e-3)
    ost, _ = O.run(p, u0, steps, O.StepControl(dt_fixed=DT))
    return u0, steps, O.velocity(p, ost)


@pytest.mark.parametrize("n", [192, 256, 384])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_free_flow_matches_the_oracle(n, dtype):
    u0, steps, ou = _case(n)
    norm = np.linalg.norm(ou)
    ref = None
    for z_pass in (0, 1, 2):
        for split in (0, 1):
            P = F.Plan(n, L, NU, 1e-3, dtype)
            P.set_schedule({"z_pass": z_pass, "split_z": split, "y_inverse": z_pass, "y_forward": z_pass})
            st = P.new_state(torch.from_numpy(u0))
            P.step(st, steps, None, dt_fixed=DT, cfl=0.0)
            u = P.velocity(st)
            if ref is None:
                ref = u
                err = np.linalg.norm(u.double().cpu().numpy() - ou) / norm
                assert err <= (1e-11 if dtype == "f64" else 2e-5)
            else:
                assert torch.equal(u, ref), (z_pass, split)
            P.close()
