"""One plan stepping several states in turn (needs an MI355X).

Between two calls for a state the plan's launch record is another state's (stepped,
initialized or autotuned on the same plan); each state must go on as if it had the
plan to itself, bit for bit.  Calls of one step leave the second time slot current,
so that a prologue that worked on the other state would show."""
import pytest
import torch

import paper_1506_06513_amd as F
import workloads as W

pytestmark = pytest.mark.gpu

N, L, NU, ETA = 32, 4.0, 0.01, 1e-3
CTL = dict(cfl=0.1)


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.name}", flush=True)
    yield
    torch.cuda.synchronize()


def _u0(seed):
    return torch.from_numpy(W.inflow_noise(N, L, seed=seed, rms=0.1, kmax=6.0))


def _solo(seed, body, dtype, calls):
    P = F.Plan(N, L, NU, ETA, dtype)
    st = P.new_state(_u0(seed))
    for k in calls:
        P.step(st, k, body, **CTL)
    return P.uhat(st), P.time(st)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("body", [None, "sphere", "insect"])
@pytest.mark.parametrize("between", ["step", "init", "autotune"])
def test_states_of_one_plan_do_not_mix(between, body, dtype):
    ins = {None: None, "sphere": W.sphere_body(L), "insect": W.model_insect(N, L)}[body]
    P = F.Plan(N, L, NU, ETA, dtype)
    a, b = P.new_state(_u0(1)), P.new_state(_u0(2))
    ca, cb = [], []
    for k in (1, 2, 1, 3, 1):
        P.step(a, k, ins, **CTL)
        ca.append(k)
        if between == "step":
            P.step(b, 1, ins, **CTL)
            cb.append(1)
        elif between == "init":
            P.new_state(_u0(3))
        else:
            P.autotune(a, ins, reps=1, **CTL)
    for st, seed, calls in ((a, 1, ca), (b, 2, cb)):
        u, t = _solo(seed, ins, dtype, calls)
        assert torch.equal(P.uhat(st), u)
        assert P.time(st) == t


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("body", [None, "sphere", "insect"])
def test_captured_step_replays_among_steps_of_another_state(body, dtype):
    # every replay brings its own launch record, whatever the plan was used for since
    ins = {None: None, "sphere": W.sphere_body(L), "insect": W.model_insect(N, L)}[body]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        P = F.Plan(N, L, NU, ETA, dtype)
        a, b = P.new_state(_u0(1)), P.new_state(_u0(2))
        P.step(a, 1, ins, **CTL)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            P.step(a, 3, ins, **CTL)
        for _ in range(3):
            g.replay()
            P.step(b, 1, ins, **CTL)
            s.synchronize()
        u, t, ub = P.uhat(a), P.time(a), P.uhat(b)
    torch.cuda.synchronize()
    ua, ta = _solo(1, ins, dtype, (1, 3, 3, 3))
    assert torch.equal(u, ua) and t == ta
    assert torch.equal(ub, _solo(2, ins, dtype, (1, 1, 1))[0])
