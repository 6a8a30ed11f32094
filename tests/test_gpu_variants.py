"""Every tile variant and both z-pass launch forms on the sizes and options whose
kernels no smaller case reaches (needs an MI355X).

Steps with and without a previous right-hand side in both launch forms (the first
call takes three steps, the second one), against the FP64 solver of the performance
cases (plain torch operations), and bit for bit against the default schedule and
against the same steps in other calls.  192 to
512 points: rows and columns in registers, with the sponge the z-pass in LDS tiles;
below: the LDS tiles with their threads per column, and Runge-Kutta steps."""
import pytest
import torch

from perf import cases

pytestmark = pytest.mark.gpu

KEYS = ("y_inverse", "x_pass", "y_forward", "z_pass", "split_z")


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.name}", flush=True)
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


CASES = [
    # n, dtype, body, sponge, integrator
    (16, "f32", "sphere", False, "ab2"), (32, "f64", "sphere", True, "ab2"), (48, "f64", "insect", False, "rk4"),
    (64, "f32", "sphere", True, "rk4"), (96, "f64", "insect", True, "ab2"), (128, "f32", "insect", True, "ab2"),
    (128, "f64", "sphere", False, "rk4"),
    (192, "f32", "insect", True, "ab2"), (192, "f64", "insect", True, "ab2"), (192, "f64", "insect", False, "ab2"),
    (192, "f32", "sphere", False, "rk4"), (256, "f32", "insect", True, "ab2"), (256, "f64", "insect", True, "ab2"),
    (256, "f64", "sphere", True, "rk4"), (384, "f32", "insect", False, "ab2"), (384, "f64", "insect", False, "ab2"),
    (384, "f64", "sphere", True, "ab2"), (512, "f32", "insect", False, "ab2"), (512, "f64", "insect", False, "ab2"),
    (512, "f32", "sphere", True, "ab2"),
]


@pytest.mark.parametrize("n,dtype,body,sponge,integrator", CASES)
def test_variants_agree_and_match_64_bits(n, dtype, body, sponge, integrator):
    case = dict(kind="solve", nx=n, n=n, dtype=dtype, body=body, steps=4, integrator=integrator, sponge=sponge,
                flow="inflow")
    ref = None
    for sched, calls in [(None, (3, 1)), (None, (1, 1, 2)), (None, (4,))] + \
            [((v, v, v, v, split), (3, 1)) for v in (0, 1, 2) for split in (0, 1)]:
        s = cases.prepare(case, 5)
        if sched is not None:
            s["plan"].set_schedule(dict(zip(KEYS, sched)))
        for k in calls:
            s["plan"].step(s["st"], k, s["p"]["insect"], **s["p"]["controls"])
        u = s["plan"].velocity(s["st"])
        s["plan"].close()
        if ref is None:
            ref = u
        else:
            assert torch.equal(u, ref), (sched, calls)
    ex = cases.exact(case, 5)["velocity"]
    err = float((ref.double() - ex).norm() / ex.norm())
    assert err <= (1e-11 if dtype == "f64" else 2e-5), err


@pytest.mark.parametrize("graph", [False, True])
def test_mixed_members_at_192_equal_their_solo_runs(graph):
    # one size group with and without the sponge (its members' steps are two z launches),
    # and one of Runge-Kutta members
    import paper_1506_06513_amd as fl
    kinds = [("sphere", True, "ab2"), ("insect", False, "ab2"), ("insect", True, "ab2"), ("sphere", False, "rk4")]
    runs = [[cases.prepare(dict(kind="solve", nx=192, n=192, dtype="f32", body=b, steps=4, integrator=i, sponge=sp,
                                flow="inflow"), 7 + j) for j, (b, sp, i) in enumerate(kinds)] for _ in range(2)]
    ens = fl.Ensemble("f32")
    for s in runs[0]:
        ens.add(s["plan"], s["st"], s["p"]["insect"], **s["p"]["controls"])
    for _ in range(2):
        ens.step(2, graph=graph)
        torch.cuda.synchronize()
    for a, b in zip(*runs):
        b["plan"].step(b["st"], 4, b["p"]["insect"], **b["p"]["controls"])
        assert torch.equal(a["plan"].velocity(a["st"]), b["plan"].velocity(b["st"]))
        assert a["plan"].time(a["st"]) == b["plan"].time(b["st"])
    ens.close()
