"""Steps recorded once in a graph and replayed after psdns_set_slot changed the forcing: the slot
table is read by the kernels at replay time, so every replay equals the same steps launched
eagerly, bitwise (the same kernels)."""
import numpy as np
import pytest

import oracle as ora
from tests.gpu_helpers import make_plan, rel_l2, set_params, to_numpy, torch_mod

pytestmark = pytest.mark.gpu

DT = 0.006


def _prm(mode, seed=7):
    kw = dict(nu=0.02, schmidt=(1.0,), mean_grad=((0.0, 1.0, 0.0),), k_force=2.0)
    if mode == "stochastic":
        return ora.Params(forcing_mode="stochastic", stoch_sigma=2.0, stoch_tl=0.5, stoch_seed=seed, **kw)
    if mode == "alvelius":
        return ora.Params(forcing_mode="alvelius", power=0.2, stoch_seed=seed, **kw)
    return ora.Params(power=0.1, **kw)


# (forcing of slot 0, active) of each leg; slot 1 keeps the constant-power forcing
LEGS = [("power", True), ("stochastic", True), ("alvelius", True), ("power", True), ("stochastic", False),
        ("stochastic", True)]


class Run:
    """Two slots on a plan of their own; step() is eager, a replay of the caller's graph, or a replay of
    the plan's."""

    def __init__(self, torch, N, dealias, how, noalloc):
        self.torch, self.how, self.noalloc = torch, how, noalloc
        self.plan = make_plan(N, 1, 64, batch=2, dealias=dealias)
        self.st, self.ws = self.plan.new_state(), self.plan.new_workspace()
        for i in range(2):
            set_params(self.plan, i, _prm("power"))
            self.plan.set_state(self.st, ora.init_field(N, 1, 40 + i, 3.0, 0.5), i)
        self.stream, self.graph = torch.cuda.Stream(), None
        if how == "caller":
            if noalloc:
                self.launch(0)  # the scratch's address, looked up once outside the capture
            torch.cuda.synchronize()
            self.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(self.graph, stream=self.stream):
                self.launch(2)
        elif how == "plan":
            self.plan.set_graph(True)

    def launch(self, n):
        if self.noalloc:
            self.plan.step_noalloc(self.st, DT, n)
        else:
            self.plan.step(self.st, self.ws, DT, n)

    def leg(self, mode, active):
        self.torch.cuda.synchronize()
        set_params(self.plan, 0, _prm(mode), active=active)
        if self.graph is not None:
            self.graph.replay()
        else:
            with self.torch.cuda.stream(self.stream):
                self.launch(2)
        self.torch.cuda.synchronize()
        return [to_numpy(self.plan.get_state(self.st, i)) for i in range(2)]


# 32: the plane pass; 16: the separate passes; 24: the general kernels; 16 with the phase shift
@pytest.mark.parametrize("N,dealias", [(32, 0), (16, 0), (24, 0), (16, 1)])
@pytest.mark.parametrize("how,noalloc", [("caller", False), ("caller", True), ("plan", False)])
def test_replays_follow_the_forcing_of_the_slot_table(N, dealias, how, noalloc):
    torch = torch_mod()
    eager, replay = Run(torch, N, dealias, "eager", noalloc), Run(torch, N, dealias, how, noalloc)
    for k, (mode, active) in enumerate(LEGS):
        a, b = eager.leg(mode, active), replay.leg(mode, active)
        for i in range(2):
            assert np.array_equal(a[i], b[i]), f"leg {k} {mode} active={active} slot {i}: {rel_l2(b[i], a[i]):.2e}"
    if not noalloc:
        assert [r["steps"] for r in replay.plan.read_step_info(replay.ws)] == [10, 12]
    replay.plan.set_graph(False)


def test_forcing_legs_differ_and_match_the_oracle():
    """The legs above do change the field, and an eager stochastic leg is the oracle's."""
    torch = torch_mod()
    run = Run(torch, 32, 0, "eager", False)
    y = to_numpy(run.plan.get_state(run.st, 0))
    got = run.leg("stochastic", True)[0]
    ref = ora.step(y, _prm("stochastic"), DT, 2, stoch_state={"b": {}, "n": 0})
    assert rel_l2(got, ref) < 1e-12
    assert rel_l2(ora.step(y, _prm("power"), DT, 2), ref) > 1e-4
