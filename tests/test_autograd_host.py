"""What the strain loss keeps for its backward pass, and in which order the reverse sweep uses it, on
the CPU: the simulation and the adjoint entry points are stand-ins that count steps (no GPU)."""
import pytest
import torch

from paper_1704_07559_amd import autograd, capi

N = 4


class Counter:
    """A simulation whose state is the number of its steps; a record holds the number of its step."""
    made = []

    def __init__(self, params, rho_u=None):
        self.params, self.level, self.log, self.ctx = params, 0, [], self
        lagged = params.visc_kind in (capi.LBM_VISC_SMAGORINSKY, capi.LBM_VISC_POWERLAW)
        self.save_planes = 3 if params.visc_kind == capi.LBM_VISC_CONST else 10
        self.adjoint_planes = 20 if lagged else 19
        Counter.made.append(self)

    def step(self, n, save=None):
        if save is not None:
            assert save.shape[0] >= n and save.shape[1:] == (self.save_planes, N)
            for i in range(n):
                save[i] = self.level + i
        self.level += n
        self.log.append(("record" if save is not None else "step", n))

    def save_state(self):
        self.log.append(("state", self.level))
        return torch.tensor(self.level)

    def load_state(self, state):
        self.level = int(state)

    def close(self):
        pass


@pytest.fixture
def counter(monkeypatch):
    def adjoint_steps(sim, n, rec, lam, lam2, gF):
        for i in reversed(range(n)):
            sim.reverse.append(int(rec[i, 0, 0]))

    def seed(sim, lam, gF):
        sim.reverse = []
        return 1.0

    monkeypatch.setattr(autograd, "LBM", Counter)
    monkeypatch.setattr(capi, "lbm_adjoint_steps", adjoint_steps)
    monkeypatch.setattr(capi, "lbm_strain_loss_seed", seed)
    monkeypatch.setattr(capi, "lbm_init_adjoint", lambda sim, rho_u, lam, gu: gu.zero_())
    Counter.made = []
    return Counter


def _problem(nsteps, every, visc=capi.LBM_VISC_CONST, **kw):
    return autograd.StrainLossProblem(capi.Params(nx=N, ny=1, nz=1, visc_kind=visc), nsteps, every, **kw)


def _inputs(**kw):
    return torch.zeros(3, 1, 1, N, **kw), torch.zeros(3, 1, 1, N, **kw)


@pytest.mark.parametrize("record_all", [False, True])
@pytest.mark.parametrize("how", ["no_grad", "inference", "no requires_grad"])
def test_an_evaluation_without_a_backward_pass_keeps_nothing(counter, how, record_all):
    prob = _problem(60, 50, capi.LBM_VISC_SMAGORINSKY, record_all=record_all)
    if how == "no requires_grad":
        J = autograd.strain_loss(*_inputs(), prob)
    else:
        u0, F = _inputs(requires_grad=True)
        with torch.no_grad() if how == "no_grad" else torch.inference_mode():
            J = autograd.strain_loss(u0, F, prob)
    sim, = counter.made
    assert not J.requires_grad and sim.level == 60
    assert {what for what, _ in sim.log} == {"step"}


@pytest.mark.parametrize("nsteps,every", [(0, 5), (1, 1), (5, 1), (7, 50), (20, 10), (20, 7), (21, 7), (24, 24)])
@pytest.mark.parametrize("visc", [capi.LBM_VISC_CONST, capi.LBM_VISC_SMAGORINSKY, capi.LBM_VISC_SMAGORINSKY_IMPLICIT])
@pytest.mark.parametrize("record_all", [False, True])
@pytest.mark.parametrize("entry", ["strain_loss", "apply"])
def test_the_reverse_sweep_takes_every_step_once_in_reverse(counter, entry, record_all, visc, nsteps, every):
    u0, F = _inputs(requires_grad=True)
    prob = _problem(nsteps, every, visc, record_all=record_all)
    J = autograd.strain_loss(u0, F, prob) if entry == "strain_loss" else autograd.StrainLoss.apply(u0, F, prob)
    sim, = counter.made
    assert sim.level == nsteps
    J.backward()
    assert sim.reverse == list(reversed(range(nsteps)))
    assert u0.grad is not None and F.grad is not None


@pytest.mark.parametrize("visc", [capi.LBM_VISC_CONST, capi.LBM_VISC_SMAGORINSKY, capi.LBM_VISC_SMAGORINSKY_IMPLICIT])
@pytest.mark.parametrize("nsteps,every", [(50, 50), (60, 50), (500, 50), (20, 10), (24, 24), (12, 12), (13, 13), (3, 3),
                                          (4, 4), (1, 1)])
def test_a_loss_holds_no_more_in_records_than_in_states(counter, nsteps, every, visc):
    """Between the forward and the backward pass, where several losses may be alive at once."""
    u0, F = _inputs(requires_grad=True)
    J = autograd.strain_loss(u0, F, _problem(nsteps, every, visc))
    sim, = counter.made
    states = 2 + sum(what == "state" for what, _ in sim.log)
    recorded = sum(n for what, n in sim.log if what == "record")
    assert recorded * sim.save_planes <= 19 * states
    last = nsteps - every * ((nsteps - 1) // every)
    # the last segment is recorded whole, in place of its checkpoint, or not at all
    assert recorded in (0, last) and states == 2 + -(-nsteps // every) - (recorded > 0)
    assert (recorded > 0) == (last * sim.save_planes <= 19 * (2 + (nsteps - 1) // every))
    J.backward()
    assert sim.reverse == list(reversed(range(nsteps)))
