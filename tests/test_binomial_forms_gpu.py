"""The binomial payload's two GPU forms, one wave per group and one lane per
call: tree depths around each form's merges, blocks of levels and its border
between registers and LDS, ragged last tiles and packages, and the borders of
the rule that picks the form. Prices equal the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import paper_1805_02755_amd as ce
from paper_1805_02755_amd import synth
from oracle import oracle as O

from gpu_util import BOTH, DEV, check_trace

pytestmark = pytest.mark.gpu
SIGMA, RATE, T, X = 0.3, 0.05, 1.0, 100.0


@pytest.fixture(scope="module")
def eng():
    e = ce.Engine()
    yield e
    e.close()


def problem(n_groups, steps):
    spots = synth.binomial_spots(n_groups, seed=n_groups + steps)
    f, pu, pd = ce.ce_binomial_table(steps, SIGMA, RATE, T)
    return spots, f, ce.ce_binomial_params(n_groups, steps, X, pu, pd)


def reference(spots, steps):
    fo, puo, pdo = O.binomial_table(steps, SIGMA, RATE, T)
    return O.binomial(spots, X, steps, fo, puo, pdo)


def engine_run(eng, spots, f, prm, devs, sched):
    n, steps = spots.shape[0], prm.steps
    s_d, f_d = torch.from_numpy(spots).to(DEV), torch.from_numpy(f).to(DEV)
    out = torch.full((n, 4), float("nan"), device=DEV)
    torch.cuda.synchronize()
    eng.use(devs, 0, 0)
    eng.work_items([(steps + 1) * n], [steps + 1])
    eng.scheduler(**sched)
    eng.program_kernel(ce.CE_KERNEL_BINOMIAL, prm)
    eng.program_out_pattern(1, steps + 1)
    eng.program_in(0, host=spots, dev=s_d, nbytes=spots.nbytes)
    eng.program_in(1, host=f, dev=f_d, nbytes=f.nbytes)
    eng.program_out(0, dev=out, nbytes=out.numel() * 4)
    eng.run()
    check_trace(eng.trace(), n, eng.stats().n_devices)
    return out.cpu().numpy()


def same(a, b):
    return np.array_equal(np.ascontiguousarray(a).view(np.uint32), np.ascontiguousarray(b).view(np.uint32))


def test_depths_call_form(eng):
    for steps in (1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 175, 176, 190, 191, 192, 193, 207, 208, 209, 223, 224, 239,
                  240, 254, 255):
        n = 16384 + 37
        spots, f, prm = problem(n, steps)
        ins = [torch.from_numpy(spots).to(DEV), torch.from_numpy(f).to(DEV)]
        out = torch.full((n, 4), float("nan"), device=DEV)
        torch.cuda.synchronize()
        ce.ce_bare_run(ce.CE_KERNEL_BINOMIAL, prm, ins, out)
        assert same(out.cpu().numpy(), reference(spots, steps)), steps


def test_depths_group_form(eng):
    for steps in (1, 2, 3, 4, 5, 31, 61, 62, 63, 64, 65, 125, 126, 127, 128, 129, 253, 255):
        spots, f, prm = problem(131, steps)
        out = engine_run(eng, spots, f, prm, ce.CE_DEV_GPU, dict(kind=ce.CE_SCHED_STATIC))
        assert same(out, reference(spots, steps)), steps


@pytest.mark.parametrize("n", [16383, 16384, 20001])
def test_schedules_on_both_sides_of_the_rule(eng, n):
    steps = 60
    spots, f, prm = problem(n, steps)
    ref = reference(spots, steps)
    for sched in (dict(kind=ce.CE_SCHED_STATIC, props=[0.9]), dict(kind=ce.CE_SCHED_STATIC, props=[0.9], n_packages=30),
                  dict(kind=ce.CE_SCHED_STATIC, props=[0.5], n_packages=100),
                  dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=511),
                  dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=513),
                  dict(kind=ce.CE_SCHED_HGUIDED, power=[40, 1], k=2),
                  dict(kind=ce.CE_SCHED_HGUIDED, power=[40, 1], k=2, min_granules=[600, 1]),
                  dict(kind=ce.CE_SCHED_HGUIDED, power=[40, 1], k=2, min_granules=[8, 1])):
        assert same(engine_run(eng, spots, f, prm, BOTH, sched), ref), (n, sched)


@pytest.mark.parametrize("pu,pd", [(1.5, -0.5), (-0.25, 1.25), (0.5, 0.5), (1e-20, 1.0), (1e-3, 1e-3)])
def test_any_weights(pu, pd):
    """Negative weights, underflow to denormals and zeros: the same bits in
    both forms as in the oracle."""
    for n, steps in ((200, 255), (16384, 255)):
        spots, f, prm = problem(n, steps)
        prm = ce.ce_binomial_params(n, steps, X, pu, pd)
        ins = [torch.from_numpy(spots).to(DEV), torch.from_numpy(f).to(DEV)]
        out = torch.full((n, 4), float("nan"), device=DEV)
        torch.cuda.synchronize()
        ce.ce_bare_run(ce.CE_KERNEL_BINOMIAL, prm, ins, out)
        at = np.arange(0, n, max(1, n // 200))
        ref = O.binomial(np.ascontiguousarray(spots[at]), X, steps, f, np.float32(pu), np.float32(pd))
        assert same(out.cpu().numpy()[at], ref), (n, pu, pd)
