"""GPU tests of the kernels' dispatch edges: each rule that picks a kernel or a
launch shape, at the sizes on both sides of its line, against the oracle."""
import numpy as np
import pytest

from oracle import dp45
from oracle import fields as F
from paper_2406_16064_amd import inputs

from _util import field_err, gpu_params, oracle_params, to_dev

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

PAR = dict(Ms=5.8e5, A=1.5e-11, D=3e-3, Ku=8e5, u=(0.2, -0.3, 1.0), H=(3e4, -2e4, 2e5), alpha=0.3)


@pytest.fixture(scope="module")
def mm():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    from paper_2406_16064_amd import mm as m
    return m


def _m(mesh, seed):
    return inputs.random_unit(*mesh[:3], np.random.default_rng(seed))


@pytest.mark.parametrize("ny", [64, 65, 95, 97])
def test_error_norm_over_many_workgroups_fp64(mm, ny):
    """The step decision gathers one workgroup a row here: up to 64 at the
    instance, beyond that over 32 arrival slots (65 and 97: one slot holds one
    more than the others, 95: one less).  Four attempts of two instances, so
    that each finds the slots as the one before left them; the error norm of
    every attempt against the oracle's."""
    mesh = (16, ny, 1, 2e-9, 2e-9, 2e-9)
    plan = mm.Plan(mesh, "f64", terms=F.ALL_TERMS, max_batch=2)
    gp, op = gpu_params(mm, PAR, F.ALL_TERMS), oracle_params(PAR, F.ALL_TERMS)
    kern = F.DemagKernel(F.Mesh(*mesh))
    f = lambda y: F.llg_rhs(y, F.Mesh(*mesh), op, kern)
    mo = [_m(mesh, 11), _m(mesh, 12)]
    md = to_dev(np.stack(mo), torch.float64)
    st = mm.new_states(2, h=2e-14)
    ost = [dp45.State(h=2e-14), dp45.State(h=2e-14)]
    for _ in range(4):
        plan.rk45_step([gp, gp], md, st)
        for b in range(2):
            mo[b], acc = dp45.step(f, mo[b], ost[b])
            assert bool(st[b].last_accepted) == acc
            assert abs(st[b].last_err - ost[b].last_err) <= 1e-9 * max(1.0, ost[b].last_err)
            assert field_err(md[b].cpu().numpy(), mo[b]) <= 1e-12
