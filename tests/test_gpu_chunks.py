"""The chunk lengths the library chooses itself (set_tile_rows 0) against one
chunk over the whole slow dimension: the same bits, at sizes where the rules
pick few planes or rows, one chunk, or a ragged last one."""
import pytest
import torch

from paper_1407_1309_amd import mpdata, synth
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu
FCT, IGA, TOT = mpdata.OPT_FCT, mpdata.OPT_IGA, mpdata.OPT_TOT


def _steps(shape, dtype, opts, bc, n_iters, g, rows, seed=7, n_steps=2):
    gen = synth.rng(seed)
    c = synth.random_advector(shape, 0.3, gen)
    if bc == 0:
        c = synth.periodic_fix(c)
    psi = synth.blob_field(shape, 4, (2.0, 6.0), "uniform", gen, periodic=False) + 0.05
    G = gen.uniform(0.7, 1.3, size=shape) if g else None
    plan = mpdata.Plan(shape, dtype=dtype, n_iters=n_iters, opts=opts, bc=bc, has_g=g)
    plan.set_tile_rows(rows)
    p = dev(psi, dtype)
    plan.step(p, [dev(x, dtype) for x in c], g=dev(G, dtype), n_steps=n_steps)
    torch.cuda.synchronize()
    return p.cpu()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("shape,opts,bc,g", [
    ((3, 16, 32), FCT, 0, False), ((4, 17, 33), TOT | IGA, 1, True),
    ((5, 20, 70), FCT, 1, False), ((41, 16, 32), 0, 0, False),
    ((130, 30, 31), FCT | IGA, 0, True), ((35, 150, 140), FCT, 1, False),
    ((23, 260, 300), TOT | IGA, 0, True)])
def test_step3d_own_chunks(shape, opts, bc, g, dtype):
    own = _steps(shape, dtype, opts, bc, 2, g, 0)
    assert torch.equal(own, _steps(shape, dtype, opts, bc, 2, g, shape[0]))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("shape,opts,bc,n_iters,g", [
    ((3, 3), FCT, 0, 2, False), ((5, 70), FCT, 0, 3, False), ((61, 77), 0, 0, 2, False),
    ((61, 77), FCT, 0, 4, False), ((700, 130), FCT, 0, 3, False),
    ((1, 1), FCT | IGA, 1, 2, False), ((61, 77), FCT | TOT, 1, 3, True),
    ((700, 130), FCT | IGA, 1, 2, False), ((33, 900), TOT, 1, 2, True)])
def test_2d_own_chunks(shape, opts, bc, n_iters, g, dtype):
    own = _steps(shape, dtype, opts, bc, n_iters, g, 0)
    assert torch.equal(own, _steps(shape, dtype, opts, bc, n_iters, g, shape[0]))


@pytest.mark.parametrize("shape", [(6, 40), (61, 77), (500, 130)])
def test_step_diag_with_own_chunks(shape):
    """The partials of the step's own diagnostics fit their buffer."""
    gen = synth.rng(11)
    psi = gen.uniform(0.1, 1.0, size=shape)
    c = synth.periodic_fix(synth.random_advector(shape, 0.3, gen))
    plan = mpdata.Plan(shape, n_iters=2, opts=FCT)
    plan.set_step_diag(True)
    p = dev(psi, torch.float64)
    plan.step(p, [dev(x, torch.float64) for x in c], n_steps=3)
    assert plan.step_diag() == pytest.approx(plan.diag(p), rel=1e-14)
