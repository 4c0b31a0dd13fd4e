"""Failure detection through the kernel instances that
tests/test_gpu_nonfinite.py does not reach: the 2-D single pass in every
variant (limited velocities for a following pass, variable G, third-order and
divergent-flow terms, the launch over the three shallow-water fields, the
recording launches of the gradient), both types, and the tiled 1-D steps.  A
NaN or an infinity in psi or in one advector wall shows in the result; the
clean run of the same inputs is finite."""
import numpy as np
import pytest
import torch

from paper_1407_1309_amd import mpdata, synth
from tests.gpu_util import dev
from tests.test_gpu_nonfinite import _diag_status, _family_inputs

pytestmark = pytest.mark.gpu
FCT, IGA, TOT, ABS, DFL, KAHAN = (mpdata.OPT_FCT, mpdata.OPT_IGA, mpdata.OPT_TOT, mpdata.OPT_ABS,
                                  mpdata.OPT_DFL, mpdata.OPT_KAHAN)
DT = [torch.float64, torch.float32]
BAD = [np.nan, np.inf, -np.inf]
BAD_ID = ["nan", "inf", "-inf"]

# (shape, n_iters, opts, with_g)
STEPS = [((70, 150), 1 + p, o, g) for p, o, g in [
    (1, 0, False), (1, FCT, False), (1, FCT | IGA, False), (1, FCT | IGA | DFL, False),
    (1, IGA | TOT, True), (1, FCT | ABS, False), (1, FCT | KAHAN, True), (1, FCT | DFL, False),
    (2, 0, False), (2, FCT, False), (2, FCT | TOT, True), (2, FCT | ABS | DFL, False),
    (3, FCT | TOT, False)]] + [((9001,), 2, FCT, False), ((9001,), 3, TOT | FCT, True)]


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("where", ["psi", "wall"])
@pytest.mark.parametrize("value", BAD, ids=BAD_ID)
@pytest.mark.parametrize("shape,n_iters,opts,with_g", STEPS)
def test_steps(shape, n_iters, opts, with_g, value, where, dtype):
    psi, c, g = _family_inputs(shape, 1, opts, with_g)
    plan = mpdata.Plan(shape, dtype=dtype, n_iters=n_iters, opts=opts, bc=1, has_g=with_g)
    gd, cd = dev(g, dtype), [dev(x, dtype) for x in c]
    p = dev(psi, dtype)
    plan.step(p, cd, g=gd, n_steps=3)
    assert _diag_status(plan, p, gd) == (mpdata.OK, 0)
    mid = tuple(s // 2 for s in shape)
    p = dev(psi, dtype)
    (p if where == "psi" else cd[-1])[mid] = value
    plan.step(p, cd, g=gd, n_steps=3)
    rc, bad = _diag_status(plan, p, gd)
    assert rc == mpdata.ENONFINITE and bad >= 1, (rc, bad)


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("value", BAD, ids=BAD_ID)
@pytest.mark.parametrize("opts", [FCT | IGA | DFL, FCT | ABS])
def test_shallow_water(opts, value, dtype):
    shape = (70, 150)
    h, q, hp, qp, dx = synth.sw_state(shape, 5, half=2.0, ring=False)
    for field in (None, 0, 1, 2):
        f = [dev(x, dtype) for x in (h + 0.3, *q, hp + 0.3, *qp)]
        if field is not None:
            f[field][35, 75] = value
        c = [torch.zeros([s + (k == d) for k, s in enumerate(shape)], dtype=dtype, device="cuda")
             for d in range(2)]
        plan = mpdata.Plan(shape, dtype=dtype, n_iters=2, opts=opts, bc=1)
        plan.sw_step(f[0], f[1:3], f[3], f[4:6], c, min(dx) / 8, dx, grav=1.0, eps=1e-8, n_steps=2)
        rc = [_diag_status(plan, x)[0] for x in f[:3]]
        assert (mpdata.ENONFINITE in rc) == (field is not None), (field, rc)


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("value", BAD, ids=BAD_ID)
@pytest.mark.parametrize("bc,n_iters,opts", [(0, 2, FCT), (1, 2, FCT | IGA), (0, 3, FCT), (1, 2, 0)])
def test_gradient(bc, n_iters, opts, value, dtype):
    """The end state of a differentiated run, and the gradient with respect to
    psi0 of a run from a non-finite state."""
    shape = (70, 150)
    psi, c, _ = _family_inputs(shape, bc, opts, False)
    for bad in (False, True):
        p, cd = dev(psi, dtype), [dev(x, dtype) for x in c]
        if bad:
            p[35, 75] = value
        plan = mpdata.Plan(shape, dtype=dtype, n_iters=n_iters, opts=opts, bc=bc, adj_steps=4,
                           ckpt_every=2)
        p.requires_grad_(True)
        cd = [x.requires_grad_(True) for x in cd]
        end = mpdata.advance(p, cd, plan, 4, ckpt_every=2)
        grads = torch.autograd.grad(end.square().sum(), [p, *cd])
        fin = [bool(torch.isfinite(x).all()) for x in (end.detach(), *grads)]
        assert fin == [not bad] * len(fin) if not bad else not fin[0] and not all(fin[1:]), fin
