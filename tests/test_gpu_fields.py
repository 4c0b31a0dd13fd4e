"""The shallow-water launch over three fields and the source term added on the
way into the workspace, at the edges of strips and chunks: against the oracle
on ragged grids, and with the divergent-flow and |psi| option sets."""
import numpy as np
import pytest
import torch

import oracle
from paper_1407_1309_amd import mpdata, synth
from tests.gpu_util import as_dtype, assert_parity, dev

pytestmark = pytest.mark.gpu
FCT, IGA, ABS, DFL = mpdata.OPT_FCT, mpdata.OPT_IGA, mpdata.OPT_ABS, mpdata.OPT_DFL
DT = [torch.float64, torch.float32]


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("opts", [FCT | IGA | DFL, FCT | ABS], ids=["iga-fct-dfl", "abs-fct"])
@pytest.mark.parametrize("bc", [0, 1], ids=["periodic", "open"])
@pytest.mark.parametrize("shape", [(3, 3), (4, 58), (9, 59), (61, 117), (130, 33)])
def test_sw_fields(shape, bc, opts, dtype):
    h, q, hp, qp, dx = synth.sw_state(shape, 5, half=2.0, ring=False)
    h, hp = h + 0.3, hp + 0.3
    f = [as_dtype(x, dtype) for x in (h, *q, hp, *qp)]
    dt = min(dx) / 8
    n = 3
    rh, rq, rhp, rqp = f[0], f[1:3], f[3], f[4:6]
    for _ in range(n):
        old = rh, rq, rhp, rqp
        (rh, rq), rhp, rqp = oracle.sw_step(rh, rq, rhp, rqp, dt, dx, eps=1e-8, grav=1.0, n_iters=2,
                                            opts=opts, bc=bc), rh, rq
    rc = oracle.vip_advector(old[1], old[0], old[3], old[2], dt, dx, eps=1e-8, bc=bc)
    plan = mpdata.Plan(shape, dtype=dtype, n_iters=2, opts=opts, bc=bc, kernel=mpdata.KERNEL_PASS)
    g = [dev(x, dtype) for x in f]
    c = [torch.full([s + (k == d) for k, s in enumerate(shape)], 9.0, dtype=dtype, device="cuda")
         for d in range(2)]
    plan.sw_step(g[0], g[1:3], g[3], g[4:6], c, dt, dx, grav=1.0, eps=1e-8, n_steps=n)
    torch.cuda.synchronize()
    for got, ref in zip(g + c, [rh, *rq, rhp, *rqp, *rc]):
        assert_parity(got.double().cpu().numpy(), ref, dtype)


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("shape,bc,opts,n_iters", [
    ((37,), 0, FCT, 2), ((6007,), 1, FCT, 2), ((40, 70), 0, FCT, 2), ((40, 70), 1, 0, 1),
    ((40, 70), 1, FCT | IGA, 2), ((9, 20, 33), 1, IGA, 2), ((9, 20, 33), 0, FCT, 3)])
def test_source_ahead_of_the_step(shape, bc, opts, n_iters, dtype):
    gen = synth.rng(3)
    psi, r0, r1 = (as_dtype(gen.uniform(0.1, 1.0, size=shape), dtype) for _ in range(3))
    c = synth.random_advector(shape, 0.3, gen)
    c = [as_dtype(x, dtype) for x in (synth.periodic_fix(c) if bc == 0 else c)]
    ref = oracle.step_rhs(psi, c, r_pre=r0, a_pre=0.1, r_post=r1, a_post=0.2, n_iters=n_iters,
                          opts=opts, bc=bc)
    plan = mpdata.Plan(shape, dtype=dtype, n_iters=n_iters, opts=opts, bc=bc)
    p = dev(psi, dtype)
    plan.set_step_diag(True)
    plan.step_rhs(p, [dev(x, dtype) for x in c], r_pre=dev(r0, dtype), a_pre=0.1,
                  r_post=dev(r1, dtype), a_post=0.2)
    torch.cuda.synchronize()
    assert_parity(p.double().cpu().numpy(), ref, dtype)
