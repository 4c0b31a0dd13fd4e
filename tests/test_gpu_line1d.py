"""1-D steps (line1d.hpp) against the oracle at the sizes where a launch
changes shape: grids of one cell, of one wave and one cell more, of the
largest one-workgroup grid and the first tiled one, ragged last tiles; every
option, both boundaries, up to eight passes; and the same bits however a call
is cut into launches."""
import numpy as np
import pytest
import torch

import oracle
from paper_1407_1309_amd import mpdata, synth
from tests.gpu_util import as_dtype, assert_parity, dev, gpu_run

pytestmark = pytest.mark.gpu
FCT, IGA, TOT, ABS, DFL, KAHAN = (mpdata.OPT_FCT, mpdata.OPT_IGA, mpdata.OPT_TOT, mpdata.OPT_ABS,
                                  mpdata.OPT_DFL, mpdata.OPT_KAHAN)
DT = [torch.float64, torch.float32]


def _inputs(n, bc, opts, with_g, seed, dtype):
    gen = synth.rng(seed)
    signed = opts & (IGA | ABS)
    psi = gen.normal(size=n) if signed else gen.uniform(0.1, 1.0, size=n)
    c = gen.uniform(-0.4, 0.4, size=n + 1)
    if bc == 0:
        c[n] = c[0]
    g = gen.uniform(0.7, 1.3, size=n) if with_g else None
    return as_dtype(psi, dtype), [as_dtype(c, dtype)], as_dtype(g, dtype)


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("bc", [0, 1], ids=["periodic", "open"])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 58, 60, 61, 119, 241, 927, 929, 1859, 2275, 2277, 4551,
                               20011])
def test_line_sizes(n, bc, dtype):
    if bc == 0 and n < 3:
        pytest.skip("a periodic dimension has at least 3 cells")
    for opts, n_iters in ((FCT, 2), (0, 3), (FCT | IGA, 2)):
        psi, c, g = _inputs(n, bc, opts, False, n + opts, dtype)
        ref = oracle.step(psi, c, n_iters=n_iters, opts=opts, bc=bc, n_steps=5)
        out = gpu_run(psi, c, g, dtype, n_iters, opts, bc, 5)
        assert_parity(out, ref, dtype, (opts, n_iters))


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("bc", [0, 1], ids=["periodic", "open"])
@pytest.mark.parametrize("opts,n_iters", [(0, 1), (KAHAN, 1), (FCT | TOT, 3), (TOT | IGA, 2),
                                          (FCT | ABS, 4), (DFL, 3), (DFL | FCT | IGA, 2),
                                          (FCT | DFL | TOT | KAHAN, 3), (FCT, 8)])
def test_line_options(opts, n_iters, bc, dtype):
    for n in (37, 700, 6007):
        for with_g in (False, True):
            psi, c, g = _inputs(n, bc, opts, with_g, n + opts + n_iters, dtype)
            if opts & DFL and not opts & IGA:
                psi = psi + 0.5
            ref = oracle.step(psi, c, g=g, n_iters=n_iters, opts=opts, bc=bc, n_steps=3)
            out = gpu_run(psi, c, g, dtype, n_iters, opts, bc, 3)
            assert_parity(out, ref, dtype, (n, with_g))


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("bc", [0, 1], ids=["periodic", "open"])
@pytest.mark.parametrize("n", [500, 5003, 300007])
def test_line_bits_do_not_depend_on_the_cut(n, bc, dtype):
    """One call of 7 steps, 7 calls of one, and 2 + 5: the same bits."""
    psi, c, _ = _inputs(n, bc, FCT, False, n, dtype)
    outs = []
    for parts in ((7,), (1,) * 7, (2, 5)):
        plan = mpdata.Plan((n,), dtype=dtype, n_iters=2, opts=FCT, bc=bc)
        p, cd = dev(psi, dtype), [dev(x, dtype) for x in c]
        for k in parts:
            plan.step(p, cd, n_steps=k)
        torch.cuda.synchronize()
        outs.append(p.cpu())
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("dtype", DT, ids=["f64", "f32"])
@pytest.mark.parametrize("n,bc,opts,with_g", [(3, 0, FCT, False), (777, 1, FCT | IGA, False),
                                              (9001, 0, FCT | IGA, False), (9001, 1, ABS | TOT, True)])
def test_line_oscillator(n, bc, opts, with_g, dtype):
    psi, c, g = _inputs(n, bc, IGA, with_g, n, dtype)
    phi = as_dtype(synth.rng(n + 1).normal(size=n), dtype)
    rx, ry = oracle.osc_step(psi, phi, c, 0.05, g=g, n_iters=2, opts=opts, bc=bc, n_steps=5)
    plan = mpdata.Plan((n,), dtype=dtype, n_iters=2, opts=opts, bc=bc, has_g=with_g)
    p, q = dev(psi, dtype), dev(phi, dtype)
    plan.osc_step(p, q, [dev(x, dtype) for x in c], 0.05, n_steps=5, g=dev(g, dtype))
    torch.cuda.synchronize()
    assert_parity(np.concatenate([p.double().cpu().numpy(), q.double().cpu().numpy()]),
                  np.concatenate([rx, ry]), dtype)
