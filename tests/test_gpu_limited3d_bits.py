"""The limited 3-D step gives the bits it has always given: SHA-256 of its
result for inputs of plain uniform numbers, against values recorded with the
general cell kernel (limited velocities and corrective pass, no contraction of
a flux with the difference it goes into).  A kernel that rounds an expression
differently changes them."""
import hashlib
import json
import os

import pytest
import torch

from paper_1407_1309_amd import mpdata, synth
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu
FCT, IGA, TOT, KAHAN = mpdata.OPT_FCT, mpdata.OPT_IGA, mpdata.OPT_TOT, mpdata.OPT_KAHAN
GOLD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "limited3d_bits.json")
CASES = [(shape, n_iters, opts, bc, g) for shape in ((11, 13, 37), (20, 33, 70))
         for n_iters, opts, bc, g in ((2, FCT, 0, False), (2, FCT, 1, True), (3, FCT, 0, False),
                                      (2, FCT | KAHAN, 1, True), (2, FCT | IGA, 0, True),
                                      (2, FCT | TOT | IGA, 1, False), (4, FCT | TOT, 1, False))]


def digest(shape, n_iters, opts, bc, with_g, dtype):
    gen = synth.rng(17)
    psi = gen.uniform(0.1, 1.0, size=shape)
    c = []
    for d in range(3):
        w = gen.uniform(-0.15, 0.15, size=[n + (k == d) for k, n in enumerate(shape)])
        if bc == 0:
            w[tuple(-1 if k == d else slice(None) for k in range(3))] = \
                w[tuple(0 if k == d else slice(None) for k in range(3))]
        c.append(w)
    g = gen.uniform(0.7, 1.3, size=shape) if with_g else None
    plan = mpdata.Plan(shape, dtype=dtype, n_iters=n_iters, opts=opts, bc=bc, has_g=with_g)
    p = dev(psi, dtype)
    plan.step(p, [dev(x, dtype) for x in c], g=dev(g, dtype), n_steps=2)
    return hashlib.sha256(p.cpu().numpy().tobytes()).hexdigest()[:16]


def key(shape, n_iters, opts, bc, with_g, dtype):
    return "%s it%d opts%d bc%d g%d %s" % ("x".join(map(str, shape)), n_iters, opts, bc, with_g,
                                           str(dtype)[6:])


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: key(*c, torch.float32)[:-8])
def test_limited_step_keeps_its_bits(case, dtype):
    gold = json.load(open(GOLD))
    assert digest(*case, dtype) == gold[key(*case, dtype)]
