"""A call that needs the residue workspace's memory gives it back and goes on without it."""
import numpy as np
import pytest

from paper_2103_08473_amd.synth import make_amplitudes, make_system

pytestmark = pytest.mark.gpu


# a budget that holds the plan without residues and the Lambda buffers, but not the residue
# workspace (which takes what is left over the plan) as well; o v = 1000 takes residue products
def test_lambda_that_releases_the_residue_workspace(lib):
    import torch
    from paper_2103_08473_amd import exacc
    o, v, X = 10, 100, 3000
    Po, Pv = o * (o - 1) // 2, v * (v - 1) // 2
    need = 16 * (o * v + Po * Pv + 3 * o * v + 2 * (o * v) ** 2 + v * v * X + 3 * o ** 3 * v + Po * Po
                 + o * o * X + X + (o + v) ** 2)
    base = exacc.memory_estimate(o, v, X, hbm_budget_bytes=1)
    budget = base + need + (4 << 20)
    assert base + (64 << 20) < exacc.memory_estimate(o, v, X, hbm_budget_bytes=budget) <= budget
    eps, B = make_system(o, v, X, seed=1)
    t, l = make_amplitudes(o, v, seed=2), make_amplitudes(o, v, seed=3)

    def run(**opts):
        with exacc.CCSD(eps, B, o, **opts) as cc:
            cc.set_amplitudes(*t)
            first = cc.residual()
            free = torch.cuda.mem_get_info()[0]
            cc.set_lambda(*l)
            r = cc.lambda_residual()
            return r, cc.residual(), first, free - torch.cuda.mem_get_info()[0]

    tight, roomy = run(hbm_budget_bytes=budget), run()
    assert tight[3] < need // 2 < roomy[3]  # only the first gave memory back
    for g, w in zip(tight[:3], roomy[:3]):
        scale = max(np.abs(x).max() for x in w)
        for x, y in zip(g, w):
            assert np.abs(x - y).max() <= 1e-12 * scale  # the bar of the parity tests
