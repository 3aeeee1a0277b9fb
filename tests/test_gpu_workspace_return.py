"""The residue workspace is extra memory: what needs its place takes it, another handle's too,
and the handle takes it again when there is room."""
import numpy as np
import pytest

from paper_2103_08473_amd.synth import make_amplitudes, make_system

pytestmark = pytest.mark.gpu


def test_workspace_comes_back_after_the_triples(lib):
    """A budget that holds the triples' temporaries only without the workspace."""
    from paper_2103_08473_amd import exacc
    # o v = 4800 takes residues; the temporaries (1.5 o v^3) are more than create's (a 2 GiB chunk
    # and half of it), which the plan has room for
    o, v, X = 24, 200, 40
    base, budget = (exacc.memory_estimate(o, v, X, hbm_budget_bytes=b) for b in (1, 0))
    eps, B = make_system(o, v, X, seed=1)
    t = make_amplitudes(o, v, seed=2)

    def run(budget, triples):
        import torch
        with exacc.CCSD(eps, B, o, hbm_budget_bytes=budget) as cc:
            cc.set_amplitudes(*t)
            first = cc.residual()
            free = torch.cuda.mem_get_info()[0]
            e = np.array(cc.triples()) if triples else 0.0
            given = torch.cuda.mem_get_info()[0] - free
            return first, cc.residual(), e, given

    first, after, e, given = run(budget, True)
    assert given >= (budget - base) // 2                            # the triples took its place
    assert all((a == b).all() for a, b in zip(first, after))        # and it was there again
    plain = run(base, False)
    assert any((a != b).any() for a, b in zip(first, plain[0]))     # which is another route
    roomy = run(0, True)
    assert roomy[3] == 0 and np.abs(e - roomy[2]).max() <= 1e-12 * np.abs(e).max()


def test_second_handle_takes_an_idle_ones_workspace(lib):
    import torch
    from paper_2103_08473_amd import exacc
    o, v, X = 24, 168, 504
    base = exacc.memory_estimate(o, v, X, hbm_budget_bytes=1)
    extra = exacc.memory_estimate(o, v, X) - base
    assert extra > 1 << 30
    eps, B = make_system(o, v, X, seed=3)
    t = make_amplitudes(o, v, seed=4)
    with exacc.CCSD(eps, B, o) as cc:
        cc.set_amplitudes(*t)
        first = cc.residual()
        free = torch.cuda.mem_get_info()[0]
        with exacc.CCSD(eps, B, o, hbm_budget_bytes=base):
            need = free - torch.cuda.mem_get_info()[0]
        # leave half a workspace less than a second handle holds
        fill = torch.empty(torch.cuda.mem_get_info()[0] - need + extra // 2, dtype=torch.uint8, device="cuda")
        with exacc.CCSD(eps, B, o) as other:
            other.set_amplitudes(*t)
            second, again = other.residual(), cc.residual()
        del fill
        torch.cuda.empty_cache()
        last = cc.residual()
    for r in (second, again):                                       # without the workspace
        for a, b in zip(first, r):
            assert np.abs(a - b).max() <= 1e-12 * np.abs(a).max()
    assert all((a == b).all() for a, b in zip(first, last))         # with it


def test_phase_answers_while_a_call_is_running(lib):
    """A thread that watches a solve is not held until the solve returns."""
    import threading
    import time
    from paper_2103_08473_amd import exacc
    o, v, X = 8, 48, 144
    eps, B = make_system(o, v, X, seed=5)
    with exacc.CCSD(eps, B, o, tol=0.0) as cc:
        cc.iterate(1)
        t0 = time.perf_counter()
        cc.iterate(20)
        steps = max(40, int(20 * 2.0 / (time.perf_counter() - t0)))  # about two seconds
        run = threading.Thread(target=cc.iterate, args=(steps,))
        run.start()
        time.sleep(0.2)
        t0 = time.perf_counter()
        cc.phase()
        waited, running = time.perf_counter() - t0, run.is_alive()
        run.join()
    assert running and waited < 0.5
