"""A request that fits the server's HBM budget without the optional residue workspace is
admitted, planned inside the budget; one that does not is refused."""
import pytest

from paper_2103_08473_amd import exacc, serve


@pytest.mark.parametrize("precision", ["FP64", "MIXED_FP32", "MIXED_BF16X3"])
def test_residue_workspace_does_not_decide_admission(monkeypatch, precision):
    shape = (20, 140, 420)
    prec = getattr(exacc, precision)
    full = exacc.memory_estimate(*shape, precision=prec)
    bare = [exacc.memory_estimate(*shape, precision=prec, ladder_defect_correction=0, hbm_budget_bytes=b)
            for b in (0, 1)]
    plan = full - (bare[0] - bare[1])   # with the mixed modes' correction arrays, without residues
    assert 0 < plan < full
    ran = []
    monkeypatch.setattr(serve, "solve_one", lambda req, opts: ran.append((req, opts)))
    for budget, status in ((full, 0), (full - 1, 0), (plan, 0), (plan - 1, exacc.ERR_NOMEM)):
        srv = serve.Server(budget, 1, dict(precision=prec))
        req = serve.Request(0, *shape, 1)
        srv.submit(req)
        srv.drain(1)
        assert req.status == status
        if status == 0:
            assert ran.pop() == (req, {"precision": prec} if budget == full else
                                 {"hbm_budget_bytes": budget, "precision": prec})
            assert plan <= req.mem <= budget
            assert srv.in_use == 0
    assert not ran
