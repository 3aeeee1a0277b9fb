"""Residue products whose sums are longer than one plane product takes (131072 terms): the
sums over the packed virtual pairs of a large basis."""
import pytest

pytestmark = pytest.mark.gpu


def test_sums_over_two_slices(lib):
    import torch
    from paper_2103_08473_amd import exacc
    o, v, X = 24, 515, 64  # 132355 virtual pairs
    g = torch.Generator(device="cuda")
    g.manual_seed(3)

    def gauss(*shape):
        return torch.randn(*shape, 2, generator=g, device="cuda", dtype=torch.float64)

    n = o + v
    eps = torch.cat([torch.linspace(-2, -1, o), torch.linspace(0.5, 3, v)]).to("cuda", torch.float64)
    B = torch.view_as_complex(gauss(X, n, n)) * 0.02
    B = (B + B.mH).contiguous()
    t1 = torch.zeros(o, v, dtype=torch.complex128, device="cuda")
    t2 = torch.view_as_complex(gauss(o, o, v, v)) * 0.01
    t2 = t2 - t2.transpose(0, 1)
    t2 = (t2 - t2.transpose(2, 3)).contiguous()
    opts = dict(doubles_only=1, diis_size=1)
    base = exacc.memory_estimate(o, v, X, hbm_budget_bytes=1, **opts)
    out = []
    for budget in (base, 0):
        with exacc.CCSD(eps, B, o, hbm_budget_bytes=budget, **opts) as cc:
            cc.set_amplitudes(t1, t2)
            s1, s2 = torch.empty_like(t1), torch.empty_like(t2)
            cc.residual(s1, s2)
            out.append(s2)
    plain, mod = out
    assert bool((plain != mod).any())  # another route was taken
    tol = v * (v - 1) // 2 * 2.0 ** -53
    d, m = float((plain - mod).abs().max()), float(plain.abs().max())
    print("max |d| / max %.2e (tolerance %.2e)" % (d / m, tol), flush=True)
    assert d <= tol * m
