"""Triples energies at sizes whose sums over virtuals run on integer residues, against the same
sums formed triple by triple with NumPy."""
import itertools

import numpy as np
import pytest

from paper_2103_08473_amd.synth import make_system

pytestmark = pytest.mark.gpu


def reference(eps, B, o, t1, t2):
    """(E(+T), E((T)), E(-T)) with the definitions of oracle.triples, one i < j < k at a time."""
    Boo, Bvo, Bvv = B[:, :o, :o], B[:, o:, :o], B[:, o:, o:]
    X, v = B.shape[0], Bvv.shape[1]
    eo, ev = eps[:o], eps[o:]
    cyc = lambda x: x + x.transpose(1, 2, 0) + x.transpose(2, 0, 1)   # abc + cab + bca
    Ve = []                                                          # [i][a, b, e] = <ab||ie>
    for i in range(o):
        x = (Bvo[:, :, i].T @ Bvv.reshape(X, -1)).reshape(v, v, v)
        Ve.append(x - x.transpose(1, 0, 2))
    am = np.einsum("Pai,Pmj->aimj", Bvo, Boo, optimize=True)         # (ai|mj)
    Vm = am.transpose(1, 3, 0, 2) - am.transpose(3, 1, 0, 2)         # [i, j, a, m] = <am||ij>
    x = np.einsum("Pai,Pbj->ijab", Bvo, Bvo, optimize=True)
    Vd = x - x.transpose(1, 0, 2, 3)
    a = np.arange(v)
    keep = (a[:, None, None] < a[None, :, None]) & (a[None, :, None] < a[None, None, :])
    e4 = e5 = ey = 0.0
    for i, j, k in itertools.combinations(range(o), 3):
        W = Z = Y = 0.0
        for p, q, r in ((i, j, k), (j, k, i), (k, i, j)):
            W = W + (Ve[p].reshape(-1, v) @ t2[q, r]).reshape(v, v, v)
            W = W + (Vm[p, q] @ t2[r].reshape(o, -1)).reshape(v, v, v)
            Z = Z + Vd[p, q][:, :, None] * t1[r]
            Y = Y + t2[p, q][:, :, None] * t1[r]
            d = t1[p][:, None, None] * t1[q][None, :, None] * t1[r]
            Y = Y + (d - d.transpose(1, 0, 2)) / 3.0
        W, Z, Y = cyc(W)[keep], cyc(Z)[keep], cyc(Y)[keep]
        D = (ev[:, None, None] + ev[None, :, None] + ev)[keep] - eo[i] - eo[j] - eo[k]
        e4 -= float((np.abs(W) ** 2 / D).sum())
        e5 -= float(((Z.conj() * W).real / D).sum())
        ey += float((Y.conj() * W).real.sum())
    return np.array([e4, e4 + e5, e4 + ey])


# well past the size from which residues are taken; nvir a multiple of 32 and not, four and five blocks of 32
@pytest.mark.parametrize("o,v", [(7, 128), (6, 140)])
def test_triples_against_numpy(lib, o, v):
    from paper_2103_08473_amd import exacc
    eps, B = make_system(o, v, 48, seed=o)
    rng = np.random.default_rng(o)
    g = lambda *s: 0.01 * (rng.normal(size=s) + 1j * rng.normal(size=s))
    t1, t2 = g(o, v), g(o, o, v, v)
    t2 = t2 - t2.transpose(1, 0, 2, 3)
    t2 = np.ascontiguousarray(t2 - t2.transpose(0, 1, 3, 2))
    ref = reference(eps, B, o, t1, t2)
    with exacc.CCSD(eps, B, o) as cc:
        cc.set_amplitudes(t1, t2)
        got = np.array(cc.triples())
    # W is off by at most 3 nvir + 3 nocc roundings of its norm here and there, and the integrals by
    # naux; the energies are quadratic in W
    tol = 2 * (6 * (v + o) + 2 * 48) * 2.0 ** -53
    print("max |d| / max %.2e (tolerance %.2e)" % (np.abs(got - ref).max() / np.abs(ref).max(), tol), flush=True)
    assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
