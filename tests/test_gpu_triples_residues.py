"""The triples' sums over virtuals on integer residues against the FP64 matrix kernel, which
several occupied blocks take."""
import numpy as np
import pytest

from paper_2103_08473_amd.synth import make_system

pytestmark = pytest.mark.gpu


def triples(o, v, X, t, **opts):
    from paper_2103_08473_amd import exacc
    eps, B = make_system(o, v, X, seed=5)
    with exacc.CCSD(eps, B, o, **opts) as cc:
        cc.set_amplitudes(*t)
        return np.array(cc.triples())


def amplitudes(o, v):
    rng = np.random.default_rng(o + v)
    t1 = 0.01 * (rng.normal(size=(o, v)) + 1j * rng.normal(size=(o, v)))
    t2 = 0.01 * (rng.normal(size=(o, o, v, v)) + 1j * rng.normal(size=(o, o, v, v)))
    t2 = t2 - t2.transpose(1, 0, 2, 3)
    return t1, np.ascontiguousarray(t2 - t2.transpose(0, 1, 3, 2))


# one past and exactly whole 32-blocks and 64-k groups of nvir, batches of i cut to one or two
# rows at the last k, nvir over four blocks (the wider tiles); one row of t2 zero throughout
@pytest.mark.parametrize("o,v,zero", [(6, 97, False), (7, 128, True), (5, 129, False), (12, 80, True)])
def test_triples_with_and_without_residues(lib, o, v, zero):
    t1, t2 = amplitudes(o, v)
    if zero:
        t2[:, :, 3] = 0
        t2[:, :, :, 3] = 0
    # a core-like row: t2 of occupied 0 is 1e-4 of the rest
    t2[0] *= 1e-4
    t2[:, 0] *= 1e-4
    mod = triples(o, v, 40, (t1, t2))
    plain = triples(o, v, 40, (t1, t2), triples_occ_block=2)
    # (the energies average the roundings of some 10^6 terms and may agree to the last bit)
    # W is off by at most 3 nvir + 3 nocc roundings of its norm, the energies are quadratic in it
    tol = 6 * (v + o) * 2.0 ** -53
    print("max |d| / max %.2e (tolerance %.2e)" % (np.abs(mod - plain).max() / np.abs(plain).max(), tol), flush=True)
    assert np.abs(mod - plain).max() <= tol * np.abs(plain).max()


def test_nan_amplitude_gives_nan(lib):
    o, v = 6, 97
    t1, t2 = amplitudes(o, v)
    t2[1, 2, 3, 4] = t2[2, 1, 4, 3] = np.nan
    t2[2, 1, 3, 4] = t2[1, 2, 4, 3] = np.nan
    assert np.isnan(triples(o, v, 40, (t1, t2))).all()
