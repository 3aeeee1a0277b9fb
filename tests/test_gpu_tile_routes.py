"""FP64 and FP32 products on every tile size, and DF factors over several chunks, against the
oracle at the edges of the tiles and chunks."""
import numpy as np
import pytest

from oracle.ccsd import build_integrals, residual
from oracle.dffactors import df_factors as df_oracle
from paper_2103_08473_amd.synth import make_amplitudes, make_system

pytestmark = pytest.mark.gpu


# nvir and naux on, one below and one past 16 and 32; o v on and past 64 (4 x 16, 5 x 13) and
# 128; a long naux, whose sums are split; nvir 33 and 47: whole and cut tiles above the wanted
# half of the ladder's grouped build
@pytest.mark.parametrize("o,v,X", [(2, 15, 31), (4, 16, 32), (5, 13, 33), (3, 17, 700), (8, 16, 64),
                                   (3, 31, 48), (4, 32, 65), (2, 33, 257), (5, 47, 96)])
@pytest.mark.parametrize("precision", ["FP64", "MIXED_FP32"])
def test_residual_at_tile_edges(lib, o, v, X, precision):
    from paper_2103_08473_amd import exacc
    eps, B = make_system(o, v, X, seed=o * 100 + v, sigma=0.2)
    t = make_amplitudes(o, v, seed=o + v, scale=0.1)
    want = residual(eps, build_integrals(B, o), *t)
    opts = {} if precision == "FP64" else {"precision": getattr(exacc, precision)}
    with exacc.CCSD(eps, B, o, **opts) as cc:
        cc.set_amplitudes(*t)
        got = cc.residual()
    tol = 1e-12 if precision == "FP64" else 1e-5  # the bars of the parity tests
    scale = max(np.abs(x).max() for x in want)
    for g, w in zip(got, want):
        assert np.abs(g - w).max() <= tol * scale


# 128 MB of half-transformed integrals hold 910 of 1000 auxiliary functions, and of the metric
# product's columns 8388 of 9216
def test_df_factors_in_chunks(lib):
    from paper_2103_08473_amd import exacc
    nao, n, X = 96, 96, 1000
    rng = np.random.default_rng(31)
    J = rng.normal(0, 0.1, (X, nao, nao)) + 1j * rng.normal(0, 0.1, (X, nao, nao))
    J = J + np.conj(J.transpose(0, 2, 1))
    A = rng.normal(0, 0.3 / np.sqrt(X), (X, X))
    V = np.eye(X) + 0.5 * (A + A.T)
    V = V @ V.T
    C = np.linalg.qr(rng.normal(size=(nao, nao)) + 1j * rng.normal(size=(nao, nao)))[0]
    want = df_oracle(C, J, V)
    B, _ = exacc.df_factors(C, J, V)
    # the bar of the parity tests
    assert np.abs(B - want).max() <= 1e-12 * max(1.0, np.abs(want).max())


# split sums are added in a fixed order: every repeat is the same
@pytest.mark.parametrize("precision", ["FP64", "MIXED_FP32"])
def test_split_sums_repeat(lib, precision):
    from paper_2103_08473_amd import exacc
    o, v, X = 4, 21, 900
    eps, B = make_system(o, v, X, seed=3, sigma=0.2)
    t = make_amplitudes(o, v, seed=5, scale=0.1)
    with exacc.CCSD(eps, B, o, precision=getattr(exacc, precision)) as cc:
        cc.set_amplitudes(*t)
        first = [x.copy() for x in cc.residual()]
        for _ in range(40):
            for a, b in zip(first, cc.residual()):
                assert np.array_equal(a, b)
