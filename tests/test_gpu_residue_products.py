"""Large FP64 products formed on integer residues against the FP64 matrix kernel: the same
residual with and without the residue workspace (which an HBM budget can leave out)."""
import numpy as np
import pytest

from paper_2103_08473_amd.synth import make_system

pytestmark = pytest.mark.gpu


def amplitudes(o, v, seed):
    rng = np.random.default_rng(seed)
    t1 = 0.01 * (rng.normal(size=(o, v)) + 1j * rng.normal(size=(o, v)))
    t2 = 0.01 * (rng.normal(size=(o, o, v, v)) + 1j * rng.normal(size=(o, o, v, v)))
    t2 = t2 - t2.transpose(1, 0, 2, 3)
    return t1, np.ascontiguousarray(t2 - t2.transpose(0, 1, 3, 2))


def residual(o, v, X, budget, t, **opts):
    from paper_2103_08473_amd import exacc
    eps, B = make_system(o, v, X, seed=3)
    with exacc.CCSD(eps, B, o, hbm_budget_bytes=budget, **opts) as cc:
        cc.set_amplitudes(*t)
        s1, s2 = cc.residual()
    return np.asarray(s1), np.asarray(s2)


# ladder tiles: the smallest nvir that takes them, whole blocks, several chunks of virtual rows
# (first rows inside and at the edge of a block); products: odd sizes off every tile, whole tiles (o v = 1280 = 5 x 256), one past a tile (o v = 1281)
# and a workspace so small that both operands are split in chunks (0: all it wants)
@pytest.mark.parametrize("o,v,X,room,opts", [
    (4, 65, 200, 0, {}), (5, 97, 131, 0, {"ladder_chunk_pairs": 700}), (5, 128, 128, 0, {"ladder_chunk_pairs": 3600}),
    (13, 87, 259, 0, {}), (13, 87, 259, 64, {}), (20, 64, 192, 0, {"ladder_group_nvir": 0}),
    (21, 61, 180, 0, {}), (30, 101, 420, 0, {"cc2": 1}), (24, 90, 270, 120, {"doubles_only": 1})])
def test_residual_with_and_without_residues(lib, o, v, X, room, opts):
    from paper_2103_08473_amd import exacc
    base = exacc.memory_estimate(o, v, X, hbm_budget_bytes=1, **opts)
    full = exacc.memory_estimate(o, v, X, **opts)
    budget = base + (room << 20) if room else full
    assert base < budget <= full
    t = amplitudes(o, v, seed=o)
    if opts.get("doubles_only"):
        t = (np.zeros_like(t[0]), t[1])
    plain = residual(o, v, X, base, t, **opts)
    mod = residual(o, v, X, budget, t, **opts)
    assert any((a != b).any() for a, b in zip(plain, mod))  # another route was taken
    # either route rounds a sum of K products to within K 2^-53 of the operands' norms; the
    # longest sum runs over the virtual pairs or over o v
    tol = max(v * (v - 1) // 2, o * v) * 2.0 ** -53
    for a, b in zip(plain, mod):
        scale = max(np.abs(a).max(), 1e-300)
        print("max |d| / max %.2e (tolerance %.2e)" % (np.abs(a - b).max() / scale, tol), flush=True)
        assert np.abs(a - b).max() <= tol * scale


def test_lambda_with_and_without_residues(lib):
    """The Lambda ladder's T1-dressed factors are not Hermitian: full build, two W chunks."""
    from paper_2103_08473_amd import exacc
    o, v, X = 6, 75, 150
    eps, B = make_system(o, v, X, seed=4)
    t, l = amplitudes(o, v, seed=5), amplitudes(o, v, seed=6)
    base = exacc.memory_estimate(o, v, X, hbm_budget_bytes=1, ladder_chunk_pairs=1500)
    out = []
    for mod in (False, True):
        with exacc.CCSD(eps, B, o, hbm_budget_bytes=0 if mod else base + (63 << 20), ladder_chunk_pairs=1500) as cc:
            cc.set_amplitudes(*t)
            cc.set_lambda(*l)
            out.append([np.asarray(x) for x in cc.lambda_residual()])
    tol = v * (v - 1) // 2 * 2.0 ** -53
    assert any((a != b).any() for a, b in zip(*out))  # another route was taken
    for a, b in zip(*out):
        assert np.abs(a - b).max() <= tol * np.abs(a).max()


@pytest.mark.parametrize("mode", ["MIXED_BF16X3", "MIXED_FP32"])
@pytest.mark.parametrize("o,v,X,pairs", [(4, 65, 200, 0), (5, 97, 131, 700), (3, 130, 128, 0)])
def test_low_precision_ladder_rows_in_groups(lib, mode, o, v, X, pairs):
    """The low-precision ladder builds several rows per product where the workspace (idle in
    that phase) holds their tiles, one row without it: the same sums."""
    from paper_2103_08473_amd import exacc
    opts = dict(precision=getattr(exacc, mode), ladder_chunk_pairs=pairs)
    base = exacc.memory_estimate(o, v, X, hbm_budget_bytes=1, **opts)
    t = amplitudes(o, v, seed=2)
    one = residual(o, v, X, base, t, **opts)
    grouped = residual(o, v, X, 0, t, **opts)
    for a, b in zip(one, grouped):
        if mode == "MIXED_BF16X3":
            assert (a == b).all()    # the same kernel per tile
        else:  # tiles and splits differ with the size: FP32 sums of P_v terms
            assert np.abs(a - b).max() <= np.sqrt(v * (v - 1) / 2) * 2.0 ** -23 * np.abs(a).max()


def test_non_finite_amplitudes_stay_non_finite(lib):
    from paper_2103_08473_amd import exacc
    o, v, X = 13, 87, 259
    t1, t2 = amplitudes(o, v, seed=1)
    t2[0, 1, 2, 3] = np.nan
    s1, s2 = residual(o, v, X, exacc.memory_estimate(o, v, X), (t1, t2))
    assert not np.isfinite(s2).all() and not np.isfinite(s1).all()
