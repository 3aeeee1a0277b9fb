"""DF factors written over their own inputs: the result is that of separate buffers."""
import numpy as np
import pytest

from paper_2103_08473_amd.synth import make_df_inputs

pytestmark = pytest.mark.gpu


# over C, over J from its first element and from a later one (the output of one auxiliary function
# then covers integrals of the next); one chunk of the transforms and several
@pytest.mark.parametrize("over", ["C", "J", "J+"])
@pytest.mark.parametrize("nao,n,X,noalloc", [(40, 30, 100, 0), (40, 30, 100, 1), (200, 150, 300, 0)])
def test_output_over_an_input(lib, nao, n, X, noalloc, over):
    import ctypes
    import torch
    from paper_2103_08473_amd import exacc
    C, J, V, _ = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in make_df_inputs(nao, n, X, seed=X))
    ref, _ = exacc.df_factors(C, J, V)
    own = C if over == "C" else J
    shift = 0 if over != "J+" else 3 * nao
    buf = torch.empty(shift + max(own.numel(), X * n * n), dtype=torch.complex128, device="cuda")
    buf[:own.numel()] = own.reshape(-1)
    B = buf[shift:shift + X * n * n]
    c, j = (buf, J) if over == "C" else (C, buf)
    L, it = exacc.load(), ctypes.c_int(0)
    torch.cuda.synchronize()
    if noalloc:
        st = L.exacc_df_factors_noalloc(nao, n, X, c.data_ptr(), j.data_ptr(), V.data_ptr(), B.data_ptr(), None,
                                        ctypes.byref(it))
    else:
        st = L.exacc_df_factors(nao, n, X, c.data_ptr(), j.data_ptr(), V.data_ptr(), B.data_ptr(), 1, None,
                                ctypes.byref(it))
    torch.cuda.synchronize()
    assert st == 0
    d = float((B.reshape(X, n, n) - ref).abs().max())
    print("max |d| %.2e" % d, flush=True)
    # the same sums, split differently where the chunks differ
    assert d <= 4 * (2 * nao + X) * 2.0 ** -53 * float(ref.abs().max())
