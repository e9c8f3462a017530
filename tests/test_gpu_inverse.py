"""The inverse of marching-on-in-time's diagonal block (stb_gj_invert, an internal
function): what it refuses, and every panel width with pivots off the diagonal."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53
OK, INTERNAL = 0, 7


@pytest.fixture(scope="module")
def invert():
    import torch
    torch.cuda.init()
    from paper_2103_16841_amd import stb
    f = stb.load()._Z13stb_gj_invertP7stb_ctxlPdS1_
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    ctx = stb.Context(0)

    def call(D):
        """(status, inverse) of a device tensor, which is left as it is."""
        work, out = D.clone(), torch.full_like(D, np.nan)
        torch.cuda.synchronize()
        return f(ctx.h, D.shape[0], work.data_ptr(), out.data_ptr()), out
    yield call
    ctx.close()


def _dev(D):
    import torch
    return torch.from_numpy(np.ascontiguousarray(D)).cuda()


@pytest.mark.parametrize("K", [1, 17, 60, 257])
def test_refuses_singular_and_non_finite(invert, K):
    D = np.random.default_rng(K).standard_normal((K, K)) + 8 * np.sqrt(K) * np.eye(K)
    assert invert(_dev(D))[0] == OK
    places = {(0, 0), (K - 1, K - 1), (K // 2, K // 3), (K - 1, 0), (0, K - 1)}
    for bad in (np.nan, np.inf, -np.inf):
        for i, j in places:
            E = D.copy()
            E[i, j] = bad
            assert invert(_dev(E))[0] == INTERNAL, (bad, i, j)
    for k in (0, K // 2, K - 1):
        for cut in (np.s_[k, :], np.s_[:, k]):
            E = D.copy()
            E[cut] = 0.0
            assert invert(_dev(E))[0] == INTERNAL, cut
    # a pivot whose reciprocal is beyond the range
    E = D.copy()
    E[:, K // 2] = 0.0
    E[K // 2, K // 2] = 1e-310
    assert invert(_dev(E))[0] == INTERNAL


def test_smallest_pivots(invert):
    """Subnormal pivots with a finite reciprocal are pivots, also beside zeros."""
    d = 6e-309
    for E in ([[d]], [[-d]], [[0.0, 1.0], [d, 0.0]], [[0.0, 0.0, d], [1.0, 0.0, 0.0], [0.0, 2.0, 0.0]]):
        s, X = invert(_dev(np.array(E)))
        ref = np.zeros((len(E), len(E)))
        for i, row in enumerate(E):
            for j, v in enumerate(row):
                ref[j, i] = 1.0 / v if v else 0.0
        assert s == OK and np.array_equal(X.cpu().numpy(), ref)
