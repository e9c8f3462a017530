"""What a refused allocation or a refused input leaves: an error, no result that
looks like one, and a library that goes on working.  Allocations are refused by
the calling thread's allowance (stb_set_alloc_allowance, an internal function)."""
import contextlib
import ctypes

import numpy as np
import pytest

from paper_2103_16841_amd import inputs

pytestmark = pytest.mark.gpu

NO_MEMORY = 3


@pytest.fixture(scope="module")
def stb():
    import torch
    torch.cuda.init()
    from paper_2103_16841_amd import stb as s
    s.load()
    return s


@contextlib.contextmanager
def allowance(stb, nbytes):
    """Device allocations of this thread are refused beyond nbytes in all."""
    f = stb.load()._Z23stb_set_alloc_allowancel
    f.argtypes, f.restype = [ctypes.c_int64], None
    f(nbytes)
    try:
        yield
    finally:
        f(-1)


def test_refused_matrix_core_copy(stb):
    """Whichever allocation of the first 16-RHS product is refused, y is written
    or the call fails; the matrix has no copy then, and the next call works."""
    import torch
    ctx = stb.Context(0)
    mesh = inputs.icosphere_mesh(1, 8)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    W = torch.from_numpy(np.random.default_rng(0).standard_normal((mesh.nt, 16))).cuda()
    ref = stb.assemble_V(ctx, M).apply(W.cpu().numpy())
    A = stb.assemble_V(ctx, M)
    Y = torch.full_like(W, np.nan)
    torch.cuda.synchronize()
    refused, budget = 0, 0
    while True:
        ok = True
        with allowance(stb, budget):
            try:
                A.apply_dev(W.data_ptr(), Y.data_ptr(), 16)
            except stb.StbError as e:
                assert e.status == NO_MEMORY
                ok = False
        torch.cuda.synchronize()
        if ok:
            break
        refused += 1
        assert bool(torch.isnan(Y).all())
        # once the copy is there, only the product's own temporary is refused
        built = budget > 0 and stb.load().stb_apply16_noalloc(
            ctx.h, A.h, ctypes.c_void_p(W.data_ptr()), ctypes.c_void_p(Y.data_ptr()), None) == 0
        torch.cuda.synchronize()
        if built:
            assert np.array_equal(Y.cpu().numpy(), ref)
            Y.fill_(np.nan)
            torch.cuda.synchronize()
        budget = budget * 2 + 64
    assert refused >= 5
    assert np.array_equal(Y.cpu().numpy(), ref)
    A.close()
    M.close()
    ctx.close()
