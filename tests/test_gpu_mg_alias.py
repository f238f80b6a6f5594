"""Sweeps alone on one level (lfine == lcoarse) have no residual: the residual's
array may be one of the other two."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sweeps", [1, 2, 5])
@pytest.mark.parametrize("alias", ["phi", "f"])
def test_sweeps_alone_with_one_array_twice(alias, sweeps):
    from paper_2607_20704_amd import api
    L = api.L
    M = api.Multigrid(5, 5)
    g = torch.Generator(device="cuda")
    g.manual_seed(sweeps)
    f = torch.randn(M.f.shape, dtype=torch.float64, device="cuda", generator=g)
    phi = torch.randn(M.f.shape, dtype=torch.float64, device="cuda", generator=g)

    def run(phi, f, r):
        L.check(L.lib().rg_mg_vcycles(ctypes.byref(M.tree._desc), phi.data_ptr(), f.data_ptr(), r.data_ptr(), 5, 5, 2,
                                      2, sweeps, 1, torch.cuda.current_stream().cuda_stream))

    a, fa = phi.clone(), f.clone()
    run(a, fa, torch.empty_like(f))
    b, fb = phi.clone(), f.clone()
    run(b, fb, b if alias == "phi" else fb)
    assert torch.equal(a[M.fine], b[M.fine])
    assert torch.equal(fa[M.fine], f[M.fine]) and torch.equal(fb[M.fine], f[M.fine])
