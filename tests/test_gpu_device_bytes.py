"""asp_device_bytes against what the allocator hands out: with its cache holding
every block that is given back, the cached bytes after a factorization and after a
solve are the planned ones."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
asp = pytest.importorskip("paper_1504_04058_amd.asp")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

CASES = [(2, 63, 12, 4, 5, {}), (2, 100, 5, 20, 17, {}), (3, 19, 5, 3, 3, {}),
         (3, 15, 4, 3, 17, dict(fact3d=asp.ASP_FACT3D_BLOCKS)), (3, 15, 4, 3, 2, dict(fact3d=asp.ASP_FACT3D_RECURSIVE))]


@pytest.mark.parametrize("prec", [asp.ASP_PREC_FP64, asp.ASP_PREC_FP32])
@pytest.mark.parametrize("dim,n,gamma,b,nrhs,opt", CASES)
def test_blocks(dim, n, gamma, b, nrhs, opt, prec):
    before = asp.asp_set_cache_limit(0)
    try:
        with asp.Plan(dim, torch.ones((n,) * dim, dtype=torch.float64).numpy(), 2 * math.pi * n / 8, n, b, gamma,
                      prec=prec, **opt) as plan:
            fac, work, ws = asp.asp_device_bytes(plan.handle, nrhs, 20)
            asp.asp_set_cache_limit(8 << 30)
            plan.factor()
            asp.asp_release_workspace(plan.handle)
            assert asp.asp_cached_bytes() == work
            asp.asp_set_cache_limit(0)
            asp.asp_set_cache_limit(8 << 30)
            f = torch.ones((nrhs, n ** dim), dtype=torch.complex128, device="cuda")
            plan.gmres(f, tol=1e-6, restart=20)
            assert asp.asp_cached_bytes() == 0
            asp.asp_release_workspace(plan.handle)
            assert asp.asp_cached_bytes() == ws
            asp.asp_set_cache_limit(0)
            asp.asp_set_cache_limit(8 << 30)
        # the factors, and the plan's tables
        assert fac <= asp.asp_cached_bytes() <= fac + (4 << 20)
    finally:
        asp.asp_set_cache_limit(before)
