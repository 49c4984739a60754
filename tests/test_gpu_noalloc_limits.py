"""asp_apply_noalloc at its limit: a request that counts as less than the fixed
array while the buffers of its batch take more (FP64, one layer) runs in passes,
bitwise equal to asp_apply, and a refusal says what the request counts as."""
import math
import re

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
asp = pytest.importorskip("paper_1504_04058_amd.asp")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

SCRATCH = 128 << 20


def counts_as(n, nrhs, rows):
    """One layer of n lines in blocks of `rows` rows, FP64: 16-byte entries."""
    slots, groups = -(-nrhs // 32) * 32, -(-nrhs // (1024 // rows))
    return 16 * (2 * nrhs * n * n + nrhs * n + 4 * n * slots + groups * n * 1024)


@pytest.mark.parametrize("n,gamma,rows,nrhs", [(24, 3, 32, 3600), (48, 5, 64, 900)])
def test_passes(n, gamma, rows, nrhs):
    print(f"noalloc passes n={n} nrhs={nrhs}", flush=True)
    c = workloads.velocity_random(n, 2, seed=2, width=3.0)
    b = n - 2 * (gamma - 1)
    assert counts_as(n, nrhs, rows) < SCRATCH - 4096 < 3 * 16 * nrhs * n * n + 16 * nrhs * rows * n
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    r = torch.randn(2 * nrhs, n * n, dtype=torch.complex128, device="cuda", generator=g)
    with asp.Plan(2, c, 2 * math.pi * (n + 1) / 8, n, b, gamma, prec=asp.ASP_PREC_FP64) as plan:
        assert len(plan.layers()[0]) == 1
        plan.factor()
        z = torch.full_like(r[:nrhs], float("nan"))
        plan.apply_noalloc(r[:nrhs].contiguous(), z)
        torch.cuda.synchronize()
        assert torch.equal(z, plan.apply(r[:nrhs].contiguous()))
        with pytest.raises(asp.AspError) as ei:
            plan.apply_noalloc(r, torch.empty_like(r))
    said = re.search(rf"{2 * nrhs} right-hand sides count as (\d+) bytes of work, .* {SCRATCH}-byte scratch", str(ei.value))
    # each of the five buffers starts at a multiple of 256 bytes
    assert said and 0 <= int(said.group(1)) - counts_as(n, 2 * nrhs, rows) < 5 * 256
