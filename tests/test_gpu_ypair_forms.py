"""The two forms of the FP32 frequency autoconvolution (the uniform operand
through scalar loads for large launches, in LDS for small ones) sum alike: a
realization of a launch past the line between them equals itself alone,
bitwise, on a grid with ragged row and column tiles."""
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,nw,W,batch", [(32, 100, 100, 520), (9, 70, 41, 3000)])
def test_large_and_small_launches_agree(nk, nw, W, batch):
    import torch
    import paper_2310_03979_amd as lib
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    wl = inp.small_grid(nk, nw, support_w=W, batch=batch, seed_base=4)
    print(f"[gpu] ypair forms {nk}x{nw} {batch}", flush=True)
    plan = lib.plan_from_workload(wl, "fp32")
    lib.srm3_plan_set_algorithm(plan, "kappa_fft")
    seeds = wl.seeds()
    many = torch.empty((batch,) + plan.coeff_shape, dtype=torch.complex64, device="cuda")
    lib.srm3_coefficients(plan, seeds, many)
    one = torch.empty((1,) + plan.coeff_shape, dtype=torch.complex64, device="cuda")
    for r in (0, batch - 1):
        lib.srm3_coefficients(plan, [int(seeds[r])], one)
        torch.cuda.synchronize()
        assert torch.equal(one[0], many[r])
