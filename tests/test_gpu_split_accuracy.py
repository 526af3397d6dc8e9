"""The split-FP16 pair sum is no less accurate than the FP32 matrix instructions
it stands in for: root mean square error of the coefficients against the FP64
form, for the default tile (split FP16) and a tile of 32 x 16 outputs (FP32
MFMAs), on grids of few and many rows with few and many partner columns (up to
the 8191 of a support of 4096, whose items are wider)."""
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,nw,batch", [(32, 64, 16), (32, 512, 8), (64, 2048, 4), (32, 4096, 2), (128, 128, 8)])
def test_error_not_above_the_fp32_instructions(nk, nw, batch):
    import torch
    import paper_2310_03979_amd as lib
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    wl = inp.small_grid(nk, nw, batch=batch, seed_base=21)
    print(f"[gpu] split accuracy {nk}x{nw}", flush=True)
    seeds = wl.seeds()
    err = {}
    p64 = lib.plan_from_workload(wl, "fp64")
    ref = torch.empty((batch,) + p64.coeff_shape, dtype=torch.complex128, device="cuda")
    lib.srm3_coefficients(p64, seeds, ref)
    for tile in (0, 1):
        plan = lib.plan_from_workload(wl, "fp32")
        lib.srm3_plan_set_algorithm(plan, "mfma")
        lib.srm3_plan_set_mfma_shape(plan, tile)
        C = torch.empty((batch,) + plan.coeff_shape, dtype=torch.complex64, device="cuda")
        lib.srm3_coefficients(plan, seeds, C)
        torch.cuda.synchronize()
        err[tile] = float((C.to(torch.complex128) - ref).norm() / ref.norm())
    print(f"relative error: split {err[0]:.3e}, FP32 instructions {err[1]:.3e}", flush=True)
    assert err[0] <= err[1]
