"""The FP64 matrix-core pair sum where one call has more work items than 32 bits
count (one kappa row, 4096 frequencies, 8200 realizations: 256 column tiles of
1024 chunks each): the call equals its realizations alone, bitwise."""
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu


def test_more_items_than_32_bits_count():
    import torch
    import paper_2310_03979_amd as lib
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    wl = inp.small_grid(1, 4096, batch=8200, seed_base=5)
    print("[gpu] fp64 queue 1x4096 8200", flush=True)
    plan = lib.plan_from_workload(wl, "fp64")
    lib.srm3_plan_set_algorithm(plan, "mfma")
    seeds = wl.seeds()
    many = torch.empty((len(seeds),) + plan.coeff_shape, dtype=torch.complex128, device="cuda")
    lib.srm3_coefficients(plan, seeds, many)
    one = torch.empty((1,) + plan.coeff_shape, dtype=torch.complex128, device="cuda")
    for r in (0, 4097, 8199):
        lib.srm3_coefficients(plan, [int(seeds[r])], one)
        torch.cuda.synchronize()
        assert torch.isfinite(torch.view_as_real(one)).all()
        assert torch.equal(one[0], many[r]), r
