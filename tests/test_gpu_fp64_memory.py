"""FP64 plans keep partial pair sums beside the workspace only where their pair
sum uses them, and no more than it uses: device memory that the first
generation of several plans takes, against the workspace they report."""
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu

MB = 1 << 20
GRAIN = 2 * MB   # of a device allocation, of which a plan makes up to three


@pytest.mark.parametrize("nk,nw,algorithm,extra", [(32, 64, "kappa_fft", 0), (8, 64, "direct", 0), (1, 100, "direct", 0),
                                                   (32, 64, "direct", 2 * MB)])
def test_memory_beside_the_workspace(nk, nw, algorithm, extra):
    import torch
    import paper_2310_03979_amd as lib
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    wl = inp.small_grid(nk, nw, batch=1, seed_base=3)
    print(f"[gpu] fp64 memory {nk}x{nw} {algorithm}", flush=True)
    n = 10
    plans = [lib.plan_from_workload(wl, "fp64") for _ in range(n + 1)]
    for p in plans:
        lib.srm3_plan_set_algorithm(p, algorithm)
    out = torch.empty((1,) + plans[0].field_shape, dtype=torch.float64, device="cuda")
    lib.srm3_generate(plans[n], [1], out)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for p in plans[:n]:
        lib.srm3_generate(p, [1], out)
    torch.cuda.synchronize()
    taken = (free0 - torch.cuda.mem_get_info()[0]) / n
    assert taken <= lib.srm3_workspace_bytes(plans[0], 1) + extra + 3 * GRAIN, taken / MB
