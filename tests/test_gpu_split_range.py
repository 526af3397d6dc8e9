"""Which FP32 plans the split-FP16 pair sum may take: pair weights near the ends
of FP32 stay with the FP32 forms (the split form scales them by 2^-10 and its
sums by 2^10), against the FP64 oracle at the FP32 forms' tolerance (coefficients
2e-5, as elsewhere in the suite)."""
import numpy as np
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu

TOL = 2e-5


@pytest.fixture(scope="module")
def lib():
    import torch
    import paper_2310_03979_amd as p
    p.load()
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    return p


@pytest.mark.parametrize("algorithm", ["direct", "mfma"])
@pytest.mark.parametrize("weight,line_c", [(2e34, None), (1e-36, 1e35)])
def test_weights_near_the_ends_of_fp32(lib, oracle_mod, algorithm, weight, line_c):
    """Weights of 2e34 (sums near 1e36: their 2^10-fold overflows), and of 1e-36
    brought back by line factors (their 2^-10-fold is subnormal)."""
    import torch
    nk, nw, W = 34, 30, 30
    wl = inp.small_grid(nk, nw, support_w=W, batch=1, seed_base=77)
    b2 = inp.random_b2_dense(W, 4, scale=0.2) * weight ** 2
    print(f"[gpu] split range {algorithm} {weight}", flush=True)
    bis = dict(kind="dense", b2=b2, beta_mode="seeded", beta_seed=11, support_w=W, cap=0.9)
    kw = {}
    if line_c is not None:
        bis["line_c"] = kw["line_c"] = np.full((nk, 2 * nw - 1), line_c)
    plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, "fp32")
    lib.srm3_plan_set_algorithm(plan, algorithm)
    C = torch.empty((1,) + plan.coeff_shape, dtype=torch.complex64, device="cuda")
    lib.srm3_coefficients(plan, [5], C)
    torch.cuda.synchronize()
    C = C.cpu().numpy().astype(np.complex128)[0]
    P = oracle_mod.Problem(nk, nw, W, wl.d_kappa, wl.d_omega, wl.spectrum(), b2, oracle_mod.biphase(W, 11), 0.9, **kw)
    ref = P.coefficients(seed=5)
    assert np.isfinite(C).all()
    assert np.linalg.norm(C - ref) <= TOL * np.linalg.norm(ref)
