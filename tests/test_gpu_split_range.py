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


@pytest.mark.parametrize("nk,nw,same", [(32, 23, False),   # vector ALUs and FP32 MFMAs
                                        (32, 24, False),   # split and FP32 MFMAs
                                        (32, 50, False),
                                        (32, 52, True),    # split both
                                        (64, 6, False), (100, 3, True)])
def test_small_grids_at_the_lines_between_the_forms(lib, oracle_mod, nk, nw, same):
    """The smallest grids stay with the FP32 forms (the default algorithm's line
    lies below that of the matrix cores'): against the oracle on both sides, the
    form told by the bits of the two algorithms."""
    import torch
    wl = inp.small_grid(nk, nw, batch=2, seed_base=9)
    print(f"[gpu] split lines {nk}x{nw}", flush=True)
    b2 = inp.random_b2_dense(nw, 9, scale=0.3)
    beta = inp.random_beta_table(nw, 10)
    bis = dict(kind="dense", b2=b2, beta=beta, beta_mode="table", support_w=nw, cap=wl.cap)
    P = oracle_mod.Problem(nk, nw, nw, wl.d_kappa, wl.d_omega, wl.spectrum(), b2, beta, wl.cap)
    ref = P.coefficients(seed=int(wl.seeds()[1]))
    C = {}
    for algorithm in ("direct", "mfma"):
        plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, "fp32")
        lib.srm3_plan_set_algorithm(plan, algorithm)
        c = torch.empty((2,) + plan.coeff_shape, dtype=torch.complex64, device="cuda")
        lib.srm3_coefficients(plan, wl.seeds(), c)
        torch.cuda.synchronize()
        C[algorithm] = c
        got = c[1].cpu().numpy().astype(np.complex128)
        assert np.linalg.norm(got - ref) <= TOL * np.linalg.norm(ref), algorithm
    assert torch.equal(C["direct"], C["mfma"]) is same
