"""The FP32 forms of the direct pair sum that plans with wide partner factors
run (vector ALUs and FP32 matrix instructions; the split-FP16 form takes the
others): several row groups, ragged columns and truncated support against the
FP64 oracle, one realization and several, in an uneven batch and served.  Which
form ran shows in the bits: vector and matrix sums round differently, while the
two algorithms of a plan within the range are the same split form.

Tolerance: the suite's for FP32 coefficients, relative L2 of 2e-5."""
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


def _factors(shape, lo, hi, seed=3):
    """Log-uniform over [lo, hi], both ends among them."""
    r = np.exp(np.random.default_rng(seed).uniform(np.log(lo), np.log(hi), size=shape))
    r.flat[0], r.flat[-1] = lo, hi
    return r


def _plan(lib, nk, nw, W, r, algorithm):
    wl = inp.small_grid(nk, nw, support_w=W, batch=3, seed_base=640)
    bis = dict(kind="dense", b2=inp.random_b2_dense(W, 4, scale=0.2), beta_mode="seeded", beta_seed=11, support_w=W, cap=0.9,
               line_r=r)
    plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, "fp32")
    lib.srm3_plan_set_algorithm(plan, algorithm)
    return wl, plan


def _coeffs(lib, plan, seeds):
    import torch
    C = torch.empty((len(seeds),) + plan.coeff_shape, dtype=torch.complex64, device="cuda")
    lib.srm3_coefficients(plan, seeds, C)
    torch.cuda.synchronize()
    return C


CASES = [
    # nk, nw, W, factors, whether they keep the plan off the split form
    (34, 30, 30, (0.01, 1.0), True),
    (70, 33, 17, (1.0, 40.0), True),        # 40^2 products, row groups of 32 with a ragged last
    (100, 75, 75, (0.5, 33.0), True),       # just above the upper bound
    (65, 140, 40, (1.0, 100.0), True),      # 100 x 2^10 is past FP16's largest number
    (40, 300, 300, (0.01, 2.0), True),      # many partner steps
    (66, 70, 50, (1.0 / 64, 32.0), False),  # both bounds in one plan
]


@pytest.mark.parametrize("case", CASES, ids=["%dx%dw%d_%g_%g" % (c[:3] + c[3]) for c in CASES])
def test_matches_oracle_and_the_expected_form_ran(lib, oracle_mod, case):
    import torch
    nk, nw, W, (lo, hi), wide = case
    r = _factors((nk, 2 * nw - 1), lo, hi)
    print(f"[gpu] wide factors {case}", flush=True)
    C = {}
    for algorithm in ("direct", "mfma"):
        wl, plan = _plan(lib, nk, nw, W, r, algorithm)
        lib.srm3_workspace_fill(plan, 3, 0x7FC00000)
        C[algorithm] = _coeffs(lib, plan, wl.seeds())
        lib.srm3_workspace_fill(plan, 1, 0x7FC00000)
        assert torch.equal(_coeffs(lib, plan, [int(wl.seeds()[1])])[0], C[algorithm][1])
    assert torch.equal(C["direct"], C["mfma"]) is not wide
    P = oracle_mod.Problem(nk, nw, W, wl.d_kappa, wl.d_omega, wl.spectrum(), inp.random_b2_dense(W, 4, scale=0.2),
                           oracle_mod.biphase(W, 11), 0.9, line_r=r)
    ref = P.coefficients(seed=int(wl.seeds()[0]))
    for algorithm, c in C.items():
        got = c[0].cpu().numpy().astype(np.complex128)
        assert np.linalg.norm(got - ref) <= TOL * np.linalg.norm(ref), algorithm


@pytest.mark.parametrize("algorithm", ["direct", "mfma"])
def test_batched_and_served_beside_split_plans(lib, algorithm):
    import torch
    from paper_2310_03979_amd import serve
    plans = []
    for nk, nw, W, (lo, hi), _ in CASES[1:]:
        plans.append(_plan(lib, nk, nw, W, _factors((nk, 2 * nw - 1), lo, hi), algorithm)[1])
    print(f"[gpu] wide factors batch {algorithm}", flush=True)
    reqs, singles = [], []
    for i in range(7):
        p = plans[i % len(plans)]
        reqs.append(dict(plan=p, seed=700 + i, out=torch.empty(p.field_shape, dtype=torch.float32, device="cuda")))
        one = torch.empty((1,) + p.field_shape, dtype=torch.float32, device="cuda")
        lib.srm3_generate(p, [700 + i], one)
        singles.append(one[0])
    lib.srm3_generate_uneven(reqs)
    torch.cuda.synchronize()
    for r, s in zip(reqs, singles):
        assert torch.equal(r["out"], s)
        r["out"].fill_(float("nan"))
        r["b2_scale"] = 1.0
    # served: as by a server alone, bitwise (its vector items have 16 rows per
    # wave, a plan's 8: single generations round differently there)
    server = lib.Server(precision="fp32", max_active=8, hbm_budget=1 << 30, pair_kernel=algorithm)
    serve.replay(server, reqs, [0.0] * len(reqs))
    for r, s in zip(reqs, singles):
        alone = dict(r, out=torch.empty_like(r["out"]))
        one = lib.Server(precision="fp32", max_active=1, hbm_budget=1 << 30, pair_kernel=algorithm)
        serve.replay(one, [alone], [0.0])
        torch.cuda.synchronize()
        assert torch.equal(r["out"], alone["out"])
        assert float((r["out"] - s).norm() / s.norm()) <= TOL
