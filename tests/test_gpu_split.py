"""The FP32 matrix-core pair sum in split FP16 against the FP64 oracle at the
edges of its tiles: row tiles of 64, 128 and 256 lines and their remainders,
several row tiles, column tiles cut by the grid, truncated support, work items
of one and several partner chunks, and a call whose realizations share the
launch with others.

Tolerance: a product drops less than 2^-23 of its factors (the split's low
times low part and its last bit), the weights and phases are rounded to 24
bits, sums run over at most 64 columns in FP32 and then over at most 32
chunks; the root mean square over a realization stays below 8 x 2^-23."""
import numpy as np
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu

TOL = 8 * 2.0 ** -23


@pytest.fixture(scope="module")
def lib():
    import torch
    import paper_2310_03979_amd as p
    p.load()
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    return p


def _coeffs(lib, plan, seeds):
    import torch
    C = torch.empty((len(seeds),) + plan.coeff_shape, dtype=torch.complex64, device="cuda")
    lib.srm3_coefficients(plan, seeds, C)
    torch.cuda.synchronize()
    return C


CASES = [
    # nk, nw, W
    (32, 40, 40),      # smallest grid of the split form
    (33, 70, 21),      # odd rows
    (64, 129, 129),    # one full tile of 64 rows, columns cut at a tile's first
    (65, 34, 34),      # the 128-row tile, one row past 64
    (128, 65, 50),     # full
    (129, 18, 18),     # the 256-row tile, one row past 128
    (200, 20, 7),      # row tiles of uneven number
    (256, 17, 17),     # full, one column past a tile
    (257, 9, 9),       # a second tile of one row (two passes)
    (300, 12, 12),     # a ragged second tile
    (520, 6, 6),       # three tiles
    (40, 300, 300),    # several partner chunks per tile
]


@pytest.mark.parametrize("case", CASES, ids=[f"{a}x{b}w{c}" for a, b, c in CASES])
def test_matches_oracle_at_tile_edges(lib, oracle_mod, case):
    nk, nw, W = case
    wl = inp.small_grid(nk, nw, support_w=W, batch=2, seed_base=640)
    print(f"[gpu] split {case}", flush=True)
    b2 = inp.random_b2_dense(W, 9, scale=0.3)
    beta = inp.random_beta_table(W, 10)
    bis = dict(kind="dense", b2=b2, beta=beta, beta_mode="table", support_w=W, cap=wl.cap)
    plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, "fp32")
    lib.srm3_plan_set_algorithm(plan, "mfma")
    C = _coeffs(lib, plan, wl.seeds()).cpu().numpy().astype(np.complex128)
    P = oracle_mod.Problem(nk, nw, W, wl.d_kappa, wl.d_omega, wl.spectrum(), b2, beta, wl.cap)
    for r, s in enumerate(wl.seeds()):
        ref = P.coefficients(seed=int(s))
        assert np.linalg.norm(C[r] - ref) <= TOL * np.linalg.norm(ref), r


@pytest.mark.parametrize("nk", [64, 100, 300])
def test_alone_equals_in_a_batch_and_poisoned(lib, nk):
    """One realization equals itself among others, bitwise, also from a
    workspace filled with NaN."""
    import torch
    wl = inp.small_grid(nk, 90, support_w=80, batch=7, seed_base=50)
    plan = lib.plan_from_workload(wl, "fp32")
    lib.srm3_plan_set_algorithm(plan, "mfma")
    seeds = wl.seeds()
    print(f"[gpu] split alone {nk}", flush=True)
    lib.srm3_workspace_fill(plan, len(seeds), 0x7FC00000)
    many = _coeffs(lib, plan, seeds)
    assert torch.isfinite(torch.view_as_real(many)).all()
    for r in (0, 6):
        lib.srm3_workspace_fill(plan, 1, 0x7FC00000)
        assert torch.equal(_coeffs(lib, plan, [int(seeds[r])])[0], many[r])


@pytest.mark.parametrize("algorithm", ["direct", "mfma"])
@pytest.mark.parametrize("factor", [1.0, 2.0 ** -6, 32.0, 2.0 ** -7])
def test_line_factors_at_the_bounds(lib, oracle_mod, algorithm, factor):
    """Partner factors spread over two octaves at both ends of the range the
    split form takes (and past its lower end, where the FP32 forms run):
    coefficients against the oracle."""
    nk, nw, W = 34, 30, 30
    wl = inp.small_grid(nk, nw, support_w=W, batch=1, seed_base=77)
    rng = np.random.default_rng(3)
    r = factor * 2.0 ** (rng.uniform(0.0, 2.0, size=(nk, 2 * nw - 1)) * (-1 if factor > 1 else 1))
    b2 = inp.random_b2_dense(W, 4, scale=0.2)
    print(f"[gpu] split factors {algorithm} {factor}", flush=True)
    bis = dict(kind="dense", b2=b2, beta_mode="seeded", beta_seed=11, support_w=W, cap=0.9, line_r=r)
    plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, "fp32")
    lib.srm3_plan_set_algorithm(plan, algorithm)
    C = _coeffs(lib, plan, [5]).cpu().numpy().astype(np.complex128)[0]
    P = oracle_mod.Problem(nk, nw, W, wl.d_kappa, wl.d_omega, wl.spectrum(), b2, oracle_mod.biphase(W, 11), 0.9, line_r=r)
    ref = P.coefficients(seed=5)
    assert np.linalg.norm(C - ref) <= TOL * np.linalg.norm(ref)
