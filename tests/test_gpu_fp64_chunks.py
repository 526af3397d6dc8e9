"""The FP64 matrix-core pair sum in chunks of partner columns (the default
algorithm from 16 rows on, and SRM3_ALGO_MFMA): against the oracle at chunk
edges and remainders, and the same sums however the chunks are run -- apart
(small calls), added in order (large ones), or one after the other (batches).

Tolerance: every product and sum is FP64; at most 2e5 terms per line give a
root-mean-square rounding far below 1e-12."""
import numpy as np
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu

TOL = 1e-12


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
    C = torch.empty((len(seeds),) + plan.coeff_shape, dtype=torch.complex128, device="cuda")
    lib.srm3_coefficients(plan, seeds, C)
    torch.cuda.synchronize()
    return C


CASES = [
    # nk, nw, W
    (16, 5, 4),       # one chunk, the first grid off the vector kernel
    (15, 30, 30),     # the vector kernel (default algorithm)
    (17, 5, 5),       # nine partners: a chunk of eight and one more
    (33, 70, 40),     # two row groups
    (40, 300, 270),   # chunks of 32
    (64, 129, 16),    # 31 partners, columns without any
]


@pytest.mark.parametrize("algorithm", ["direct", "mfma"])
@pytest.mark.parametrize("case", CASES, ids=[f"{a}x{b}w{c}" for a, b, c in CASES])
def test_matches_oracle_at_chunk_edges(lib, oracle_mod, case, algorithm):
    nk, nw, W = case
    wl = inp.small_grid(nk, nw, support_w=W, batch=1, seed_base=12)
    print(f"[gpu] fp64 chunks {case} {algorithm}", flush=True)
    b2 = inp.random_b2_dense(W, 2, scale=0.3)
    beta = inp.random_beta_table(W, 3)
    bis = dict(kind="dense", b2=b2, beta=beta, beta_mode="table", support_w=W, cap=wl.cap)
    plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, "fp64")
    lib.srm3_plan_set_algorithm(plan, algorithm)
    C = _coeffs(lib, plan, wl.seeds()).cpu().numpy()[0]
    P = oracle_mod.Problem(nk, nw, W, wl.d_kappa, wl.d_omega, wl.spectrum(), b2, beta, wl.cap)
    ref = P.coefficients(seed=int(wl.seeds()[0]))
    assert np.linalg.norm(C - ref) <= TOL * np.linalg.norm(ref)


@pytest.mark.parametrize("algorithm", ["direct", "mfma"])
@pytest.mark.parametrize("grid", [(20, 60), (40, 300)])
def test_chunks_apart_in_order_and_in_a_batch_agree(lib, grid, algorithm):
    import torch
    wl = inp.small_grid(*grid, batch=64 if grid[0] == 20 else 9, seed_base=31)
    print(f"[gpu] fp64 chunks {grid} {algorithm} runs", flush=True)
    plan = lib.plan_from_workload(wl, "fp64")
    lib.srm3_plan_set_algorithm(plan, algorithm)
    seeds = wl.seeds()
    shape = plan.field_shape
    lib.srm3_workspace_fill(plan, len(seeds), 0x7FF80000)
    many = torch.empty((len(seeds),) + shape, dtype=torch.float64, device="cuda")
    lib.srm3_generate(plan, seeds, many)           # too many for the separate sums: added in order
    one = torch.empty((1,) + shape, dtype=torch.float64, device="cuda")
    lib.srm3_generate(plan, seeds[3:4], one)       # apart
    assert torch.equal(one[0], many[3])
    reqs = [dict(plan=plan, seed=int(s), out=torch.empty(shape, dtype=torch.float64, device="cuda")) for s in seeds[:5]]
    lib.srm3_generate_uneven(reqs)                 # one after the other
    torch.cuda.synchronize()
    for r, m in zip(reqs, many):
        assert torch.equal(r["out"], m)
