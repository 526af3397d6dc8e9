"""The FP64 matrix-core pair sum over its launch forms (whole tiles, chunks added
in order, chunk sums apart), its chunk sizes (32, 64 and 128 partner columns and
their remainders), tile shapes and idle row tiles: against the oracle, and the
same bits alone, in a batch of realizations, in an uneven batch and served.

Tolerance: every product and sum is FP64; at most 4e5 terms per line give a
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


CASES = [
    # nk, nw, W, tile shape
    (16, 140, 130, 0),    # chunks of 64, one remainder column; the second row tile idle
    (17, 20, 17, 1),      # 33 partners: a quarter of four columns and an empty one
    (33, 12, 9, 2),       # row groups of 16, the last of one row
    (49, 33, 33, 0),      # the last group's second row tile idle
    (64, 140, 129, 0),    # 257 partners in chunks of 64, 64 rows
    (48, 200, 129, 1),    # chunks of 128, 257 partners
    (20, 16, 1, 0),       # a single partner
    (3, 40, 40, 2),       # few rows (the algorithm chosen)
]


@pytest.mark.parametrize("case", CASES, ids=["%dx%dw%ds%d" % c for c in CASES])
def test_matches_oracle(lib, oracle_mod, case):
    import torch
    nk, nw, W, shape = case
    wl = inp.small_grid(nk, nw, support_w=W, batch=1, seed_base=12)
    print(f"[gpu] fp64 tiles {case}", flush=True)
    b2 = inp.random_b2_dense(W, 2, scale=0.3)
    beta = inp.random_beta_table(W, 3)
    bis = dict(kind="dense", b2=b2, beta=beta, beta_mode="table", support_w=W, cap=wl.cap)
    plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, "fp64")
    lib.srm3_plan_set_algorithm(plan, "mfma")
    lib.srm3_plan_set_mfma_shape(plan, shape)
    lib.srm3_workspace_fill(plan, 1, 0x7FF80000)
    C = torch.empty((1,) + plan.coeff_shape, dtype=torch.complex128, device="cuda")
    lib.srm3_coefficients(plan, wl.seeds(), C)
    torch.cuda.synchronize()
    P = oracle_mod.Problem(nk, nw, W, wl.d_kappa, wl.d_omega, wl.spectrum(), b2, beta, wl.cap)
    ref = P.coefficients(seed=int(wl.seeds()[0]))
    assert np.linalg.norm(C.cpu().numpy()[0] - ref) <= TOL * np.linalg.norm(ref)


@pytest.mark.parametrize("nk,nw,batch", [(8, 64, 70),     # whole tiles; alone: apart
                                         (16, 300, 24),   # whole tiles, chunks of 64; alone: apart
                                         (32, 64, 400),   # many tiles whole; some in order; alone: apart
                                         (33, 300, 12)])  # in order; alone: apart
def test_forms_agree(lib, nk, nw, batch):
    import torch
    wl = inp.small_grid(nk, nw, batch=batch, seed_base=31)
    print(f"[gpu] fp64 forms {nk}x{nw} {batch}", flush=True)
    plan = lib.plan_from_workload(wl, "fp64")
    lib.srm3_plan_set_algorithm(plan, "mfma")
    seeds = wl.seeds()
    shape = plan.field_shape
    lib.srm3_workspace_fill(plan, len(seeds), 0x7FF80000)
    many = torch.empty((len(seeds),) + shape, dtype=torch.float64, device="cuda")
    lib.srm3_generate(plan, seeds, many)
    for n in (1, 3, max(3, batch // 4)):
        some = torch.empty((n,) + shape, dtype=torch.float64, device="cuda")
        lib.srm3_workspace_fill(plan, n, 0x7FF80000)
        lib.srm3_generate(plan, seeds[:n], some)
        torch.cuda.synchronize()
        assert torch.equal(some, many[:n]), n
    reqs = [dict(plan=plan, seed=int(s), out=torch.empty(shape, dtype=torch.float64, device="cuda")) for s in seeds[:6]]
    lib.srm3_generate_uneven(reqs)
    torch.cuda.synchronize()
    for r, m in zip(reqs, many):
        assert torch.equal(r["out"], m)
    from paper_2310_03979_amd import serve
    for r in reqs:
        r["out"].fill_(float("nan"))
        r["b2_scale"] = 1.0
    server = lib.Server(precision="fp64", max_active=8, hbm_budget=1 << 30, pair_kernel="mfma")
    serve.replay(server, reqs, [0.0] * len(reqs))
    torch.cuda.synchronize()
    for r, m in zip(reqs, many):
        assert torch.equal(r["out"], m)
