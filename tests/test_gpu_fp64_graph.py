"""The FP64 matrix-core pair sum from graphs, in its launch forms (chunk sums
apart, added in order, whole tiles): replays of srm3_generate and of an uneven
batch equal the eager results, with eager work and synchronisations between
them.  A capture without a call of that form before it allocates nothing (its
chunk sums are added in order then)."""
import pytest

import srm3_inputs as inp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    import paper_2310_03979_amd as p
    p.load()
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    return p


def _between(junk):
    import torch
    junk.mul_(1.0001).add_(0.5)
    torch.cuda.synchronize()


@pytest.mark.parametrize("nk,nw,batch,cold", [(32, 64, 1, False), (40, 300, 9, False), (8, 64, 70, False),
                                              (32, 64, 1, True)])
def test_generate_replays(lib, nk, nw, batch, cold):
    import torch
    wl = inp.small_grid(nk, nw, batch=batch, seed_base=5)
    print(f"[gpu] fp64 graph {nk}x{nw} {batch} {cold}", flush=True)
    seeds = wl.seeds()
    plan = lib.plan_from_workload(wl, "fp64")
    lib.srm3_plan_set_algorithm(plan, "mfma")
    shape = (batch,) + plan.field_shape
    ref = torch.empty(shape, dtype=torch.float64, device="cuda")
    lib.srm3_generate(plan, seeds, ref)
    if cold:   # a plan whose workspace another algorithm sized
        plan = lib.plan_from_workload(wl, "fp64")
        lib.srm3_plan_set_algorithm(plan, "kappa_fft")
        lib.srm3_generate(plan, seeds, torch.empty_like(ref))
        lib.srm3_plan_set_algorithm(plan, "mfma")
    out = torch.zeros_like(ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lib.srm3_generate(plan, seeds, out)
    junk = torch.randn(1 << 20, device="cuda")
    for _ in range(4):
        out.zero_()
        _between(junk)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def test_batch_replays(lib):
    import torch
    plans = []
    for nk, nw in ((33, 300), (16, 100), (64, 64)):
        wl = inp.small_grid(nk, nw)
        p = lib.plan_from_workload(wl, "fp64")
        lib.srm3_plan_set_algorithm(p, "mfma")
        plans.append(p)
    print("[gpu] fp64 batch graph", flush=True)
    reqs = [dict(plan=plans[i % 3], seed=i, out=torch.empty(plans[i % 3].field_shape, dtype=torch.float64, device="cuda"))
            for i in range(7)]
    batch = lib.Batch(reqs, flags=lib.SRM3_BATCH_GRAPH)
    junk = torch.randn(1 << 20, device="cuda")
    for k in range(3):
        seeds = [100 * k + i for i in range(7)]
        batch.run(seeds)
        torch.cuda.synchronize()
        for r, s in zip(reqs, seeds):
            one = torch.empty((1,) + r["plan"].field_shape, dtype=torch.float64, device="cuda")
            lib.srm3_generate(r["plan"], [s], one)
            torch.cuda.synchronize()
            assert torch.equal(r["out"], one[0]), (k, s)
        _between(junk)
