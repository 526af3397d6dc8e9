"""The uneven-batch autotuner and the form of the pair sum: a choice cached for
the same grids in another form (plans whose factors keep them off the split-FP16
form, or a cache written before there was one) does not reach a batch, and a
batch whose launches have nothing to choose neither reads nor writes the cache."""
import numpy as np
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


def _batch(lib, nk, precision, line_r=None, algorithm="mfma"):
    import torch
    wl = inp.small_grid(nk, 50)
    bis = dict(kind="dense", b2=inp.random_b2_dense(50, 4, scale=0.2), beta_mode="seeded", beta_seed=11, support_w=50, cap=0.9)
    if line_r is not None:
        bis["line_r"] = np.full((nk, 99), line_r)
    plan = lib.srm3_plan(wl.grid_dict(), wl.spectrum(), bis, precision)
    lib.srm3_plan_set_algorithm(plan, algorithm)
    reqs = [dict(plan=plan, seed=7 + i, out=torch.empty(plan.field_shape, dtype=plan.real_dtype, device="cuda"))
            for i in range(3)]
    return lib.Batch(reqs, flags=lib.SRM3_BATCH_AUTOTUNE)


def test_choices_of_another_form_are_not_taken(lib, tmp_path, monkeypatch):
    import torch
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("SRM3_TUNE_CACHE", str(path))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # as an earlier library wrote it: the same grids, a tile of 32 x 16
    old = "".join(f"fp32;mfma;cu{cus};{nk}x50w50*3 8 3 1\n" for nk in (34, 24))
    path.write_text(old)
    print("[gpu] tune forms", flush=True)
    split = _batch(lib, 34, "fp32")
    split.run()
    assert split.info()["mfma_shape"] == 0 and path.read_text() == old
    mfma = _batch(lib, 34, "fp32", line_r=100.0)       # factors off the split form: tuned, under a signature of its own
    mfma.run()
    lines = path.read_text().splitlines()
    assert len(lines) == 3 and "/mfma" in lines[2] and lines[2].startswith(f"fp32;mfma;cu{cus};34x50w50/mfma*3 ")
    # its choice, had it been another tile, stays its own
    path.write_text(old + lines[2].rsplit(" ", 1)[0] + " 1\n")
    again, split = _batch(lib, 34, "fp32", line_r=100.0), _batch(lib, 34, "fp32")
    again.run()
    split.run()
    assert again.info()["mfma_shape"] == 1 and split.info()["mfma_shape"] == 0
    f64 = _batch(lib, 34, "fp64")
    f64.run()
    assert "fp64;mfma" in path.read_text()
    before = path.read_text()
    f64d = _batch(lib, 34, "fp64", algorithm="direct")
    f64d.run()
    torch.cuda.synchronize()
    assert path.read_text() == before
