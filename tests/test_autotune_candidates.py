"""The autotuner measures the untuned configuration too, so that its choice is never
slower than none (the step times are made up here: no GPU)."""
import pytest

from paper_2311_11322_amd import dem, serve
from paper_2311_11322_amd import workloads as W


@pytest.mark.parametrize("prec", [dem.PREC_FP64, dem.PREC_FP32_FORCE])
@pytest.mark.parametrize("G", [0.0, 1.0])
def test_untuned_configuration_is_a_candidate(monkeypatch, prec, G):
    asked = []

    def run_batch(workloads, steps, precision, tuning=None, warmup=1):
        asked.append(tuning)
        return {"ms_per_step": 1.0 if tuning == (0, 1.0) else 2.0, "sims": []}

    monkeypatch.setattr(serve, "run_batch", run_batch)
    w = W.periodic_box(seed=1, n_agg=4)
    w.params["G"] = G
    out = serve.autotune([w], prec, cache={})
    assert (out["gravity_tile"], out["cell_scale"]) == (0, 1.0)
    sizes = dem.gravity_tiles(prec) if G else [0]
    assert len(out["candidates"]) == len(asked) == 4 * len(sizes)
    # given sizes are taken as they are
    given = serve.autotune([w], prec, tiles=[256, 512], cache={})
    assert {c["gravity_tile"] for c in given["candidates"]} == ({256, 512} if G else {256})
