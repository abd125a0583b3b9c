"""What the autotuner chose is what runs: the stage kernel at a height, or the
kernel that a batch takes by itself.  The tile count of the batch tells them
apart (63 x height tiles, or the 16 x 8 tiles of these small channels)."""
import json

import numpy as np
import pytest

import olb_inputs as I

pytestmark = pytest.mark.gpu

SIZES = ((70, 20), (40, 33), (129, 12))


def _olb():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    from paper_1702_01690_amd import olb
    return olb


def _cases(precision):
    cases = [I.channel(nx, ny, tw=0.8 * I.T_CRIT, seed=11) for nx, ny in SIZES]
    for c in cases:
        c.params["precision"] = precision
        c.params["rho_ref"] = I.N_CRIT
    return cases


def _tiles(width, height):
    return sum(-(-nx // width) * -(-ny // height) for nx, ny in SIZES)


def _f(batch, cases):
    for i, c in enumerate(cases):
        batch.set_fields(i, *c.fields)
    batch.step(5)
    return [batch.get_f(i) for i in range(len(cases))]


@pytest.mark.parametrize("precision", [0, 1])
def test_the_choice_is_what_runs(tmp_path, precision):
    olb = _olb()
    cases = _cases(precision)
    params = [c.params for c in cases]
    cache = tmp_path / "tune.json"
    b = olb.Batch(params)
    assert b.tiles() == (_tiles(16, 8), 8)
    want = _f(b, cases)
    b.autotune(trial_steps=2, cache_path=str(cache))
    data = json.loads(cache.read_text())
    (key, entry), = data.items()
    print(f"[autotune] precision={precision}: {entry}", flush=True)
    assert {"by8", "by16", "auto"} <= set(entry["ms_per_step"])
    assert b.tiles() == ((_tiles(16, 8), 8) if entry["auto"] else (_tiles(63, entry["by"]), entry["by"]))
    for auto, by in ((0, 16), (0, 8), (1, 8)) + (((0, 12),) if precision else ()):
        data[key].update(auto=auto, by=by)
        cache.write_text(json.dumps(data))
        other = olb.Batch(params)
        assert other.autotune(trial_steps=2, cache_path=str(cache)) == by
        assert other.tiles() == ((_tiles(16, 8), 8) if auto else (_tiles(63, by), by))
        for got, ref in zip(_f(other, cases), want):
            np.testing.assert_array_equal(got, ref)
        other.close()
    b.close()


def test_entries_of_a_search_over_heights_alone_are_left_alone(tmp_path):
    """Files from before there was more than one kernel name a height whatever
    ran: the search is made again and their entries stay as they are."""
    olb = _olb()
    cases = _cases(0)
    nodes = sum(nx * ny for nx, ny in SIZES)
    old = {f"fp64-walls-n{len(SIZES)}-nodes{nodes}-direct": {"by": 16, "strip": 4, "graph": 0, "ms_per_step": {"by16": 0.1}}}
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps(old))
    b = olb.Batch([c.params for c in cases])
    b.autotune(trial_steps=2, cache_path=str(cache))
    data = json.loads(cache.read_text())
    assert len(data) == 2 and all(data[k] == v for k, v in old.items())
    b.close()
