"""The benchmark times the kernels that a program gets: it chooses a tile height
only when it is asked to.  CPU only (the lattices are stand-ins that stop the
run before the first step)."""
import sys

import pytest

import bench
import olb_inputs as I
from paper_1702_01690_amd import olb


class _Stop(Exception):
    pass


class _Recorder:
    chosen = []
    stream = None

    def __init__(self, params, device=None):
        pass

    def set_tile(self, by):
        self.chosen.append(by)

    def set_fields(self, *args):
        raise _Stop

    def use_graph(self, steps):
        pass

    def set_base_temperature(self, *args):
        pass


@pytest.mark.parametrize("workload,options", [("wave2048", []), ("channels", []), ("channels", ["--sequential"])],
                         ids=["lattice", "batch", "sequential"])
def test_a_tile_height_is_chosen_on_request_only(monkeypatch, workload, options):
    cases = [I.channel(20, 12)] if workload == "channels" else [I.shear32()]
    monkeypatch.setattr(bench, "make_cases", lambda name: cases)
    monkeypatch.setattr(olb, "Lattice", _Recorder)
    monkeypatch.setattr(olb, "Batch", _Recorder)
    for extra, want in (([], []), (["--tile", "16"], [16])):
        monkeypatch.setattr(sys, "argv", ["bench.py", "--workload", workload, "--no-cpu"] + options + extra)
        monkeypatch.setattr(_Recorder, "chosen", [])
        with pytest.raises(_Stop):
            bench.main()
        assert _Recorder.chosen == want
