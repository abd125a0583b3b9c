"""Which kernel a lattice takes by itself.  The tests that compare those kernels
with the stage kernel would pass as well if the default were the stage kernel:
here every size they use is looked up by its workgroup count, which is another
for each kernel unless the lattice is smaller than a tile."""
import pytest

from test_gpu_small import CASES, _case

pytestmark = pytest.mark.gpu


def _olb():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    from paper_1702_01690_amd import olb
    return olb


def _workgroups(route, nx, ny):
    if route == "resident":
        return 1
    width = {"split": 16, "wide": 64, "stage": 63}[route]
    return -(-nx // width) * -(-ny // 8)


def _expected(kind, nx, ny):
    """One workgroup holds 192 nodes, 208 with the ghost rows of two walls;
    larger ones of a few hundred nodes a side take 16 x 8 tiles; 512 across, two
    64 x 8 tiles on each of 256 compute units instead of three 63 x 8."""
    if not kind.startswith("box") and nx * ny <= 192 and (kind == "noisy" or nx * (ny + 6) <= 208):
        return "resident"
    return "wide" if nx > 500 else "split"


@pytest.mark.parametrize("precision", [0, 1])
def test_small_lattices_take_the_kernels_made_for_them(precision):
    import torch
    olb = _olb()
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    told_apart = {}
    for kind, (nx, ny) in CASES + [("noisy", (448, 448)), ("noisy", (192, 1)), ("channel", (26, 3))]:
        p = dict(_case(kind, nx, ny).params)
        p["precision"], p["rho_ref"] = precision, 2.0
        b = olb.Batch([p])
        route = "stage" if (nx, ny) == (448, 448) else _expected(kind, nx, ny)
        assert b.tiles() == (_workgroups(route, nx, ny), 8), (kind, nx, ny, route)
        if all(_workgroups(route, nx, ny) != _workgroups(r, nx, ny)
               for r in ("resident", "split", "wide", "stage") if r != route):
            told_apart[route] = told_apart.get(route, 0) + 1
        b.set_tile(16)
        assert b.tiles() == (-(-nx // 63) * -(-ny // 16), 16)
        b.close()
    print(f"[routes] precision={precision}: told apart {told_apart}", flush=True)
    assert told_apart["resident"] >= 8 and told_apart["split"] >= 3 and told_apart["wide"] >= 2


def test_a_batch_held_in_workgroups_counts_its_instances():
    """Thirteen half channels of 1 x 160 nodes, one workgroup each; with one that
    does not fit among them they take tiles, all of them."""
    olb = _olb()
    p = _case("half", 1, 40).params
    columns = [dict(p, ny=160)] * 13
    b = olb.Batch(columns)
    assert b.tiles() == (13, 8)
    b.close()
    b = olb.Batch(columns + [dict(p, nx=2, ny=160)])
    assert b.tiles() == (14 * 20, 8)
    b.close()
