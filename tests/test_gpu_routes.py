"""Which kernel a lattice takes by itself.  The tests that compare those kernels
with the stage kernel would pass as well if the default were the stage kernel:
here every size they use is looked up by its workgroup count, which is another
for each kernel unless the lattice is smaller than a tile.  And the tile orders
of the kernels that have one."""
import numpy as np
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
    """One workgroup holds 2 to 192 nodes, 208 with the ghost rows of two walls;
    larger ones of a few hundred nodes a side take 16 x 8 tiles; 512 across, two
    64 x 8 tiles on each of 256 compute units instead of three 63 x 8."""
    if not kind.startswith("box") and 2 <= nx * ny <= 192 and (kind == "noisy" or nx * (ny + 6) <= 208):
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


def _steps(case, precision, strip, by=None):
    """f after four steps, at a tile order (None: the default) and a chosen
    height (None: none)."""
    olb = _olb()
    lat = olb.Lattice(dict(case.params, precision=precision, rho_ref=2.0))
    if by:
        lat.set_tile(by)
    if strip is not None:
        lat.set_tile_order(strip)
    lat.set_fields(*case.fields)
    lat.step(4)
    f = lat.get_f()
    lat.close()
    return f


@pytest.mark.parametrize("precision,by", [(0, 8), (0, 16), (1, 8), (1, 12), (1, 16)])
def test_stage_kernel_strips_visit_every_tile_once(precision, by):
    """150 nodes are three tile columns: strips of one, of two with a narrower
    last one, wider than the grid, and rows, on the stage kernel at each height
    (which a chosen height selects; the default of this size has no strips)."""
    case = _case("noisy", 150, 37)
    ref = _steps(case, precision, None)
    for strip in (0, 1, 2, 5, 64):
        np.testing.assert_array_equal(_steps(case, precision, strip, by), ref, err_msg=f"strip {strip}")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind,size", [("noisy", (512, 457)), ("half", (510, 470))], ids=["periodic", "half"])
def test_wide_kernel_strips_visit_every_tile_once(kind, size, precision):
    """Eight columns of 64 x 8 tiles: strips of one, of three with a narrower
    last one, of the whole grid, and rows."""
    case = _case(kind, *size)
    ref = _steps(case, precision, None, 8)
    for strip in (0, 1, 3, 8):
        np.testing.assert_array_equal(_steps(case, precision, strip), ref, err_msg=f"strip {strip}")


@pytest.mark.parametrize("precision", [0, 1])
def test_stage_kernel_strips_of_a_walled_batch(precision):
    olb = _olb()
    cases = [_case("channel", *size) for size in ((70, 20), (40, 33), (129, 12))]
    got = []
    for strip in (0, 1, 2):
        b = olb.Batch([dict(c.params, precision=precision, rho_ref=2.0) for c in cases])
        b.set_tile(8)
        b.set_tile_order(strip)
        for i, c in enumerate(cases):
            b.set_fields(i, *c.fields)
        b.step(5)
        got.append([b.get_f(i) for i in range(len(cases))])
        b.close()
    for other in got[1:]:
        for x, y in zip(got[0], other):
            np.testing.assert_array_equal(x, y)


def _batch_route(sizes, precision):
    """(workgroups, those of each kernel) of a periodic batch of these sizes."""
    olb = _olb()
    p = _case("noisy", 8, 8).params
    b = olb.Batch([dict(p, nx=nx, ny=ny, precision=precision, rho_ref=2.0) for nx, ny in sizes])
    got = b.tiles()[0]
    b.close()
    return got, {r: sum(_workgroups(r, nx, ny) for nx, ny in sizes) for r in ("split", "wide", "stage")}


@pytest.mark.parametrize("sizes,precision,route", [
    # three 16 x 8 tiles to one of 63 x 8, FP32 five to two: they win where the others
    # just start another round of one per compute unit, and lose in many rounds
    ([(40, 40)] * 110, 0, "split"), ([(40, 40)] * 600, 0, "stage"),
    ([(30, 40), (40, 40)] * 60, 1, "split"), ([(30, 40), (40, 40)] * 250, 1, "stage"),
    ([(30, 40)] * 600, 0, "split"), ([(30, 40)] * 600, 1, "split"),
    # 64 x 8 tiles: 3 rounds against 4, and 10 against 11 with hardly fewer in all
    ([(60, 320)] * 18 + [(64, 320)], 0, "wide"), ([(60, 320)] * 63 + [(64, 240)], 0, "stage"),
    ([(60, 320)] * 63 + [(64, 240)], 1, "stage"), ([(1024, 1024)], 0, "wide"), ([(1024, 1024)], 1, "wide"),
], ids=lambda v: f"{len(v)}x{v[0][0]}x{v[0][1]}" if isinstance(v, list) else str(v))
def test_routes_of_batches_with_many_tiles(sizes, precision, route):
    got, tiles = _batch_route(sizes, precision)
    assert got == tiles[route], (got, tiles)


@pytest.mark.parametrize("nx,ny,box,route", [(16, 700000, False, "split"), (30, 380000, True, "split"),
                                             (512, 22000, False, "wide")])
def test_routes_on_plane_storage(nx, ny, box, route):
    """Distribution arrays of more than 2^31 bytes are stored plane by plane: the
    thin ones still take 16 x 8 tiles, others 64 x 8, with the stage kernel's
    bits."""
    import torch
    olb = _olb()
    assert 25 * nx * (ny + 6) * 8 >= 2 ** 31
    p = dict(_case("box2" if box else "noisy", 8, 8).params, nx=nx, ny=ny)
    fields = torch.ones(4, ny, nx, dtype=torch.float64, device="cuda:0")
    fields[0] = 2.0 + 0.01 * torch.sin(torch.arange(nx * ny, device="cuda:0", dtype=torch.float64)).reshape(ny, nx)
    fields[1:3] = 0.0
    got = []
    for by in (None, 8):
        b = olb.Batch([p])
        torch.cuda.synchronize()          # the batch works on a stream of its own
        if by:
            b.set_tile(by)
        else:
            assert b.tiles()[0] == _workgroups(route, nx, ny)
        b.set_fields_device(0, fields)
        b.step(2)
        out = torch.empty_like(fields)
        torch.cuda.synchronize()
        b.moments_device(0, out)
        b.sync()
        got.append(out)
        b.close()
    assert torch.equal(*got) and torch.isfinite(got[0]).all()
    assert not torch.equal(got[0], fields)
