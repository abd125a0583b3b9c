"""Small lattices: the kernels that update them (16 x 8 tiles split by
velocity rows, wall ghosts formed in the tile; whole steps in one workgroup
for lattices of up to 192 nodes) and the 64 x 8 tiles of some larger ones
against the stage kernel, which a chosen tile height selects.  And the closure's gradients on small and ragged
lattices.  Every node's sums are taken in the same
order by both, so f, the moments and the wall densities agree to the bit."""
import numpy as np
import pytest

import olb_inputs as I

pytestmark = pytest.mark.gpu


def _olb():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    from paper_1702_01690_amd import olb
    return olb


def _noisy(nx, ny, seed=5):
    U = I.uniform(seed, 4 * nx * ny).reshape(4, ny, nx)
    p = dict(nx=nx, ny=ny, ds=1 / 64, dt=5e-4, tau=0.01, a=I.VDW_A, b=I.VDW_B, sigma=1e-4, bc_x=0, bc_y=0)
    return I.Case(f"noisy{nx}x{ny}", p, 2.0 * (1 + 0.02 * (2 * U[0] - 1)), 0.02 * (2 * U[1] - 1),
                  0.02 * (2 * U[2] - 1), 1.0 + 0.02 * (2 * U[3] - 1), 0)


# sizes at the edges of the 16 x 8 tiles: one node, one short, exact, one over,
# ragged in both directions, walls one to three rows past a tile's end
CASES = ([("noisy", s) for s in ((1, 1), (5, 3), (16, 8), (17, 9), (15, 7), (33, 16), (70, 37))]
         + [("channel", s) for s in ((1, 3), (3, 3), (16, 8), (33, 9), (40, 10), (17, 11), (67, 20))]
         + [("half", s) for s in ((5, 3), (16, 9), (40, 70))]
         + [("box0", s) for s in ((3, 12), (17, 8), (70, 37))]
         + [("box1", s) for s in ((3, 5), (16, 16), (35, 19))]
         + [("box2", s) for s in ((3, 4), (16, 8), (70, 13))]
         # one workgroup per lattice: 64, 128 and 192 nodes, ghost rows included
         # 80, 144 and 208 places; the last that fits each and the first that does not
         + [("noisy", s) for s in ((1, 60), (64, 1), (65, 1), (8, 16), (129, 1), (3, 64), (193, 1))]
         + [("channel", s) for s in ((8, 4), (1, 160), (1, 186), (1, 187), (2, 40), (23, 3), (24, 3))]
         + [("half", s) for s in ((1, 40), (16, 3), (7, 17))]
         # tiles of 64 x 8 where they put fewer on a CU: whole tiles across, a
         # cell over eight of 63, and the last tile short of both
         + [("noisy", s) for s in ((512, 457), (505, 483))]
         + [("channel", (512, 461)), ("half", (510, 470))])


def _case(kind, nx, ny):
    if kind == "noisy":
        return _noisy(nx, ny)
    if kind == "channel":
        return I.channel(nx, ny, seed=9, tw=0.8 * I.T_CRIT, uw=0.01)
    if kind == "half":
        return I.half_channel(nx, ny, seed=9, tw=0.8 * I.T_CRIT, uw=0.02)
    return I.box(nx, ny, seed=31, bc_y=int(kind[3]), uw=0.0 if kind == "box0" else 0.015)


def _run(case, precision, by, steps):
    olb = _olb()
    p = dict(case.params)
    p["precision"] = precision
    p["rho_ref"] = float(np.mean(case.n)) if precision else 1.0
    lat = olb.Lattice(p)
    if by:
        lat.set_tile(by)
    if precision:
        lat.set_base_temperature(float(np.mean(case.T)))
    lat.set_fields(*case.fields)
    out = []
    for k in steps:          # the carried fields pass from one call to the next
        lat.step(k)
        out += [lat.get_f(), *lat.moments()]
        if p["bc_y"]:
            out += lat.wall_density()
    lat.close()
    return out


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind,size", CASES, ids=lambda v: v if isinstance(v, str) else f"{v[0]}x{v[1]}")
def test_small_lattice_kernels_equal_the_stage_kernel(kind, size, precision):
    case = _case(kind, *size)
    print(f"[small] {case.name} precision={precision}", flush=True)
    for a, b in zip(_run(case, precision, None, (1, 4)), _run(case, precision, 8, (1, 4))):
        np.testing.assert_array_equal(a, b)


def test_batch_of_small_lattices_equals_the_stage_kernel():
    """Ragged walled instances in one batch: default kernels against a chosen
    tile height, and a chosen height at two tile orders (strips narrower than
    the tile grid)."""
    olb = _olb()
    cases = [I.channel(nx, ny, seed=20 + nx, tw=0.8 * I.T_CRIT) for nx, ny in ((150, 21), (3, 40), (17, 8))]
    got = []
    for by, strip in ((None, None), (8, 0), (16, 2)):
        b = olb.Batch([c.params for c in cases])
        if by:
            b.set_tile(by)
            b.set_tile_order(strip)
        for i, c in enumerate(cases):
            b.set_fields(i, *c.fields)
        b.step(5)
        got.append([(b.get_f(i), *b.wall_density(i)) for i in range(len(cases))])
        b.close()
    for other in got[1:]:
        for x, y in zip(got[0], other):
            for u, v in zip(x, y):
                np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("kind", ["waves", "columns"])
def test_resident_batch_steps_and_graphs(kind):
    """Batches of one-dimensional lattices: odd and long step counts (more than
    one launch holds) and graph replays give the stage kernel's bits."""
    olb = _olb()
    if kind == "waves":
        cases = [I.shear_wave(n, 0.3 * i, *m) for i, (n, m) in enumerate(
            ((20, (1.0, 0.0, 0.0, 0.0)), (60, (1.9327, 9 / 8, 1 / 3, 1e-4)), (33, (0.2397, 9 / 8, 1 / 3, 1e-4))))]
    else:
        cases = [I.planar_interface(tw, 0.2397, 1.9327, cells=c) for tw, c in ((0.8, 160), (0.85, 47), (0.9, 100))]
    got = []
    for by, graph in ((8, 0), (None, 0), (None, 4)):
        b = olb.Batch([c.params for c in cases])
        if by:
            b.set_tile(by)
        if graph:
            b.use_graph(graph)
        for i, c in enumerate(cases):
            b.set_fields(i, *c.fields)
        out = []
        for steps in (4, 3, 1, 260):
            b.step(steps)
            out += [b.get_f(i) for i in range(len(cases))]
            if kind == "columns":
                out += [w for i in range(len(cases)) for w in b.wall_density(i)]
        got.append(out)
        b.close()
    for other in got[1:]:
        for u, v in zip(got[0], other):
            np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("shape", [(5, 3), (8, 8), (9, 17), (130, 24), (7, 300), (300, 260)],
                         ids=lambda v: f"{v[0]}x{v[1]}")
def test_closure_gradients_at_tile_edges(shape):
    """The fused gradient kernel on lattices smaller than its 8 x 8 tile's
    halo, exact and ragged tiles, and more tiles than workgroups, against the
    oracle with the kernels' bf16 roundings.  What is left is FP32 summation
    order, which moves a bf16 rounding (2^-8) of one activation or gradient in
    some thousands: well below 5e-3 of a block's norm."""
    import torch
    from oracle import cnn
    olb = _olb()
    nx, ny = shape
    params = I.closure_params(seed=7)
    m = I.closure_moments(nx, ny, seed=21)
    norm = (m.mean(axis=(1, 2)), np.maximum(m.std(axis=(1, 2)), 1e-3), np.array([1e-3, 2e-4, 2e-4, 1e-4]))
    U = 2.0 * I.uniform(22, 4 * nx * ny).reshape(4, ny, nx) - 1.0
    ref = m + U * norm[2][:, None, None]
    c = olb.Closure(nx, ny)
    assert not c.get_params().any()          # zero until set
    c.set_norm(*norm)
    c.set_params(params)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda:0").contiguous()
    g, loss = c.gradients(dev(m), dev(ref))
    want_loss, want = cnn.loss_and_gradient(params, m, ref, norm, bf16_mirror=True)
    print(f"[closure] gradients {nx}x{ny}: loss {loss:.6e} oracle {want_loss:.6e}", flush=True)
    assert abs(loss - want_loss) <= 1e-4 * want_loss
    o = 0
    for name, block in cnn.BLOCKS:
        k = int(np.prod(block))
        e = np.linalg.norm(g[o:o + k] - want[o:o + k]) / np.linalg.norm(want[o:o + k])
        assert e < 5e-3, (name, e)
        o += k
    # a training step reports the same loss and steps along the same gradient
    assert c.train_step(dev(m), dev(ref), 1e-3) == loss
    step = (params - c.get_params()) / 1e-3
    far = np.abs(g) > 1e-3 * np.abs(g).max()
    np.testing.assert_allclose(step[far], np.sign(g[far]), atol=2e-3)


@pytest.mark.parametrize("factor", [2, 3, 4, 8])
@pytest.mark.parametrize("cells", [(1, 1), (65, 3)], ids=lambda v: f"{v[0]}x{v[1]}")
def test_restriction_factors(factor, cells):
    """Every factor with loads of its own and the general one, with rows that
    start on odd multiples of 8 bytes, against the oracle: sums of r^2 terms
    and a handful of roundings after them, each 2^-53 of the largest value."""
    import torch
    from oracle import cnn
    olb = _olb()
    nx, ny = factor * cells[0], factor * cells[1]
    m = I.closure_moments(nx, ny, seed=31, amplitude=0.05)
    buf = torch.zeros(4 * nx * ny + 1, dtype=torch.float64, device="cuda:0")
    fine = buf[1:]                            # 8 bytes past an aligned start
    fine.copy_(torch.tensor(m.ravel(), dtype=torch.float64))
    got = olb.restrict(fine, nx, ny, factor).cpu().numpy().reshape(4, cells[1], cells[0])
    want = cnn.restrict(m, factor)
    np.testing.assert_allclose(got, want, rtol=0, atol=(factor * factor + 16) * 2.0 ** -53 * 8 * np.abs(m).max())


@pytest.mark.parametrize("ny", [1118, 1119])
def test_moments_of_large_lattices(ny):
    """The last f that is read through the caches and the first that is read
    past them: the moments of f^eq are the fields it was formed from, up to
    the roundings of 25 terms and as many of their sums."""
    olb = _olb()
    case = _noisy(1200, ny)
    lat = olb.Lattice(case.params)
    lat.set_fields(*case.fields)
    tol = 50 * 2.0 ** -53 * 16 * np.abs(case.n).max()
    for got, want in zip(lat.moments(), case.fields):
        np.testing.assert_allclose(got.reshape(want.shape), want, rtol=0, atol=tol)
    lat.close()
