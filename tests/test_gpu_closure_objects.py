"""Closure objects beside other work: the host buffers through which gradients
and losses come back outlive the objects, so that neither freeing one waits
for other streams nor two threads meet in one."""
import threading

import numpy as np
import pytest

import olb_inputs as I

pytestmark = pytest.mark.gpu


def _olb():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    from paper_1702_01690_amd import olb
    return torch, olb


def _pair(torch, nx, ny, seed):
    m = I.closure_moments(nx, ny, seed=seed)
    norm = (m.mean(axis=(1, 2)), np.maximum(m.std(axis=(1, 2)), 1e-3), np.array([1e-3, 2e-4, 2e-4, 1e-4]))
    U = 2.0 * I.uniform(seed + 1, 4 * nx * ny).reshape(4, ny, nx) - 1.0
    dev = lambda a: torch.tensor(a.ravel(), dtype=torch.float64, device="cuda:0")
    return norm, dev(m), dev(m + U * norm[2][:, None, None])


def test_freeing_an_object_waits_for_no_other_stream():
    """A tenth of a second of steps is queued on another stream when the object
    goes; they are still running after it has gone."""
    torch, olb = _olb()
    norm, m, ref = _pair(torch, 40, 24, 3)
    c = olb.Closure(40, 24)
    c.set_norm(*norm)
    c.set_params(I.closure_params(seed=7))
    c.gradients(m, ref)
    nx, ny = 2048, 1024
    lat = olb.Lattice(dict(nx=nx, ny=ny, ds=1 / 64, dt=5e-4, tau=0.01, a=I.VDW_A, b=I.VDW_B, sigma=1e-4, bc_x=0, bc_y=0),
                      stream=torch.cuda.Stream())
    rest = np.ones((ny, nx))
    lat.set_fields(rest, 0 * rest, 0 * rest, rest)
    done = torch.cuda.Event()
    torch.cuda.synchronize()
    lat.step(120)
    done.record(lat.stream)
    c.close()
    assert not done.query()
    lat.sync()
    assert done.query()
    lat.close()


def test_gradients_of_objects_in_two_threads():
    """Objects made, used and freed in two threads at once, each on a stream of
    its own: every call returns the bits it returns alone."""
    torch, olb = _olb()
    work = []
    for k, (nx, ny) in enumerate(((40, 24), (130, 17))):
        norm, m, ref = _pair(torch, nx, ny, 11 + k)
        work.append((nx, ny, norm, m, ref, I.closure_params(seed=20 + k), torch.cuda.Stream()))
    torch.cuda.synchronize()

    def gradients(w):
        nx, ny, norm, m, ref, params, stream = w
        c = olb.Closure(nx, ny, stream=stream)
        c.set_norm(*norm)
        c.set_params(params)
        g, loss = c.gradients(m, ref)
        again = c.train_step(m, ref, 1e-3)
        c.close()
        return g, loss, again

    alone = [gradients(w) for w in work]
    got = [[], []]

    def run(k):
        for _ in range(20):
            got[k].append(gradients(work[k]))

    threads = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):
        assert len(got[k]) == 20
        for g, loss, again in got[k]:
            np.testing.assert_array_equal(g, alone[k][0])
            assert loss == alone[k][1] and again == alone[k][2] == loss
