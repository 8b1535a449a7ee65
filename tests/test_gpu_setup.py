"""Set-up of geometries beside other work on the device."""
import threading
import time

import numpy as np
import pytest

from lspr_inputs import octasphere

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_1812_10722_amd import lspr
    assert torch.cuda.is_available()
    return lspr


def _busy(stream, seconds):
    """Keeps a stream busy for about that long (a bounded spin); an event behind it."""
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with torch.cuda.stream(stream):
        torch.cuda._sleep(50_000_000)  # the clock rises first
        t0.record()
        torch.cuda._sleep(50_000_000)
        t1.record()
    stream.synchronize()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(int(50_000_000 * seconds * 1e3 / t0.elapsed_time(t1)))
        end = torch.cuda.Event()
        end.record()
    return end


def test_setup_does_not_wait_for_a_setup_on_another_stream(lib):
    """A set-up queued on a busy stream leaves staging buffers behind that the device has still to
    read; a set-up on another stream neither waits for them nor takes them."""
    v, t = octasphere(8, 10.0)
    mesh = [(torch.as_tensor(v).cuda(), torch.as_tensor(t.astype(np.int32)).cuda())]
    kw = dict(method="dense", precision="fp64")
    a = torch.cuda.Stream()
    for _ in range(2):  # buffers as a running program has them
        lib.Geometry(mesh, stream=a, **kw).close()
    torch.cuda.synchronize()
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    end = _busy(a, 2.0)
    made = []
    other = threading.Thread(target=lambda: made.append(lib.Geometry(mesh, stream=a, **kw)))
    other.start()
    time.sleep(0.3)  # its first upload is queued, and it waits for its first read-back
    # a stream whose work is not queued behind the busy one's
    for _ in range(8):
        b = torch.cuda.Stream()
        with torch.cuda.stream(b):
            x.add_(1.0)
            done = torch.cuda.Event()
            done.record()
        time.sleep(0.02)
        if done.query():
            break
    else:
        other.join()
        pytest.skip("no stream runs beside the busy one")
    assert not end.query()
    start = time.perf_counter()
    for _ in range(3):
        lib.Geometry(mesh, stream=b, **kw).close()
    took, waited = time.perf_counter() - start, end.query()
    other.join()
    torch.cuda.synchronize()
    rhs = [g.rhs(1.7733, np.array([[-3.0 + 0.3j]])) for g in (made[0], lib.Geometry(mesh, **kw))]
    assert torch.equal(*rhs)  # the delayed uploads arrived as they were given
    assert not waited, took


# the sort without a scan (up to 262144 panels) and with one: a mesh given in another panel order is the
# same problem, so the right-hand side only moves with the panels.  The trees are the same; sums of up
# to 265000 products in another order within equal keys differ by their rounding, 1e-11 of the largest.
@pytest.mark.parametrize("nu", [181, 182])
def test_setup_does_not_depend_on_the_panels_order(lib, nu):
    v, t = octasphere(nu, 10.0)
    order = np.random.default_rng(nu).permutation(len(t))
    kw = dict(method="treecode", precision="fp64", p=2, theta=0.5)
    em, es, e = np.array([1.7733]), np.array([[-3.38 + 0.2j]]), (0.3, -0.5, 1.2)
    rhs = []
    for tri in (t, t[order]):
        geo = lib.Geometry([(v, tri)], **kw)
        rhs.append(geo.rhs(em, es, e).cpu().numpy()[0].reshape(2, -1))
        geo.close()
    assert np.abs(rhs[1] - rhs[0][:, order]).max() < 1e-11 * np.abs(rhs[0]).max()


def test_device_bytes_counts_slabs(lib):
    """Small buffers are pieces of slabs of 1 MiB and more, which a handle holds as long as one piece."""
    v, t = octasphere(1, 10.0)
    geo = lib.Geometry([(v, t)], method="dense", precision="fp64")
    assert 1 << 20 <= geo.info()["device_bytes"] <= 32 << 20
    geo.close()
