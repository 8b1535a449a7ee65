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
        t0.record()
        torch.cuda._sleep(1_000_000)
        t1.record()
    stream.synchronize()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(int(1_000_000 * seconds * 1e3 / t0.elapsed_time(t1)))
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
    for _ in range(3):
        lib.Geometry(mesh, stream=b, **kw).close()
    waited = end.query()
    other.join()
    torch.cuda.synchronize()
    rhs = [g.rhs(1.7733, np.array([[-3.0 + 0.3j]])) for g in (made[0], lib.Geometry(mesh, **kw))]
    assert torch.equal(*rhs)  # the delayed uploads arrived as they were given
    assert not waited
