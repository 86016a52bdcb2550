"""The sketch's one-launch tridiagonalisation needs all its workgroups on the
chip at once.  Where they cannot be (a stream of some of the compute units)
the columns go by launches without a wait for that; two host threads' sketches
on two streams follow each other instead of holding a part of the chip each.
The wait is set to two seconds here: a call that ran into it would show.
"""
import ctypes
import threading
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import banner, to_dev
from tests.test_gpu_tridiag import _case, tri_wait

pytestmark = pytest.mark.gpu

WAIT_US = 2_000_000


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


def _masked_stream():
    """Half of the compute units: every other eight, so that each part of the
    chip keeps half of its own however the mask is dealt out."""
    from paper_2604_02917_amd import api
    words = (torch.cuda.get_device_properties(0).multi_processor_count + 31) // 32
    mask = (ctypes.c_uint32 * words)(*([0x00FF00FF] * words))
    s = ctypes.c_void_p()
    fn = api._lib.hipExtStreamCreateWithCUMask
    fn.restype, fn.argtypes = ctypes.c_int, [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint32, ctypes.c_void_p]
    assert fn(ctypes.byref(s), words, mask) == 0
    return s.value


@pytest.mark.parametrize("k", [400, 2100])
def test_stream_of_half_the_chip(npga, k):
    banner(f"sketch on a masked stream k={k}")
    L, S, ell = _case(k)
    Ld, Sd = to_dev(L), to_dev(S)
    _, sg, gam = npga.sketch_str(Ld, Sd, ell)
    stream = torch.cuda.ExternalStream(_masked_stream())
    stream.wait_stream(torch.cuda.current_stream())
    with tri_wait(WAIT_US), torch.cuda.stream(stream):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, sg1, gam1 = npga.sketch_str(Ld, Sd, ell)
        torch.cuda.synchronize()
        took = time.perf_counter() - t0
    np.testing.assert_allclose(sg1.cpu().numpy(), sg.cpu().numpy(), rtol=2.0 ** -23)
    assert gam == gam1
    assert took < 1e-6 * WAIT_US, took


def test_two_threads(npga):
    banner("sketches of two threads")
    L, S, ell = _case(1500)
    Ld, Sd = to_dev(L), to_dev(S)
    _, sg, gam = npga.sketch_str(Ld, Sd, ell)
    torch.cuda.synchronize()
    reps, got, errors = 12, [], []
    ready = threading.Barrier(2)

    def work():
        try:
            stream = torch.cuda.Stream()
            with tri_wait(WAIT_US), torch.cuda.stream(stream):
                ready.wait(30)
                for _ in range(reps):
                    _, s, g = npga.sketch_str(Ld, Sd, ell)
                    got.append((torch.equal(s, sg), g == gam))
        except Exception as e:  # shown by the test
            errors.append(e)

    threads = [threading.Thread(target=work) for _ in range(2)]
    t0 = time.perf_counter()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    took = time.perf_counter() - t0
    assert not errors and got == [(True, True)] * (2 * reps)
    assert took < 1e-6 * WAIT_US, took
