"""GPU test of a serving step that fails on the host at an admission (an error of
the runtime that the calling thread left unread): the requests that it was to
admit wait on, and every one of them completes with the oracle's words."""
import ctypes
import time

import numpy as np
import pytest

import oracle
import synth
from helpers import empty_u32, np_u32, to_dev
from test_gpu_scratch_keep import hip_runtime

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("count", [3, 20, 40])     # one pointer update, several, two ingest launches
def test_requests_outlive_a_failed_admission(count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    n, primes, d0, d1 = 32, synth.PRIMES_N4096, 70, 24
    dhat = oracle.ntt_db(synth.db_coeffs(180, d0, d1, len(primes), n), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_MFMA)
    pir.pir_db_load_ntt(db, to_dev(dhat).view(-1), domain=pir.PIR_DOMAIN_NTT)
    queries = synth.query_uniform(181, count, d0, primes, n)
    wants = oracle.rowsel(queries, dhat, primes)
    qs = [to_dev(q) for q in queries]
    outs = [empty_u32(wants[i].size) for i in range(count)]
    srv = pir.pir_server_create(db, max_clients=40, chunks=2)
    torch.cuda.synchronize()
    arrivals = [(i, qs[i], outs[i]) for i in range(count)]
    pir.pir_serve_step(srv, ())
    hip, p = hip_runtime(), ctypes.c_void_p()
    hip.hipMalloc.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    assert hip.hipMalloc(ctypes.byref(p), 1 << 60) != 0       # refused; the error stays with the thread
    with pytest.raises(pir.PirError) as e:
        pir.pir_serve_step(srv, arrivals)
    assert e.value.status == pir.PIR_EDEVICE
    got, t0 = {}, time.time()
    while len(got) < count and time.time() - t0 < 60:
        for c in pir.pir_serve_step(srv, ()):
            got[c.id] = c
    torch.cuda.synchronize()
    assert len(got) == count and all(c.status == 0 for c in got.values())
    for i in range(count):
        assert np.array_equal(np_u32(outs[i]).reshape(wants[i].shape), wants[i]), f"request {i}"
    pir.pir_server_destroy(srv)
    pir.pir_db_free(db)
