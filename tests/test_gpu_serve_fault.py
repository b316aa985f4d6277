"""GPU tests of serving steps that fail on the host (an error of the runtime that
the calling thread left unread): the requests that an admission was to take wait
on, a step that was under way is launched again, and every request completes with
the oracle's words."""
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


def leave_an_error():
    hip, p = hip_runtime(), ctypes.c_void_p()
    hip.hipMalloc.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    assert hip.hipMalloc(ctypes.byref(p), 1 << 60) != 0       # refused


def setup(pir, count):
    n, primes, d0, d1 = 32, synth.PRIMES_N4096, 70, 24
    dhat = oracle.ntt_db(synth.db_coeffs(180, d0, d1, len(primes), n), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_MFMA)
    pir.pir_db_load_ntt(db, to_dev(dhat).view(-1), domain=pir.PIR_DOMAIN_NTT)
    queries = synth.query_uniform(181, count, d0, primes, n)
    wants = oracle.rowsel(queries, dhat, primes)
    qs = [to_dev(q) for q in queries]
    outs = [empty_u32(wants[i].size) for i in range(count)]
    torch.cuda.synchronize()
    return db, [(i, qs[i], outs[i]) for i in range(count)], wants


def finish(pir, srv, count, got, arrivals, wants):
    t0 = time.time()
    while len(got) < count and time.time() - t0 < 60:
        for c in pir.pir_serve_step(srv, ()):
            got[c.id] = c
    torch.cuda.synchronize()
    assert len(got) == count and all(c.status == 0 for c in got.values())
    for i, _, out in arrivals[:count]:
        assert np.array_equal(np_u32(out).reshape(wants[i].shape), wants[i]), f"request {i}"


@pytest.mark.parametrize("count", [3, 20, 40])     # one pointer update, several, two ingest launches
def test_requests_outlive_a_failed_admission(count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    db, arrivals, wants = setup(pir, count)
    srv = pir.pir_server_create(db, max_clients=40, chunks=2)
    pir.pir_serve_step(srv, ())
    leave_an_error()
    with pytest.raises(pir.PirError) as e:
        pir.pir_serve_step(srv, arrivals)
    assert e.value.status == pir.PIR_EDEVICE
    finish(pir, srv, count, {}, arrivals, wants)
    pir.pir_server_destroy(srv)
    pir.pir_db_free(db)


@pytest.mark.parametrize("steps_before", [1, 2, 3])     # of four: the last one fails with clients finishing
@pytest.mark.parametrize("count", [2, 24])
def test_a_failed_step_is_launched_again(count, steps_before):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    db, arrivals, wants = setup(pir, count + 1)
    srv = pir.pir_server_create(db, max_clients=count, chunks=4)
    got = {c.id: c for c in pir.pir_serve_step(srv, arrivals[:count])}
    torch.cuda.synchronize()
    for _ in range(steps_before - 1):
        pir.pir_serve_step(srv, ())
        torch.cuda.synchronize()
    leave_an_error()
    with pytest.raises(pir.PirError) as e:
        pir.pir_serve_step(srv, ())
    assert e.value.status == pir.PIR_EDEVICE
    finish(pir, srv, count, got, arrivals, wants)
    # a slot that was emptied serves another request
    got = {c.id: c for c in pir.pir_serve_step(srv, arrivals[count:])}
    t0 = time.time()
    while not got and time.time() - t0 < 60:
        got = {c.id: c for c in pir.pir_serve_step(srv, ())}
    torch.cuda.synchronize()
    assert np.array_equal(np_u32(arrivals[count][2]).reshape(wants[count].shape), wants[count])
    pir.pir_server_destroy(srv)
    pir.pir_db_free(db)
