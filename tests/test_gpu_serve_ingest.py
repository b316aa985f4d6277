"""GPU test of the ingest of several requests in one launch: odd and even
counts around one launch's 32 requests admitted at one step boundary, into
scattered free slots, on 28-bit and 32-bit primes and with a first dimension that
is no multiple of a K block; every output word against the oracle."""
import time

import numpy as np
import pytest

import oracle
import synth
from helpers import empty_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("primes,n,d0,waves", [
    (synth.PRIMES_N4096, 32, 70, (1, 31, 32, 33)),
    (synth.PRIMES_N4096, 16, 64, (3, 65, 2)),
    (synth.PRIMES_W32, 32, 33, (5, 33, 1)),
], ids=["28bit", "65-at-once", "32bit"])
def test_requests_admitted_together(primes, n, d0, waves):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    d1, count = 24, sum(waves)
    dhat = oracle.ntt_db(synth.db_coeffs(84, d0, d1, len(primes), n), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_MFMA)
    pir.pir_db_load_ntt(db, to_dev(dhat), domain=pir.PIR_DOMAIN_NTT)
    queries = synth.query_uniform(85, count, d0, primes, n)
    wants = oracle.rowsel(queries, dhat, primes)
    qs = [to_dev(q) for q in queries]
    outs = [empty_u32(wants[i].size) for i in range(count)]
    srv = pir.pir_server_create(db, max_clients=66, chunks=2, pipeline=2)
    first, got = 0, {}
    for wave in waves:      # each wave arrives while the one before may still run
        for c in pir.pir_serve_step(srv, [(i, qs[i], outs[i]) for i in range(first, first + wave)]):
            got[c.id] = c
        first += wave
    t0 = time.time()
    while len(got) < count and time.time() - t0 < 60:
        for c in pir.pir_serve_step(srv, ()):
            got[c.id] = c
    torch.cuda.synchronize()
    assert len(got) == count and all(got[i].status == 0 for i in range(count))
    for i in range(count):
        assert np.array_equal(np_u32(outs[i]).reshape(wants[i].shape), wants[i]), f"request {i}"
    pir.pir_server_destroy(srv)
    pir.pir_db_free(db)
