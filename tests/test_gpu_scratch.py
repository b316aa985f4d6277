"""Scratch blocks that the library keeps between calls: calls queued on several
streams and from several threads, with nothing waited for in between and
streams that come and go, give the same words as one call alone."""
import threading

import numpy as np
import pytest

import oracle
import synth
from helpers import empty_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, PRIMES, D0, D1 = 64, synth.PRIMES_N4096, 40, 37


@pytest.mark.parametrize("threads", [1, 3])
def test_queued_calls_on_streams_and_threads(threads):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    coeffs = synth.db_coeffs(71, D0, D1, len(PRIMES), N)
    dbn = oracle.ntt_db(coeffs, PRIMES)
    db = pir.pir_db_create(pir.make_params(N, PRIMES, D0, D1))
    pir.pir_db_load_ntt(db, to_dev(coeffs), domain=pir.PIR_DOMAIN_COEFF)
    clients = (1, 6, 3, 20)          # scratch of four sizes
    queries = [synth.query_uniform(72 + b, b, D0, PRIMES, N) for b in clients]
    want = [oracle.rowsel(q, dbn, PRIMES) for q in queries]
    dev = [to_dev(q) for q in queries]
    torch.cuda.synchronize()
    got, errors = {}, []

    def work(t):
        try:
            for rep in range(4):
                streams = [torch.cuda.Stream(), torch.cuda.Stream()]
                for i, (b, q) in enumerate(zip(clients, dev)):
                    st = streams[(i + rep) % 2]
                    for path in (pir.PIR_PATH_VALU, pir.PIR_PATH_MFMA_I8):
                        with torch.cuda.stream(st):
                            out = empty_u32(b * 2 * D1 * len(PRIMES) * N)
                        pir.pir_rowsel(db, q, out, path, stream=st)
                        got[t, rep, i, path] = (out, st)
        except Exception as e:   # reported by the test's own thread
            errors.append(e)

    jobs = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for j in jobs:
        j.start()
    for j in jobs:
        j.join()
    torch.cuda.synchronize()
    assert not errors, errors
    assert len(got) == threads * 4 * len(clients) * 2
    for (t, rep, i, path), (out, _) in got.items():
        assert np.array_equal(np_u32(out).reshape(want[i].shape), want[i]), (t, rep, i, path)
    pir.pir_db_free(db)
