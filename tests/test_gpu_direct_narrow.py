"""GPU parity of 9 to 16 clients around the lines between the small-batch kernel
and the tiled one (fewer than 64 columns, more than eight 64-row chunks, a tile
for every CU), in single calls and in serving steps, against the CPU oracle, word
for word."""
import time

import numpy as np
import pytest

import oracle
import synth
from helpers import assert_guards, empty_u32, guarded_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # (N, primes, D0, D1, B)
    (512, synth.PRIMES_N4096, 513, 63, 9),    # 256 groups, 9 chunks: tiled
    (512, synth.PRIMES_N4096, 512, 5, 9),     # 8 chunks: small-batch
    (512, synth.PRIMES_N4096, 576, 64, 9),    # 64 columns: small-batch
    (512, synth.PRIMES_N4096[:1], 600, 3, 16),   # 128 groups: small-batch
    (512, synth.PRIMES_N4096, 600, 3, 8),     # 16 rows: small-batch
    (512, synth.PRIMES_W32, 700, 1, 16),      # tiled, 32-bit primes
]


@pytest.mark.parametrize("case", CASES, ids=[f"N{c[0]}L{len(c[1])}_{c[2]}x{c[3]}_B{c[4]}" for c in CASES])
def test_narrow_batches_match_oracle(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("narrow batch", case, flush=True)
    n, primes, d0, d1, B = case
    dhat = oracle.ntt_db(synth.db_coeffs(160, d0, d1, len(primes), n), primes)
    query = synth.query_uniform(161, B, d0, primes, n)
    want = oracle.rowsel(query, dhat, primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_MFMA)
    pir.pir_db_load_ntt(db, to_dev(dhat).view(-1), domain=pir.PIR_DOMAIN_NTT)
    q = to_dev(query)
    guard, out = guarded_u32(want.size)
    pir.pir_rowsel(db, q, out)
    torch.cuda.synchronize()
    assert_guards(guard)
    assert np.array_equal(np_u32(out).reshape(want.shape), want)
    # the same clients through a server, in one step a sweep
    srv = pir.pir_server_create(db, max_clients=B, chunks=1)
    outs = [empty_u32(want[b].size) for b in range(B)]
    left = len(pir.pir_serve_step(srv, [(b, q.view(B, -1)[b].contiguous(), outs[b]) for b in range(B)]))
    t0 = time.time()
    while left < B and time.time() - t0 < 60:
        left += len(pir.pir_serve_step(srv, ()))
    torch.cuda.synchronize()
    assert left == B
    for b in range(B):
        assert np.array_equal(np_u32(outs[b]).reshape(want[b].shape), want[b]), b
    pir.pir_server_destroy(srv)
    pir.pir_db_free(db)
