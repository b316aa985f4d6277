"""GPU parity of the streaming kernel's two ways out, straight to the boundary
layout for outputs of up to 16 MiB and through the staging above, on both sides
of the line, against the CPU oracle (sampled columns at the line), word for
word, with 30- and 32-bit primes."""
import numpy as np
import pytest

import oracle
import synth
from helpers import assert_guards, guarded_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [
    # (N, primes, D0, D1, B)
    (8, synth.PRIMES_N4096, 1, 1, 1),
    (64, synth.PRIMES_N4096, 37, 300, 1),
    (64, synth.PRIMES_N4096, 20, 257, 4),
    (64, synth.PRIMES_W32, 33, 300, 3),
    (4096, synth.PRIMES_N4096, 2, 256, 1),    # exactly 16 MiB
    (4096, synth.PRIMES_N4096, 2, 257, 1),    # one column more
    (4096, synth.PRIMES_W32, 2, 256, 2),      # a client per pass, 16 MiB each
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"N{s[0]}L{len(s[1])}_{s[2]}x{s[3]}_B{s[4]}" for s in SHAPES])
def test_stream_matches_oracle(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("streaming rowsel", shape, flush=True)
    n, primes, d0, d1, B = shape
    coeffs = synth.db_coeffs(95, d0, d1, len(primes), n)
    query = synth.query_uniform(96, B, d0, primes, n)
    cols = np.arange(d1) if d1 * n <= 1 << 15 else np.unique([0, 1, 100, 254, 255, d1 - 1])
    want = oracle.rowsel(query, oracle.ntt_db(np.ascontiguousarray(coeffs[:, cols]), primes), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_VALU)
    pir.pir_db_load_ntt(db, to_dev(coeffs), domain=pir.PIR_DOMAIN_COEFF)
    guard, out = guarded_u32(B * 2 * d1 * len(primes) * n)
    pir.pir_rowsel(db, to_dev(query), out, pir.PIR_PATH_VALU)
    torch.cuda.synchronize()
    assert_guards(guard)
    got = np_u32(out).reshape(B, 2, d1, len(primes), n)[:, :, cols]
    assert np.array_equal(got, want), f"{(got != want).sum()} of {want.size} words differ"
    pir.pir_db_free(db)
