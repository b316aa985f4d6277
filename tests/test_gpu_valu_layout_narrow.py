"""GPU parity of batches on a DB that holds only the VALU layout, against the CPU
oracle, word for word: few columns on a long D0 (the matrix-core kernel's units of
64 columns, most of them past D1) with flushes, 16- and 32-row units, 30- and
32-bit primes; and both sides of each line between that kernel and the vector
ALUs, over the rows, the clients and the points."""
import numpy as np
import pytest

import oracle
import synth
from helpers import assert_guards, guarded_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P2 = synth.PRIMES_N4096
SHAPES = [
    # (N, primes, D0, D1, B)
    (8, P2, 1024, 1, 3),             # one column, fewer units than blocks
    (8, P2, 1023, 1, 3),             # the vector ALUs
    (64, P2, 1100, 1, 9),            # 18 rows in 32-row units
    (64, P2, 2100, 1, 4),            # flushes at 32 and 33 chunks
    (512, P2, 1024, 1, 17),          # two row blocks, as many units as blocks
    (64, P2, 513, 2, 3),
    (64, P2, 350, 3, 20),
    (64, P2, 70, 15, 16),
    (64, synth.PRIMES_W32, 1030, 1, 2),
    (16, synth.PRIMES_W32, 2200, 2, 12),
    # either side of the lines (matrix cores first)
    (64, P2, 48, 70, 3),
    (64, P2, 47, 70, 3),
    (64, synth.PRIMES_W32, 64, 70, 2),
    (64, synth.PRIMES_W32, 63, 70, 2),
    (64, synth.PRIMES_W32, 16, 70, 4),
    (64, P2, 32, 70, 4),
    (64, P2, 31, 70, 4),
    (64, P2, 16, 70, 5),
    (64, P2, 16, 70, 16),
    (64, P2, 31, 70, 17),            # (vector ALUs)
    (2048, P2, 16, 128, 17),
    (2048, P2, 16, 127, 17),
    (1024, P2, 16, 128, 17),         # (vector ALUs)
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"N{s[0]}L{len(s[1])}_{s[2]}x{s[3]}_B{s[4]}" for s in SHAPES])
def test_few_columns_match_oracle(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("few columns", shape, flush=True)
    n, primes, d0, d1, B = shape
    dhat = oracle.ntt_db(synth.db_coeffs(190, d0, d1, len(primes), n), primes)
    query = synth.query_uniform(191, B, d0, primes, n)
    want = oracle.rowsel(query, dhat, primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_VALU)
    pir.pir_db_load_ntt(db, to_dev(dhat).view(-1), domain=pir.PIR_DOMAIN_NTT)
    guard, out = guarded_u32(want.size)
    pir.pir_rowsel(db, to_dev(query), out)
    torch.cuda.synchronize()
    assert_guards(guard)
    got = np_u32(out).reshape(want.shape)
    assert np.array_equal(got, want), f"{(got != want).sum()} of {want.size} words differ"
    pir.pir_db_free(db)
