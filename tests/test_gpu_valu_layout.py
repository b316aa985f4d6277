"""GPU parity of batches on a DB that holds only the VALU layout, with no path
asked for (the matrix-core kernel that cuts the records into digits itself),
against the CPU oracle, word for word: 16- and 32-row units and several row
blocks, D1 ragged against the 64-column units and the 256-column strips, D0
ragged against the 64-row chunks and above the 2048-row accumulation, the
recombination forms, 32-bit primes, and a coefficient-domain query."""
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
    (8, P2, 33, 1, 3),               # one column, fewer units than blocks
    (64, P2, 64, 64, 8),             # one whole chunk, whole units, 16 rows
    (64, P2, 129, 257, 9),           # 18 rows, three chunks, a strip of one column
    (64, P2, 200, 300, 16),          # 32 rows, a ragged unit in the second strip
    (64, P2, 65, 130, 17),           # 34 rows: two row blocks, the last of two rows
    (16, P2, 2100, 70, 4),           # flushes at 32 and 33 chunks
    (16, P2, 4200, 20, 40),          # flushes, three row blocks
    (1024, P2, 40, 65, 5),           # more units than blocks
    (64, (954376193,), 600, 24, 3),  # split recombination
    (64, (954376193, 1073692673), 130, 40, 13),
    (64, synth.PRIMES_Q108, 130, 129, 9),
    (64, synth.PRIMES_W32, 200, 260, 2),    # 32-bit primes
    (64, synth.PRIMES_W32, 2200, 20, 12),
    (64, P2, 25, 40, 12),            # few records: the vector ALUs
    (64, P2, 16, 64, 12),            # 1024 of them
]


@pytest.mark.parametrize("coeff", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=[f"N{s[0]}L{len(s[1])}_{s[2]}x{s[3]}_B{s[4]}" for s in SHAPES])
def test_valu_layout_matches_oracle(shape, coeff):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("rowsel on the VALU layout", shape, coeff, flush=True)
    n, primes, d0, d1, B = shape
    coeffs = synth.db_coeffs(90, d0, d1, len(primes), n)
    query = synth.query_uniform(91, B, d0, primes, n)
    hat = oracle.ntt_db(query.reshape(B * 2, d0, len(primes), n), primes).reshape(query.shape) if coeff else query
    want = oracle.rowsel(hat, oracle.ntt_db(coeffs, primes), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_VALU)
    pir.pir_db_load_ntt(db, to_dev(coeffs), domain=pir.PIR_DOMAIN_COEFF)
    guard, out = guarded_u32(want.size)
    (pir.pir_rowsel_coeff if coeff else pir.pir_rowsel)(db, to_dev(query), out)
    torch.cuda.synchronize()
    assert_guards(guard)
    got = np_u32(out).reshape(want.shape)
    assert np.array_equal(got, want), f"{(got != want).sum()} of {want.size} words differ"
    pir.pir_db_free(db)
