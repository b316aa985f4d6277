"""GPU parity of the small-batch INT8 MFMA kernel (up to 32 query rows, DB
fragments straight from memory) against the CPU oracle, word for word: its
three unit shapes at D1 ragged against their rounds of columns, one to 66
chunks of k (query digits of one LDS segment and of several, the last short,
flushes that add to earlier ones), the recombination forms, and fewer and more
units than persistent blocks."""
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
    (8, P2, 1, 1, 1),                # one chunk, one column, fewer units than blocks
    (64, P2, 130, 256, 8),           # 16 rows, 32 columns a step, a whole round, 3 chunks
    (64, P2, 512, 500, 5),           # 10 rows, two rounds, the last ragged, one LDS segment
    (64, P2, 70, 133, 3),            # 16 columns a step, two rounds, 2 chunks
    (16, P2, 530, 33, 2),            # 9 chunks: a second segment of one
    (16, P2, 770, 300, 4),           # 13 chunks, three rounds of 128 columns
    (16, P2, 4200, 250, 2),          # 66 chunks: flushes at 32, 64, 66
    (16, P2, 4200, 130, 9),          # 18 rows in 32-row units, flushes, two rounds
    (64, P2, 512, 257, 16),          # 32 rows, a round of one column at the end
    (1024, P2, 100, 40, 11),         # 2048 units
    (64, (954376193,), 600, 24, 3),  # split recombination
    (64, (954376193, 1073692673), 130, 40, 13),
    (64, synth.PRIMES_Q108, 130, 129, 9),
    (64, synth.PRIMES_W32, 200, 260, 4),    # 32-bit primes
    (64, synth.PRIMES_W32, 2200, 20, 12),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"N{s[0]}L{len(s[1])}_{s[2]}x{s[3]}_B{s[4]}" for s in SHAPES])
def test_direct_matches_oracle(shape, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("small-batch rowsel", shape, flush=True)
    n, primes, d0, d1, B = shape
    coeffs = synth.db_coeffs(80, d0, d1, len(primes), n)
    query = synth.query_uniform(81, B, d0, primes, n)
    want = oracle.rowsel(query, oracle.ntt_db(coeffs, primes), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_MFMA)
    pir.pir_db_load_ntt(db, to_dev(coeffs), domain=pir.PIR_DOMAIN_COEFF)
    q = to_dev(query)
    for kernel in ("", "tile"):
        monkeypatch.setenv("PIR_MFMA_KERNEL", kernel)
        guard, out = guarded_u32(want.size)
        pir.pir_rowsel(db, q, out, pir.PIR_PATH_MFMA_I8)
        torch.cuda.synchronize()
        assert_guards(guard)
        got = np_u32(out).reshape(want.shape)
        assert np.array_equal(got, want), f"{kernel}: {(got != want).sum()} of {want.size} words differ"
    pir.pir_db_free(db)
