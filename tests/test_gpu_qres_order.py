"""GPU parity of the query-resident INT8 MFMA kernel against the CPU oracle, word
for word, on both sides of the lines inside it: waves whose order is turned (one
unit's columns, row groups of four waves: 64- and 96-row units) or not, and the
128-row unit with its loads issued before or after the first products, over one
and several units a block, with flushes, 30- and 32-bit primes."""
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
    (8, P2, 65, 1, 17),                       # 64-row units, one column
    (64, P2, 65, 32, 32),                     # 32 columns: one wave of each row group
    (256, P2, 130, 64, 20),                   # half a unit's columns, two units a block
    (64, synth.PRIMES_W32, 100, 65, 32),
    (64, P2, 130, 128, 32),                   # a unit's columns
    (64, P2, 130, 129, 32),                   # one more: not turned
    (16, P2, 2100, 40, 24),                   # two flushes
    (64, synth.PRIMES_W32, 130, 17, 48),      # 96-row units
    (256, P2, 65, 64, 40),
    (64, P2, 65, 65, 40),                     # (not turned)
    (64, P2, 449, 129, 50),                   # 128-row units, loads after the products
    (64, synth.PRIMES_W32, 512, 150, 64),
    (64, P2, 449, 128, 50),                   # before: two units a point
    (64, P2, 448, 129, 50),                   # before: seven chunks
    (64, synth.PRIMES_W32, 65, 200, 64),      # before: the fewest chunks
    (16, P2, 2100, 130, 100),                 # after, two row blocks, two flushes
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"N{s[0]}_{s[2]}x{s[3]}_B{s[4]}_{'32' if s[1] is not P2 else '30'}bit"
                                               for s in SHAPES])
def test_both_sides_of_the_lines(shape, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    n, primes, d0, d1, B = shape
    print("qres rowsel", shape, flush=True)
    coeffs = synth.db_coeffs(62, d0, d1, len(primes), n)
    query = synth.query_uniform(63, B, d0, primes, n)
    want = oracle.rowsel(query, oracle.ntt_db(coeffs, primes), primes)
    monkeypatch.setenv("PIR_MFMA_KERNEL", "qres")
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_MFMA)
    pir.pir_db_load_ntt(db, to_dev(coeffs), domain=pir.PIR_DOMAIN_COEFF)
    guard, out = guarded_u32(want.size)
    for rep in range(2):                      # a second call on buffers that hold the first one's
        pir.pir_rowsel(db, to_dev(query), out, pir.PIR_PATH_MFMA_I8)
        torch.cuda.synchronize()
        got = np_u32(out).reshape(want.shape)
        assert np.array_equal(got, want), f"{(got != want).sum()} of {want.size} words differ"
    assert_guards(guard)
    pir.pir_db_free(db)
