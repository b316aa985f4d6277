"""GPU parity of loading coefficients into a DB with the VALU layout (transform
straight into the layout, digit planes made from it where whole 64-row chunks
are loaded), through RowSel on every layout the DB holds, against the CPU
oracle, word for word: every ring size that takes this way and one on either
side, D1 ragged against the four-column blocks, the 64-column blocks and the
256-column strips, row ranges that are whole chunks and ranges that are not,
30- and 32-bit primes, coefficients of any 32-bit value."""
import numpy as np
import pytest

import oracle
import synth
from helpers import guarded_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P2 = synth.PRIMES_N4096
CASES = [
    # (N, primes, D0, D1, row ranges)
    (128, P2, 70, 9, [70]),
    (256, P2, 65, 5, [65]),
    (256, P2, 130, 67, [64, 66]),                # whole chunks, the last short
    (256, P2, 130, 7, [64, 64, 2]),
    (256, P2, 130, 7, [40, 90]),                 # no whole chunks: the general way
    (256, P2, 3, 261, [3]),                      # a second strip
    (512, synth.PRIMES_Q108, 66, 6, [66]),
    (1024, P2[:1], 64, 3, [64]),
    (2048, synth.PRIMES_Q108[:3], 20, 9, [20]),
    (4096, P2, 10, 10, [10]),
    (8192, (1073692673,), 5, 3, [5]),
    (256, synth.PRIMES_W32, 70, 66, [64, 6]),
    (4096, synth.PRIMES_W32, 6, 5, [6]),
]


@pytest.mark.parametrize("layouts", ["valu", "both"])
@pytest.mark.parametrize("case", CASES, ids=[f"N{c[0]}L{len(c[1])}_{c[2]}x{c[3]}_{'_'.join(map(str, c[4]))}" for c in CASES])
def test_load_matches_oracle(case, layouts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("load", case, layouts, flush=True)
    n, primes, d0, d1, ranges = case
    L, B = len(primes), 2
    coeffs = np.random.default_rng(97).integers(0, 1 << 32, (d0, d1, L, n), dtype=np.uint32)
    coeffs[0, 0, :, :4] = [0, 0xFFFFFFFF, primes[0] - 1, primes[0]]
    reduced = np.stack([coeffs[:, :, l] % np.uint32(q) for l, q in enumerate(primes)], axis=2)
    query = synth.query_uniform(98, B, d0, primes, n)
    want = oracle.rowsel(query, oracle.ntt_db(np.ascontiguousarray(reduced), primes), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1),
                           pir.PIR_LAYOUT_VALU | (pir.PIR_LAYOUT_MFMA if layouts == "both" else 0))
    row = 0
    for k in ranges:
        pir.pir_db_load_ntt(db, to_dev(coeffs[row:row + k]).view(-1), row, k, pir.PIR_DOMAIN_COEFF)
        row += k
    assert row == d0
    q = to_dev(query)
    for path in (pir.PIR_PATH_VALU, pir.PIR_PATH_MFMA_I8)[:2 if layouts == "both" else 1]:
        _, out = guarded_u32(want.size)
        pir.pir_rowsel(db, q, out, path)
        torch.cuda.synchronize()
        got = np_u32(out).reshape(want.shape)
        assert np.array_equal(got, want), f"path {path}: {(got != want).sum()} of {want.size} words differ"
    pir.pir_db_free(db)
