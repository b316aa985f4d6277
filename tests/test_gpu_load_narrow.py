"""GPU parity of loading coefficients into a DB with both layouts around the
number of columns from which the digit planes are made from the VALU layout (12;
below, from an NTT-domain copy), against the CPU oracle, word for word."""
import numpy as np
import pytest

import oracle
import synth
from helpers import guarded_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d1", [1, 2, 11, 12, 13])
@pytest.mark.parametrize("n,primes", [(256, synth.PRIMES_N4096), (512, synth.PRIMES_W32)], ids=["30bit", "32bit"])
def test_narrow_load_matches_oracle(n, primes, d1):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("narrow load", n, d1, flush=True)
    L, B, d0 = len(primes), 3, 130
    coeffs = np.random.default_rng(130).integers(0, 1 << 32, (d0, d1, L, n), dtype=np.uint32)
    reduced = np.stack([coeffs[:, :, l] % np.uint32(q) for l, q in enumerate(primes)], axis=2)
    query = synth.query_uniform(131, B, d0, primes, n)
    want = oracle.rowsel(query, oracle.ntt_db(np.ascontiguousarray(reduced), primes), primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1))
    for row, k in ((64, 66), (0, 64)):       # whole chunks, the last short
        pir.pir_db_load_ntt(db, to_dev(coeffs[row:row + k]).view(-1), row, k, pir.PIR_DOMAIN_COEFF)
    q = to_dev(query)
    for path in (pir.PIR_PATH_VALU, pir.PIR_PATH_MFMA_I8):
        _, out = guarded_u32(want.size)
        pir.pir_rowsel(db, q, out, path)
        torch.cuda.synchronize()
        got = np_u32(out).reshape(want.shape)
        assert np.array_equal(got, want), f"path {path}: {(got != want).sum()} of {want.size} words differ"
    pir.pir_db_free(db)
