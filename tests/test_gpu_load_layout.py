"""GPU parity of loading NTT-domain records into the VALU layout: tiles of
consecutive records that cross rows (D1 from one column up, around the tile's
width and the 256-column strips), row ranges that start and end inside a tile,
rings of 2 to 48 point groups around each tile shape, against the CPU oracle,
word for word; and a DB whose single column makes 2^24 short runs of groups."""
import numpy as np
import pytest

import oracle
import synth
from helpers import empty_u32, guarded_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P2, Q108 = synth.PRIMES_N4096, synth.PRIMES_Q108
CASES = [
    # (N, primes, D0, D1, row ranges)
    (64, P2, 70, 1, [70]),               # 32 groups: tiles of 64 records
    (64, P2, 200, 1, [1, 63, 136]),
    (64, P2, 45, 3, [44, 1]),
    (64, P2, 21, 7, [9, 12]),
    (64, P2, 5, 63, [5]),
    (64, P2, 5, 65, [2, 3]),
    (64, P2, 3, 256, [3]),
    (64, P2, 3, 257, [1, 2]),            # a second strip of one column
    (64, P2, 9, 300, [9]),
    (64, P2, 3, 520, [3]),               # two whole strips and eight columns
    (64, Q108[:3], 30, 5, [17, 13]),     # 48 groups: a half-full second block of them
    (8, Q108[:1], 2100, 1, [2100]),      # 2 groups: tiles of 1024 records
    (8, Q108[:3], 700, 3, [350, 350]),   # 6 groups
    (8, Q108, 300, 5, [299, 1]),         # 8 groups: tiles of 256 records
    (32, Q108[:3], 60, 9, [60]),         # 24 groups
    (32, P2, 40, 258, [11, 29]),         # 16 groups, two strips
    (256, synth.PRIMES_W32, 66, 2, [66]),
]


@pytest.mark.parametrize("case", CASES, ids=[f"N{c[0]}L{len(c[1])}_{c[2]}x{c[3]}_{'_'.join(map(str, c[4]))}" for c in CASES])
def test_ntt_records_match_oracle(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("load layout", case, flush=True)
    n, primes, d0, d1, ranges = case
    dhat = oracle.ntt_db(synth.db_coeffs(120, d0, d1, len(primes), n), primes)
    query = synth.query_uniform(121, 1, d0, primes, n)
    want = oracle.rowsel(query, dhat, primes)
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), pir.PIR_LAYOUT_VALU)
    row = 0
    for k in ranges:
        pir.pir_db_load_ntt(db, to_dev(dhat[row:row + k]).view(-1), row, k, pir.PIR_DOMAIN_NTT)
        row += k
    assert row == d0
    _, out = guarded_u32(want.size)
    pir.pir_rowsel(db, to_dev(query), out, pir.PIR_PATH_VALU)
    torch.cuda.synchronize()
    got = np_u32(out).reshape(want.shape)
    assert np.array_equal(got, want), f"{(got != want).sum()} of {want.size} words differ"
    pir.pir_db_free(db)


def test_one_column_of_large_records():
    # 32768 rows of one 256 KiB record, loaded at once (8 GiB): 512 blocks of 32
    # groups a row would make a launch of 2^32 threads, which the runtime
    # refuses.  Queries of one 1 each read single rows back.
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    n, primes, d0 = 16384, (1073643521, 1073479681, 1073184769, 1073053697), 32768
    words = len(primes) * n
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 48 GiB of free device memory")
    src = torch.randint(0, primes[-1], (d0, words), dtype=torch.int32, device="cuda")
    db = pir.pir_db_create(pir.make_params(n, primes, d0, 1), pir.PIR_LAYOUT_VALU)
    pir.pir_db_load_ntt(db, src.view(-1), domain=pir.PIR_DOMAIN_NTT)
    query = torch.zeros((2, d0, words), dtype=torch.int32, device="cuda")
    out = empty_u32(2 * words)
    for a, b in ((0, d0 - 1), (63, 64), (20001, 12345)):
        query[0, a], query[1, b] = 1, 1
        pir.pir_rowsel(db, query.view(-1), out, pir.PIR_PATH_VALU)
        torch.cuda.synchronize()
        assert torch.equal(out.view(2, words), torch.stack([src[a], src[b]])), (a, b)
        query[0, a], query[1, b] = 0, 0
    pir.pir_db_free(db)
