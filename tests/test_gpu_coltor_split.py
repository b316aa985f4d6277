"""GPU parity of the ColTor stage around the line where the digit polynomials of
a node are split over several blocks (few nodes) or stay in one (many), against
the CPU oracle, word for word: as many parts as digits, shares of unequal size,
two parts, one, an unpaired last column, and the three butterfly forms."""
import numpy as np
import pytest

import synth
from helpers import assert_guards, guarded_u32, np_u32, to_dev
from oracle import coltor
from test_gpu_coltor import residues

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

Q108 = synth.PRIMES_Q108
CASES = [
    # (N, primes, log2z, ell, B, ncols): nodes * L blocks before the split
    (1024, Q108, 22, 5, 1, 2),                     # 4: ten parts of one digit
    (256, Q108, 22, 5, 5, 7),                      # 80, unpaired column: five parts of two
    (256, Q108[:3], 22, 4, 7, 12),                 # 126: four parts of two
    (256, Q108[:3], 27, 3, 10, 9),                 # 150: three parts of two
    (256, Q108[:2], 19, 3, 16, 15),                # 256: two parts of three
    (256, Q108[:2], 19, 3, 17, 16),                # 272: one part
    (512, Q108, 22, 5, 13, 11),                    # 312: one part, unpaired column
    (256, synth.PRIMES_N4096, 20, 3, 3, 5),        # lazy butterflies, split
    (256, synth.PRIMES_N4096, 20, 3, 45, 6),       # and not
    (256, synth.PRIMES_W32, 22, 3, 4, 3),          # 32-bit primes, split
    (256, synth.PRIMES_W32, 22, 3, 45, 6),         # and not
]


@pytest.mark.parametrize("case", CASES, ids=[f"N{c[0]}L{len(c[1])}_z{c[2]}l{c[3]}_B{c[4]}c{c[5]}" for c in CASES])
def test_coltor_split_matches_oracle(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("coltor split", case, flush=True)
    n, primes, log2z, ell, B, ncols = case
    cts = residues(310, (B, 2, ncols), primes, n)
    rg = residues(311, (B, 2, ell, 2), primes, n)
    want = coltor.coltor_stage(cts, rg, primes, log2z, ell)
    guard, out = guarded_u32(want.size)
    pir.pir_coltor_stage(n, primes, to_dev(cts), B, ncols, to_dev(rg), log2z, ell, out)
    torch.cuda.synchronize()
    assert_guards(guard)
    got = np_u32(out).reshape(want.shape)
    assert np.array_equal(got, want), f"{(got != want).sum()} of {want.size} words differ"
