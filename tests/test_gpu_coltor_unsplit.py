"""GPU parity of the ColTor stage with more (node, limb) blocks than the line up
to which digit polynomials are split over several blocks, on rings whose
transforms take several waves (N = 1024 to 16384): unreduced, lazy and wide
butterflies, paired and unpaired last columns, and both sides of the line for
the rings where a CU holds one block.  Nodes are sampled over the launch
and compared with the CPU oracle, word for word."""
import numpy as np
import pytest

import oracle
import synth
from helpers import assert_guards, empty_u32, guarded_u32, np_u32
from oracle import coltor

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

Q108, P2, W32 = synth.PRIMES_Q108, synth.PRIMES_N4096, synth.PRIMES_W32
CASES = [
    # (N, primes or bits of one prime, log2z, ell, B, ncols): nodes * L
    (1024, Q108, 22, 5, 3, 45),        # 276, unreduced
    (1024, P2, 20, 3, 2, 131),         # 264, lazy
    (1024, W32, 22, 3, 2, 132),        # 264, wide
    (2048, Q108[:2], 22, 3, 2, 131),   # 264, unreduced
    (2048, 30, 16, 2, 1, 515),         # 258, lazy
    (2048, W32, 22, 3, 2, 131),        # 264, wide
    (4096, P2, 20, 3, 1, 259),         # 260, lazy
    (4096, W32, 22, 3, 1, 259),        # 260, wide
    (8192, 27, 14, 2, 1, 512),         # 256: one part (N <= 4096: two)
    (8192, 27, 14, 2, 1, 256),         # 128: two parts
    (8192, 30, 16, 2, 1, 515),         # 258, lazy
    (8192, 30, 16, 2, 1, 257),         # 129, lazy, one part
    (8192, 32, 17, 2, 1, 515),         # 258, wide
    (16384, 27, 14, 2, 1, 515),        # 258, unreduced
    (16384, 30, 16, 2, 1, 511),        # 256, lazy, one part
    (16384, 30, 16, 2, 1, 255),        # 128, lazy, two parts
    (16384, 32, 17, 2, 1, 515),        # 258, wide
]


@pytest.mark.parametrize("case", CASES, ids=[
    f"N{c[0]}_{c[1] if isinstance(c[1], int) else f'{len(c[1])}x{int(c[1][0]).bit_length()}'}bit_l{c[3]}_B{c[4]}c{c[5]}" for c in CASES])
def test_coltor_many_nodes_match_oracle(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    print("coltor many nodes", case, flush=True)
    n, primes, log2z, ell, B, ncols = case
    if isinstance(primes, int):
        primes = tuple(oracle.ntt_primes(n, primes, 1))
    L, nout = len(primes), (ncols + 1) // 2
    ct, rg = empty_u32(B * 2 * ncols * L * n), empty_u32(B * 2 * ell * 2 * L * n)
    pir.pir_synth_query(ct, synth.stream_key(140, synth.TAG_QUERY), 0, B, ncols, primes, n)
    pir.pir_synth_query(rg, synth.stream_key(141, synth.TAG_QUERY), 0, B * ell * 2, 1, primes, n)
    guard, out = guarded_u32(B * 2 * nout * L * n)
    pir.pir_coltor_stage(n, primes, ct, B, ncols, rg, log2z, ell, out)
    torch.cuda.synchronize()
    assert_guards(guard)
    ct_h = np_u32(ct).reshape(B, 2, ncols, L, n)
    rg_h = np_u32(rg).reshape(B, 2, ell, 2, L, n)
    got = np_u32(out).reshape(B, 2, nout, L, n)
    pairs = ncols // 2
    for b, t in {(0, 0), (B - 1, pairs - 1), (B // 2, pairs // 2), (0, pairs // 3), (B - 1, 7)}:
        want = coltor.cmux(ct_h[b, :, 2 * t], ct_h[b, :, 2 * t + 1], rg_h[b], primes, log2z, ell)
        assert np.array_equal(got[b, :, t], want), (b, t)
    if ncols % 2:
        assert np.array_equal(got[:, :, -1], ct_h[:, :, -1])
