"""GPU parity of the NTT helpers on small rings around the counts at which a
block takes one, several and eight polynomials, against the CPU oracle, word for
word, in place; and more polynomials than one launch takes."""
import numpy as np
import pytest

import oracle
import synth
from helpers import guarded_u32, assert_guards, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("count", [1, 7, 511, 1023, 1025, 1537, 4095, 4097])
@pytest.mark.parametrize("n,q", [(8, synth.PRIMES_N4096[0]), (64, synth.PRIMES_W32[0]), (128, synth.PRIMES_N4096[1])])
def test_small_ring_transforms(n, q, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    a = np.random.default_rng(150).integers(0, q, (count, n), dtype=np.uint32)
    guard, buf = guarded_u32(a.size)
    buf.copy_(to_dev(a).view(-1))
    pir.pir_ntt_forward(buf, buf, n, q)
    torch.cuda.synchronize()
    assert_guards(guard)
    assert np.array_equal(np_u32(buf).reshape(a.shape), oracle.ntt_forward(a, q))
    pir.pir_ntt_inverse(buf, buf, n, q)
    torch.cuda.synchronize()
    assert_guards(guard)
    assert np.array_equal(np_u32(buf).reshape(a.shape), a)


def test_more_polynomials_than_a_launch_takes():
    # 2^27 + 5 polynomials of N = 8 (4 GiB): at 32 threads each more than the 2^32
    # threads of one launch.  Samples around the parts' borders against the
    # oracle, and everything by the inverse.
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pir
    n, q, count = 8, synth.PRIMES_N4096[0], (1 << 27) + 5
    a = torch.randint(0, q, (count * n,), dtype=torch.int32, device="cuda")
    out = torch.empty_like(a)
    pir.pir_ntt_forward(a, out, n, q)
    torch.cuda.synchronize()
    for c in (0, (1 << 26) - 2, (1 << 27) - 2, count - 4):
        part = slice(c * n, (c + 4) * n)
        want = oracle.ntt_forward(np_u32(a[part]).reshape(4, n), q)
        assert np.array_equal(np_u32(out[part]).reshape(4, n), want), c
    pir.pir_ntt_inverse(out, out, n, q)
    torch.cuda.synchronize()
    assert torch.equal(out, a)
