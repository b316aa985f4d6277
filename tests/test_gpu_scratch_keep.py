"""The bounds of the scratch memory held between calls: given back to the device
by pir_scratch_trim and by a library allocation that runs out of memory, held not
at all or only up to a few blocks where PIR_SCRATCH_KEEP says so (blocks then
leave while other streams work), not held where it would be more than stays
free, taken up by another stream once its event has passed, and by streams
whose handle an earlier one had.  Words against the CPU oracle."""
import ctypes
import threading

import numpy as np
import pytest

import oracle
import synth
from helpers import empty_u32, np_u32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MIB = 1 << 20
N, PRIMES, D0, D1 = 64, synth.PRIMES_N4096, 40, 37
CLIENTS = (6, 1, 20, 40, 3)          # scratch of 1 to 4 MiB and more
Q108 = synth.PRIMES_Q108


@pytest.fixture
def pir():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04696_amd as pkg
    yield pkg
    torch.cuda.synchronize()
    pkg.pir_scratch_trim()


def free_now():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


class Stage:
    """A ColTor stage whose digits take 2 * 5 * 4096 words a node."""

    def __init__(self, pir, nodes):
        self.pir, self.cols, words = pir, 2 * nodes, len(Q108) * 4096
        self.ct, self.rg, self.out = (torch.zeros(k * words, dtype=torch.int32, device="cuda")
                                      for k in (2 * self.cols, 4 * 5, 2 * nodes))

    def __call__(self, stream=None):
        self.pir.pir_coltor_stage(4096, Q108, self.ct, 1, self.cols, self.rg, 22, 5, self.out, stream=stream)


def test_trim_gives_memory_back(pir):
    stage = Stage(pir, 1024)             # 160 MiB of digits
    before = free_now()
    stage()
    held = before - free_now()
    assert held >= 160 * MIB
    assert pir.pir_scratch_trim() >= 160 * MIB
    assert before - free_now() <= held - 160 * MIB
    assert pir.pir_scratch_trim() == 0


def test_trim_behind_unfinished_work(pir):
    # nothing waited for: before the allocation, nor before the trim
    stage = Stage(pir, 1024)
    stage()
    pir.pir_scratch_trim()
    before = free_now()
    big = torch.empty(1 << 28, dtype=torch.int32, device="cuda")
    for _ in range(20):
        big.zero_()
    stage()
    assert pir.pir_scratch_trim() >= 160 * MIB
    del big
    assert before - free_now() <= 8 * MIB


def test_nothing_held_when_told(pir, monkeypatch):
    stage = Stage(pir, 1024)
    pir.pir_scratch_trim()
    monkeypatch.setenv("PIR_SCRATCH_KEEP", "0")
    for _ in range(3):
        stage()
    assert pir.pir_scratch_trim() == 0


def test_library_allocation_takes_it_back(pir):
    # a server of 550 GB: the allocation fails, after a second try without the
    # scratch
    stage = Stage(pir, 1024)
    db = pir.pir_db_create(pir.make_params(4096, PRIMES, 2048, 1), pir.PIR_LAYOUT_MFMA)
    stage()
    pir.pir_scratch_trim()
    before = free_now()
    stage()
    assert before - free_now() >= 160 * MIB
    with pytest.raises(pir.PirError) as e:
        pir.pir_server_create(db, max_clients=4096, hbm_budget=1 << 40)
    assert e.value.status == pir.PIR_ENOMEM
    assert before - free_now() <= 8 * MIB
    assert pir.pir_scratch_trim() == 0
    pir.pir_db_free(db)


def test_one_block_serves_streams_in_turn(pir):
    stage = Stage(pir, 1024)
    stage()
    one = pir.pir_scratch_trim()
    for _ in range(8):
        stage(torch.cuda.Stream())
        torch.cuda.synchronize()
    assert pir.pir_scratch_trim() == one


def test_held_no_more_than_stays_free(pir):
    stage = Stage(pir, 8192)             # 1.25 GiB of digits
    stage()
    assert pir.pir_scratch_trim() >= 1280 * MIB
    try:
        hold = torch.empty(free_now() - 2048 * MIB, dtype=torch.uint8, device="cuda")
    except torch.OutOfMemoryError:
        pytest.skip("the device's free memory is not one allocation")
    stage()
    torch.cuda.synchronize()
    assert pir.pir_scratch_trim() <= 64 * MIB
    del hold
    torch.cuda.empty_cache()
    stage()                              # room again
    assert pir.pir_scratch_trim() >= 1280 * MIB


def lookup_db(pir):
    coeffs = synth.db_coeffs(170, D0, D1, len(PRIMES), N)
    db = pir.pir_db_create(pir.make_params(N, PRIMES, D0, D1))
    pir.pir_db_load_ntt(db, to_dev(coeffs), domain=pir.PIR_DOMAIN_COEFF)
    queries = [synth.query_uniform(171 + b, b, D0, PRIMES, N) for b in CLIENTS]
    dbn = oracle.ntt_db(coeffs, PRIMES)
    return db, [to_dev(q) for q in queries], [oracle.rowsel(q, dbn, PRIMES) for q in queries]


@pytest.mark.parametrize("keep", [0, 1 * MIB, 5 * MIB])
@pytest.mark.parametrize("threads", [1, 3])
def test_blocks_leave_while_streams_work(pir, monkeypatch, threads, keep):
    monkeypatch.setenv("PIR_SCRATCH_KEEP", str(keep))
    db, dev, want = lookup_db(pir)
    torch.cuda.synchronize()
    got, errors = [], []

    def work():
        try:
            streams = [torch.cuda.Stream() for _ in range(3)]
            for rep in range(6):
                for i, (b, q) in enumerate(zip(CLIENTS, dev)):
                    st = streams[(i + rep) % 3]
                    with torch.cuda.stream(st):
                        out = empty_u32(want[i].size)
                    pir.pir_rowsel(db, q, out, pir.PIR_PATH_MFMA_I8, stream=st)
                    got.append((i, out, st))
        except Exception as e:   # reported by the test's own thread
            errors.append(e)

    jobs = [threading.Thread(target=work) for _ in range(threads)]
    for j in jobs:
        j.start()
    for j in jobs:
        j.join()
    torch.cuda.synchronize()
    assert not errors, errors
    assert len(got) == threads * 6 * len(CLIENTS)
    for i, out, _ in got:
        assert np.array_equal(np_u32(out).reshape(want[i].shape), want[i]), CLIENTS[i]
    assert pir.pir_scratch_trim() <= keep
    pir.pir_db_free(db)


def hip_runtime():
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64.so" in line}
    return ctypes.CDLL(sorted(paths)[0])


def test_streams_made_and_destroyed(pir):
    db, dev, want = lookup_db(pir)
    outs = [[empty_u32(w.size) for w in want] for _ in range(12)]
    torch.cuda.synchronize()
    hip, handles = hip_runtime(), set()
    hip.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    for row in outs:
        st = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(st), 1) == 0     # non-blocking
        handles.add(st.value)
        for q, out in zip(dev, row):
            pir.pir_rowsel(db, q, out, pir.PIR_PATH_MFMA_I8, stream=st.value)
        assert hip.hipStreamDestroy(st) == 0    # its work goes on; a later stream may get the handle
    torch.cuda.synchronize()
    print("handles", len(handles), flush=True)
    for row in outs:
        for w, out in zip(want, row):
            assert np.array_equal(np_u32(out).reshape(w.shape), w)
    pir.pir_db_free(db)
