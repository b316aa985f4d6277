"""Performance cases: the work a program gives this library, through its
public entry points, from the smallest call to the largest.

Every case is a dict of plain values; ``kind`` says which calls one pass makes:

  rowsel   pir_rowsel of ``clients`` clients on a resident DB (NTT-domain query)
  answer   pir_rowsel_coeff (coefficient-domain query, as query expansion leaves
           it), then ``stages`` ColTor stages on its output
  coltor   ``stages`` chained ColTor stages on RowSel's output columns
  reload   pir_db_load_ntt of every DB row from coefficients, then one client's
           pir_rowsel on the reloaded DB
  grouped  one pir_rowsel_grouped call over ``count`` uneven instances
  serve    ``requests`` requests through pir_serve_step with ``slots`` client slots

Rings are given as ``n`` (ring dimension), ``limbs`` and ``bits`` (the largest
``limbs`` primes below 2^bits with q = 1 mod 2n: the primes the benchmark's
workloads use).  ``layouts`` names the DB layouts a program holds: "valu",
"mfma" or "both".  DB records have 16-bit coefficients, the same in every limb;
queries, ciphertexts and RGSW rows are uniform residues.
"""
import math
import random

import torch

import paper_2604_04696_amd as pir

LAYOUTS = {"valu": pir.PIR_LAYOUT_VALU, "mfma": pir.PIR_LAYOUT_MFMA,
           "both": pir.PIR_LAYOUT_VALU | pir.PIR_LAYOUT_MFMA}


def listed():
    return [
        # the smallest call: one client's lookup in a toy-sized DB (1 MiB), where latency and launches count
        dict(name="rowsel_tiny", kind="rowsel", n=1024, limbs=1, bits=30, d0=16, d1=16, clients=1, layouts="both"),
        # the headline: one client against 8 GiB, a pure stream of the DB
        dict(name="rowsel_one", kind="rowsel", n=4096, limbs=2, bits=30, d0=512, d1=512, clients=1, layouts="valu"),
        # a few clients at once, as a lightly loaded server batches them
        dict(name="rowsel_few", kind="rowsel", n=4096, limbs=2, bits=30, d0=512, d1=512, clients=8, layouts="mfma"),
        # a full batch of 64 clients on the same DB
        dict(name="rowsel_batch", kind="rowsel", n=4096, limbs=2, bits=30, d0=512, d1=512, clients=64,
             layouts="mfma"),
        # full 32-bit primes, a small batch, a DB that holds both layouts
        dict(name="rowsel_wide", kind="rowsel", n=4096, limbs=2, bits=32, d0=512, d1=512, clients=4, layouts="both"),
        # odd sizes and three limbs on a program that keeps the 64-bit layout alone
        dict(name="rowsel_ragged", kind="rowsel", n=2048, limbs=3, bits=30, d0=333, d1=301, clients=13,
             layouts="valu"),
        # 32 clients at the paper's parameters (four 27-bit limbs, D0 = 256): coefficient-domain selectors to the
        # first tournament stage
        dict(name="answer_batch", kind="answer", n=4096, limbs=4, bits=27, d0=256, d1=512, clients=32, stages=1,
             log2z=22, ell=5, layouts="mfma"),
        # the first tournament stage alone, 32 clients x 512 columns
        dict(name="coltor_batch", kind="coltor", n=4096, limbs=4, bits=27, clients=32, cols=512, stages=1, log2z=22,
             ell=5),
        # one client's whole tournament, 512 columns down to one: the late stages have few nodes
        dict(name="coltor_one", kind="coltor", n=4096, limbs=4, bits=27, clients=1, cols=512, stages=9, log2z=22,
             ell=5),
        # a DB whose records changed: 1 GiB of coefficients loaded into both layouts, then a lookup
        dict(name="reload", kind="reload", n=4096, limbs=2, bits=30, d0=128, d1=256, clients=1, layouts="both"),
        # uneven tenants in one call
        dict(name="grouped", kind="grouped", n=4096, limbs=2, bits=30, count=8, mix=4),
        # continuous batching: more requests than client slots, all waiting at the start
        dict(name="serve", kind="serve", n=4096, limbs=2, bits=30, d0=512, d1=512, slots=32, requests=48),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _gadget(rng, limbs, bits):
    """(log2z, ell) with z^ell > Q and digits below the primes."""
    total = limbs * bits
    ell = rng.choice([e for e in range(2, 9) if -(-total // e) < min(bits, 30)])
    return -(-total // ell), ell


def _within(case):
    """Whether the case costs no more than the largest listed ones."""
    w = work({"stages": 1, "log2z": 1, "ell": 1, **case})
    return w["bytes"] <= 1.2e10 and w["flops"] <= 2e11


def draw(rng):
    """One more case of the same ranges (sizes log-uniform, odd ones among them)."""
    while True:
        kind = rng.choice(["rowsel"] * 4 + ["answer", "coltor", "coltor", "reload", "grouped", "serve"])
        n = rng.choice([1024, 2048, 4096, 4096, 8192])
        bits = rng.choice([27, 30, 30, 32])
        limbs = rng.randint(1, 4)
        c = dict(kind=kind, n=n, limbs=limbs, bits=bits)
        slots = n * limbs
        if kind in ("coltor", "answer") and (slots > 16384 or limbs == 1 or bits == 32 and limbs == 4):
            continue
        if kind == "grouped":
            c.update(count=rng.randint(2, 10), mix=rng.randrange(1 << 20))
            if not _within(c):
                continue
            return c
        if kind == "coltor":
            c.update(clients=_log_int(rng, 1, 32), cols=_log_int(rng, 2, 512))
            c["stages"] = rng.choice([1, (c["cols"] - 1).bit_length()])
            c["log2z"], c["ell"] = _gadget(rng, limbs, bits)
            if c["clients"] * c["cols"] * slots * c["ell"] > 32 * 512 * 16384 * 5 // 2:
                continue
            return c
        c.update(d0=_log_int(rng, 16, 1024), d1=_log_int(rng, 16, 1024))
        db_words = slots * c["d0"] * c["d1"]
        if db_words > 1 << 31:
            continue
        if kind == "serve":
            c.update(slots=_log_int(rng, 2, 64), requests=_log_int(rng, 2, 96))
            if not _within(c):
                continue
            return c
        c["layouts"] = rng.choice(["both", "mfma", "valu"])
        c["clients"] = 1 if kind == "reload" else _log_int(rng, 1, 96)
        macs = 2 * c["clients"] * db_words
        if c["layouts"] == "valu" and macs > 1 << 34 or not _within(c):
            continue
        if kind == "answer":
            c["stages"] = 1
            c["log2z"], c["ell"] = _gadget(rng, limbs, bits)
            if c["clients"] * c["d1"] * slots * c["ell"] > 32 * 512 * 16384 * 5 // 2:
                continue
        return c


# ------------------------------------------------------------------ inputs
def _is_prime(x):
    return x > 1 and all(x % d for d in range(2, math.isqrt(x) + 1))


def _primes(case):
    step, found = 2 * case["n"], []
    q = ((1 << case["bits"]) - 2) // step * step + 1
    while len(found) < case["limbs"]:
        if q < 1 << case["bits"] and _is_prime(q):
            found.append(q)
        q -= step
    return found


def _mix(case):
    """Instance shapes (D0, D1, clients) of a grouped case, as uneven as the benchmark's."""
    rng = random.Random(case["mix"])
    return [(32 * rng.randint(1, 16), 16 * rng.randint(1, 16), rng.randint(1, 96)) for _ in range(case["count"])]


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed, *tags):
    return torch.Generator(device=_device()).manual_seed(random.Random(repr((seed, tags))).getrandbits(48))


def _residues(gen, polys, primes, n):
    """[polys][L][N] uniform residues as 32-bit words."""
    out = torch.empty(polys, len(primes), n, dtype=torch.int32, device=_device())
    step = max(1, (1 << 27) // n)
    for r in range(0, polys, step):
        k = min(step, polys - r)
        for l, q in enumerate(primes):
            if q < 1 << 31:
                out[r:r + k, l] = torch.randint(0, q, (k, n), generator=gen, device=_device(), dtype=torch.int32)
            else:
                v = torch.randint(0, q, (k, n), generator=gen, device=_device(), dtype=torch.int64)
                out[r:r + k, l] = _word(v)
    return out.view(-1)


def _word(x):
    """64-bit values in [0, 2^32) as 32-bit words (the same bits)."""
    return torch.where(x >= 1 << 31, x - (1 << 32), x).to(torch.int32)


def _coeff_rows(gen, rows, d1, n):
    return torch.randint(0, 1 << 16, (rows, d1, n), generator=gen, device=_device(), dtype=torch.int32)


def _row_step(d1, limbs, n):
    return max(1, (1 << 26) // (d1 * limbs * n))


def _build_db(seed, tag, n, primes, d0, d1, layouts):
    db = pir.pir_db_create(pir.make_params(n, primes, d0, d1), LAYOUTS[layouts])
    gen, step = _gen(seed, "db", tag), _row_step(d1, len(primes), n)
    for r in range(0, d0, step):
        k = min(step, d0 - r)
        rec = _coeff_rows(gen, k, d1, n)[:, :, None, :].expand(k, d1, len(primes), n).contiguous()
        pir.pir_db_load_ntt(db, rec.view(-1), r, k)
    return db


def _empty(words):
    return torch.empty(words, dtype=torch.int32, device="cuda")


def _stage_buffers(case, cols):
    """Output buffers of the chained ColTor stages, and the column count before each."""
    words = case["clients"] * 2 * case["limbs"] * case["n"]
    bufs, counts = [], []
    for _ in range(case["stages"]):
        counts.append(cols)
        cols = (cols + 1) // 2
        bufs.append(_empty(words * cols))
    return bufs, counts


def _rgsw(case, seed, primes):
    rows = case["clients"] * 2 * case["ell"] * 2
    return [_residues(_gen(seed, "rgsw", s), rows, primes, case["n"]) for s in range(case["stages"])]


def prepare(case, seed):
    kind, n, primes = case["kind"], case["n"], _primes(case)
    slots = n * len(primes)
    st = {"case": case, "primes": primes}
    if kind in ("rowsel", "answer", "reload"):
        d0, d1, B = case["d0"], case["d1"], case["clients"]
        st["q"] = _residues(_gen(seed, "query"), B * 2 * d0, primes, n)
        st["out"] = _empty(B * 2 * d1 * slots)
        if kind == "reload":
            st["db"] = pir.pir_db_create(pir.make_params(n, primes, d0, d1), LAYOUTS[case["layouts"]])
            gen = _gen(seed, "db", 0)
            st["coeffs"] = torch.cat([_coeff_rows(gen, min(s, d0 - r), d1, n) for s in (_row_step(d1, len(primes), n),)
                                      for r in range(0, d0, s)])[:, :, None, :].expand(d0, d1, len(primes), n) \
                .contiguous().view(-1)
        else:
            st["db"] = _build_db(seed, 0, n, primes, d0, d1, case["layouts"])
        if kind == "answer":
            st["rgsw"] = _rgsw(case, seed, primes)
            st["bufs"], st["counts"] = _stage_buffers(case, d1)
    elif kind == "coltor":
        st["ct"] = _residues(_gen(seed, "ct"), case["clients"] * 2 * case["cols"], primes, n)
        st["rgsw"] = _rgsw(case, seed, primes)
        st["bufs"], st["counts"] = _stage_buffers(case, case["cols"])
    elif kind == "grouped":
        st["items"] = []
        for i, (d0, d1, B) in enumerate(_mix(case)):
            st["items"].append((_build_db(seed, i, n, primes, d0, d1, "mfma"),
                                _residues(_gen(seed, "query", i), B * 2 * d0, primes, n), B,
                                _empty(B * 2 * d1 * slots)))
        pir.pir_rowsel_grouped(st["items"])   # builds the plan that later calls use
    elif kind == "serve":
        d0, d1 = case["d0"], case["d1"]
        st["db"] = _build_db(seed, 0, n, primes, d0, d1, "mfma")
        st["qs"] = [_residues(_gen(seed, "query", i), 2 * d0, primes, n) for i in range(case["requests"])]
        st["outs"] = [_empty(2 * d1 * slots) for _ in range(case["requests"])]
        st["server"] = pir.pir_server_create(st["db"], max_clients=case["slots"])
    else:
        raise ValueError(kind)
    torch.cuda.synchronize()
    return st


def _stages(st, ct):
    case = st["case"]
    for rgsw, buf, cols in zip(st["rgsw"], st["bufs"], st["counts"]):
        pir.pir_coltor_stage(case["n"], st["primes"], ct, case["clients"], cols, rgsw, case["log2z"], case["ell"],
                             buf)
        ct = buf


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "rowsel":
        pir.pir_rowsel(st["db"], st["q"], st["out"])
        return st["out"]
    if kind == "answer":
        pir.pir_rowsel_coeff(st["db"], st["q"], st["out"])
        _stages(st, st["out"])
        return [st["out"], *st["bufs"]]
    if kind == "coltor":
        _stages(st, st["ct"])
        return st["bufs"]
    if kind == "reload":
        pir.pir_db_load_ntt(st["db"], st["coeffs"])
        pir.pir_rowsel(st["db"], st["q"], st["out"])
        return st["out"]
    if kind == "grouped":
        pir.pir_rowsel_grouped(st["items"])
        return [out for *_, out in st["items"]]
    # serve: every request at the first step; the loop ends with the last completion
    arrivals = [(i, q, out) for i, (q, out) in enumerate(zip(st["qs"], st["outs"]))]
    finished = 0
    while finished < len(st["qs"]):
        finished += len(pir.pir_serve_step(st["server"], arrivals))
        arrivals = ()
    return st["outs"]


# ------------------------------------------------------------------ work
def _nodes(case, cols):
    """ColTor nodes of every stage, and output columns of every stage."""
    nodes, outs = 0, 0
    for _ in range(case["stages"]):
        nodes += case["clients"] * (cols // 2)
        cols = (cols + 1) // 2
        outs += case["clients"] * cols
    return nodes, outs


def _rowsel_work(slots, d0, d1, B):
    return 4 * slots * (d0 * d1 + 2 * B * (d0 + d1)), 2 * slots * 2 * B * d0 * d1


def _coltor_work(case, cols, read_ct):
    n, L, ell = case["n"], case["limbs"], case["ell"]
    nodes, outs = _nodes(case, cols)
    rgsw = case["stages"] * case["clients"] * 4 * ell * n * L
    ct = case["clients"] * 2 * cols * n * L if read_ct else 0
    butterflies = nodes * (2 * L + 2 * ell * L) * (n // 2) * (n.bit_length() - 1)
    return 4 * (ct + rgsw + outs * 2 * n * L), 3 * butterflies + 2 * nodes * 4 * ell * n * L


def work(case):
    """Bytes: every input read once, every output written once.  Operations: a
    multiply and an add per mod-q multiply-add, a multiply, an add and a
    subtraction per butterfly."""
    kind, n, L = case["kind"], case["n"], case["limbs"]
    slots, logn = n * L, n.bit_length() - 1
    if kind in ("rowsel", "reload", "answer"):
        by, ops = _rowsel_work(slots, case["d0"], case["d1"], case["clients"])
        if kind == "reload":   # the records are read, the layouts written; the lookup reads one of them
            records = slots * case["d0"] * case["d1"]
            by += 4 * records * (3 if case["layouts"] == "both" else 2)
            ops += 3 * records // 2 * logn
        if kind == "answer":
            ops += 3 * case["clients"] * 2 * case["d0"] * slots // 2 * logn
            b2, o2 = _coltor_work(case, case["d1"], False)
            by, ops = by + b2, ops + o2
    elif kind == "coltor":
        by, ops = _coltor_work(case, case["cols"], True)
    elif kind == "grouped":
        parts = [_rowsel_work(slots, *shape) for shape in _mix(case)]
        by, ops = sum(p[0] for p in parts), sum(p[1] for p in parts)
    else:
        sweeps = -(-case["requests"] // case["slots"])
        by, ops = _rowsel_work(slots, case["d0"], case["d1"], case["requests"])
        by += 4 * slots * case["d0"] * case["d1"] * (sweeps - 1)
    return {"bytes": by, "flops": ops}


# ------------------------------------------------------------------ exact
MOST_MACS = 40_000_000_000       # mod-q multiply-adds worked out in plain 64-bit arithmetic
MOST_COEFFS = 1_200_000          # ColTor coefficients worked out in Python integers


def _mulmod(a, b, q):
    """a b mod q of int64 values below q < 2^32."""
    return (((a * (b >> 16)) % q << 16) + a * (b & 0xFFFF)) % q


def _psi(q, n):
    rest, factors = q - 1, []
    for d in range(2, 1 << 16):
        if rest % d == 0:
            factors.append(d)
            while rest % d == 0:
                rest //= d
    factors += [rest] if rest > 1 else []
    g = next(g for g in range(2, q) if all(pow(g, (q - 1) // f, q) != 1 for f in factors))
    return pow(g, (q - 1) // (2 * n), q)


def _powers(w, count, q):
    out = [1]
    for _ in range(count - 1):
        out.append(out[-1] * w % q)
    return torch.tensor(out, dtype=torch.int64, device=_device())


def _dft(x, w, q):
    """y_i = sum_j x_j w^(ij) mod q over the last axis, w of order N."""
    n = x.shape[-1]
    bits = n.bit_length() - 1
    idx = torch.arange(n, device=x.device)
    rev = sum(((idx >> b) & 1) << (bits - 1 - b) for b in range(bits))
    x = x[..., rev]
    for b in range(bits):
        half = 1 << b
        v = x.view(*x.shape[:-1], n // (2 * half), 2, half)
        t = _mulmod(v[..., 1, :], _powers(pow(w, n // (2 * half), q), half, q), q)
        u = v[..., 0, :]
        x = torch.stack([(u + t) % q, (u - t) % q], dim=-2).reshape(x.shape)
    return x


def _ntt(x, q):
    """ahat_i = a(psi^(2i+1)), natural order."""
    n = x.shape[-1]
    psi = _psi(q, n)
    return _dft(_mulmod(x % q, _powers(psi, n, q), q), psi * psi % q, q)


def _intt(x, q):
    n = x.shape[-1]
    inv = pow(_psi(q, n), -1, q)
    y = _dft(x, inv * inv % q, q)
    return _mulmod(y, _powers(inv, n, q) * pow(n, -1, q) % q, q) if q < 1 << 31 else \
        _mulmod(_mulmod(y, _powers(inv, n, q), q), torch.full_like(y[..., :1], pow(n, -1, q)), q)


def _unsigned(words):
    return words.to(torch.int64) & 0xFFFFFFFF


def _exact_rowsel(seed, tag, n, primes, d0, d1, B, coeff_query, query_tag=()):
    L = len(primes)
    q_all = _residues(_gen(seed, "query", *query_tag), B * 2 * d0, primes, n).view(2 * B, d0, L, n)
    acc = torch.zeros(L, 2 * B, d1, n, dtype=torch.int64, device=_device())
    gen, step = _gen(seed, "db", tag), _row_step(d1, L, n)
    for r in range(0, d0, step):
        k = min(step, d0 - r)
        rec = _coeff_rows(gen, k, d1, n)
        for l, q in enumerate(primes):
            for i in range(k):
                hat = _ntt(rec[i].to(torch.int64), q)                      # [D1][N]
                sel = _unsigned(q_all[:, r + i, l])                        # [2B][N]
                sel = _ntt(sel, q) if coeff_query else sel
                for m in range(2 * B):
                    acc[l, m] = (acc[l, m] + _mulmod(hat, sel[m], q)) % q
    return acc.permute(1, 2, 0, 3).contiguous()                            # [2B][D1][L][N]


def _exact_stage(ct, rgsw, primes, log2z, ell):
    """ct [B][2][cols][L][N], rgsw [B][2][ell][2][L][N] (int64) -> [B][2][ceil(cols/2)][L][N]."""
    import numpy as np
    B, _, cols, L, n = ct.shape
    Q = math.prod(primes)
    half, z = (Q - 1) // 2, 1 << log2z
    offset = sum((z // 2) * z**i for i in range(ell - 1))
    out = ct[:, :, 0::2].clone()
    pairs = cols // 2
    total = 0
    for l, q in enumerate(primes):
        diff = (ct[:, :, 1::2, l] - ct[:, :, 0:2 * pairs:2, l]) % q
        y = _intt(diff, q) * pow(Q // q, -1, q) % q if q < 1 << 31 else \
            _mulmod(_intt(diff, q), torch.full_like(diff[..., :1], pow(Q // q, -1, q)), q)
        total = total + y.cpu().numpy().astype(object) * (Q // q)
    v = (total + half) % Q - half + offset
    digits = []
    for i in range(ell):
        d = v if i == ell - 1 else (v & (z - 1)) - z // 2
        digits.append(torch.from_numpy(np.asarray(d, dtype=np.int64)).to(ct.device))
        v = v >> log2z
    for l, q in enumerate(primes):
        for i, d in enumerate(digits):
            hat = _ntt(d, q)                                               # [B][2][pairs][N]
            for p in range(2):
                for c in range(2):
                    prod = _mulmod(hat[:, p], rgsw[:, p, i, c, l][:, None, :], q)
                    out[:, c, :pairs, l] = (out[:, c, :pairs, l] + prod) % q
    return out


def _exact_stages(case, seed, primes, ct):
    out = []
    for words in _rgsw(case, seed, primes):
        rg = _unsigned(words).view(case["clients"], 2, case["ell"], 2, len(primes), case["n"])
        ct = _exact_stage(ct, rg, primes, case["log2z"], case["ell"])
        out.append(_word(ct).view(-1))
    return out


def exact(case, seed):
    kind, n, primes = case["kind"], case["n"], _primes(case)
    slots = n * len(primes)
    if "ell" in case:
        nodes, _ = _nodes(case, case.get("cols", case.get("d1")))
        if nodes * 2 * n > MOST_COEFFS:
            return None
    if kind in ("rowsel", "answer", "reload"):
        d0, d1, B = case["d0"], case["d1"], case["clients"]
        # (rows x limbs x output rows: small kernels, one after the other)
        if 2 * B * d0 * d1 * slots > MOST_MACS or d0 * len(primes) * (B + 8) > 60_000:
            return None
        out = _exact_rowsel(seed, 0, n, primes, d0, d1, B, kind == "answer")
        if kind != "answer":
            return _word(out).view(-1)
        ct = out.view(B, 2, d1, len(primes), n)
        return [_word(out).view(-1), *_exact_stages(case, seed, primes, ct)]
    if kind == "coltor":
        words = _residues(_gen(seed, "ct"), case["clients"] * 2 * case["cols"], primes, n)
        ct = _unsigned(words).view(case["clients"], 2, case["cols"], len(primes), n)
        return _exact_stages(case, seed, primes, ct)
    return None
