"""The work that a user of this library has it do, as measurable cases.

A case is a dict of plain values; its ``kind`` names the public entry point and the rest
its sizes and options.  Sizes are those of the benchmark and the tests: the bare ring
product (N = 2^10, Q = 2^120), HE-mults at N = 2^14 / logq = 438 and N = 2^16 /
logq = 1555, a batch of uneven HE-mults, 2^16-point transforms of 64 polynomials, the
operations of the operation table at N = 2^16 / logq = 1024 on a CipherTensor of 4,
encryption with decryption, and bootstrapping.  ``draw`` spreads over the ranges between
them: 2^10 <= N <= 2^16, 60 <= logq <= 1555, CipherTensors of 1 to 8, both schemes.

Ciphertexts, plaintexts and keys are uniform limbs, the distribution of RLWE ciphertexts
and keys; secrets and errors are ternary and rounded Gaussian.  Every output is a tensor
of whole 32-bit words, exact by the library's contract.
"""
import math

import numpy as np
import torch

import paper_2607_05920_amd as fhe

PRIME_BITS = 30  # residues are modulo 30-bit primes
T_BGV = 65537
SCALE = 40       # CKKS scale and rescale, in bits
LEVELS = (218, 438, 874, 1555)


def listed():
    return [
        # one bare ring product, the smallest call: latency and launches
        {"name": "ring_n10_q120", "kind": "ring", "logN": 10, "logq": 120, "cnum": 1},
        # one CKKS HE-mult with relinearization and rescale at the usual single size
        {"name": "mult_n14_q438", "kind": "mult", "logN": 14, "logq": 438, "cnum": 1, "bgv": False, "bits": SCALE},
        # a small uneven BGV CipherTensor at a middle level and an odd log N
        {"name": "mult_bgv_n15_q874_c3", "kind": "mult", "logN": 15, "logq": 874, "cnum": 3, "bgv": True, "bits": 32},
        # one HE-mult of bootstrapping size: the latency of a large single operation
        {"name": "mult_n16_q1555", "kind": "mult", "logN": 16, "logq": 1555, "cnum": 1, "bgv": False, "bits": SCALE},
        # the same on a CipherTensor of 4: the benchmark's throughput step
        {"name": "mult_n16_q1555_c4", "kind": "mult", "logN": 16, "logq": 1555, "cnum": 4, "bgv": False,
         "bits": SCALE},
        # uneven HE-mults as one planned, captured batch
        {"name": "batch_64", "kind": "batch", "jobs": 64, "mix": 4000},
        # standalone transforms of 64 polynomials, both directions; the inverse in natural
        # order and at an odd log N, as a caller outside the HE-mult takes it
        {"name": "ntt_fwd_n16", "kind": "ntt", "logN": 16, "primes": 106, "count": 64, "inverse": False,
         "bitrev": True},
        {"name": "ntt_inv_n13", "kind": "ntt", "logN": 13, "primes": 31, "count": 16, "inverse": True,
         "bitrev": False},
        # a slot rotation of a CipherTensor (Galois key switch)
        {"name": "rotate_n16_q1024_c4", "kind": "rotate", "logN": 16, "logq": 1024, "cnum": 4},
        # a linear step without a ring product: add, integer constant, rescale
        {"name": "linear_n16_q1024_c4", "kind": "linear", "logN": 16, "logq": 1024, "cnum": 4, "bits": 60},
        # the client's side: public-key encryption and decryption of one ciphertext
        {"name": "crypt_n14_q438", "kind": "crypt", "logN": 14, "logq": 438, "bgv": False},
        # a whole circuit: bootstrapping of one ciphertext with 4 slots
        {"name": "bootstrap_n14_q1024", "kind": "boot", "logN": 14, "logq": 1024},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["ring", "mult", "mult", "mult", "batch", "ntt", "ntt", "rotate", "linear", "crypt", "vec"])
    if kind == "batch":
        return {"kind": kind, "jobs": _log_int(rng, 4, 64), "mix": rng.randrange(1 << 16)}
    logN = rng.randint(10, 16)
    if kind == "ntt":
        return {"kind": kind, "logN": logN, "primes": _log_int(rng, 3, 106), "count": _log_int(rng, 1, 64),
                "inverse": rng.random() < 0.5, "bitrev": rng.random() < 0.5}
    logq = _log_int(rng, 60, 1555)
    if kind == "crypt":
        return {"kind": kind, "logN": logN, "logq": logq, "bgv": rng.random() < 0.5}
    cnum = _log_int(rng, 1, 4 if logN == 16 and logq > 1024 else 8)
    case = {"kind": kind, "logN": logN, "logq": logq, "cnum": cnum}
    if kind == "mult":
        case["bgv"] = rng.random() < 0.3
        case["bits"] = rng.choice([0, 32, SCALE])
    if kind == "linear":
        case["bits"] = rng.randint(20, 59)
    return case


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform(g, bits, N, count=1):
    """Uniform values of [0, 2^bits) as limb words, int32[count, L, N] on the GPU."""
    L = fhe.nlimbs(bits)
    w = torch.randint(-(1 << 31), 1 << 31, (count, L, N), dtype=torch.int32, device="cuda", generator=g)
    if bits % 32:
        w[:, L - 1] &= (1 << (bits % 32)) - 1
    return w


def _empty(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def _key(ctx, g, logN, logQ, logP, bgv=False, galois=0):
    """A key of uniform limbs, which reach the library from host memory."""
    N = 1 << logN
    b, a = (fhe.to_host(_uniform(g, logP + logQ, N))[0] for _ in range(2))
    return fhe.EvalKey(ctx, fhe.BGV if bgv else fhe.CKKS, T_BGV if bgv else 0, logN, logQ, logP, b, a, g=galois)


def _ct(c0, c1, logN, logq, logp, cnum=1):
    return fhe.Ciphertext(c0, c1, logN, logq, logp, fhe.CKKS, 0, 1, cnum)


def _mix(case):
    """The batch's (logN, logq) pairs: log N of 13 to 16 and the four levels, uniform."""
    r = np.random.default_rng(case["mix"])
    n = r.integers(13, 17, size=case["jobs"])
    return list(zip(n.tolist(), [LEVELS[i] for i in r.integers(0, 4, size=case["jobs"])]))


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, _gen(seed))


def run(state):
    return state["go"]()


def _prepare_ring(case, g):
    n, q, c = case["logN"], case["logq"], case["cnum"]
    ctx = fhe.Context(q, q)
    a, b = (_uniform(g, q, 1 << n, c) for _ in range(2))
    out = torch.empty_like(a)

    def go():
        ctx.ring_mul(n, q, a, b, out, c)
        return out
    return {"go": go}


def _prepare_mult(case, g):
    n, q, c, bits = case["logN"], case["logq"], case["cnum"], case["bits"]
    ctx = fhe.Context(q, q)
    key = _key(ctx, g, n, q, q, case["bgv"])
    key.prepare(q)
    ins = [_uniform(g, q, 1 << n, c) for _ in range(4)]
    outs = [_empty(c, fhe.nlimbs(q - bits), 1 << n) for _ in range(2)]

    def go():
        if bits:
            ctx.mul_relin_rescale(key, q, bits, *ins, *outs, cnum=c)
        else:
            ctx.mul_relin(key, q, *ins, *outs, cnum=c)
        return outs
    return {"go": go}


def _prepare_batch(case, g):
    mix = _mix(case)
    top = max(q for _, q in mix)
    ctx = fhe.Context(top, top)
    keys = {n: _key(ctx, g, n, top, top) for n in sorted({n for n, _ in mix})}
    words = [fhe.nlimbs(q - SCALE) << n for n, q in mix]
    outs = [_empty(sum(words)) for _ in range(2)]
    jobs, at = [], 0
    for (n, q), w in zip(mix, words):
        ins = [_uniform(g, q, 1 << n) for _ in range(4)]
        jobs.append((keys[n], q, SCALE, *ins, *(o[at:at + w] for o in outs)))
        at += w
    plan = fhe.BatchPlan(ctx, jobs, flags=fhe.PLAN_GRAPH | fhe.PLAN_AUTOTUNE)

    def go():
        plan.run()
        return outs
    return {"go": go, "plan": plan, "jobs": jobs}


def _prepare_ntt(case, g):
    n, k, c = case["logN"], case["primes"], case["count"]
    logq = max(60, PRIME_BITS * k // 3)  # a context of at least k primes (its largest product has 3 logq bits)
    ctx = fhe.Context(logq, logq)
    q = torch.tensor([ctx.prime_info(i)[0] for i in range(k)], dtype=torch.int32, device="cuda")
    data = torch.randint(0, 1 << 29, (c, k, 1 << n), dtype=torch.int32, device="cuda", generator=g) % q[:, None]

    def go():  # in place: each pass transforms what the last one left, as canonical residues
        ctx.ntt(n, k, data, count=c, inverse=case["inverse"], bitrev=case["bitrev"])
        return data
    return {"go": go}


def _prepare_rotate(case, g):
    n, q, c = case["logN"], case["logq"], case["cnum"]
    ctx = fhe.Context(q, q)
    key = _key(ctx, g, n, q, q, galois=5)
    key.prepare(q)
    x = _ct(_uniform(g, q, 1 << n, c), _uniform(g, q, 1 << n, c), n, q, SCALE, c)
    outs = (torch.empty_like(x.c0), torch.empty_like(x.c1))

    def go():
        ctx.ct_leftrotate(key, 1, x, outs)
        return outs
    return {"go": go}


def _prepare_vec(case, g):
    """Ciphertexts times one plaintext each (multconstvec, pairwise)."""
    n, q, c = case["logN"], case["logq"], case["cnum"]
    ctx = fhe.Context(q, q)
    x = _ct(_uniform(g, q, 1 << n, c), _uniform(g, q, 1 << n, c), n, q, SCALE, c)
    m = _uniform(g, q, 1 << n, c)
    outs = (torch.empty_like(x.c0), torch.empty_like(x.c1))

    def go():
        ctx.ct_multconstvec(x, m, c, outs, logp_m=SCALE)
        return outs
    return {"go": go}


def _prepare_linear(case, g):
    n, q, c, bits = case["logN"], case["logq"], case["cnum"], case["bits"]
    ctx = fhe.Context(q, q)
    x, y = (_ct(_uniform(g, q, 1 << n, c), _uniform(g, q, 1 << n, c), n, q, bits, c) for _ in range(2))
    k = (1 << (bits - 1)) + 12345
    s, p = ((torch.empty_like(x.c0), torch.empty_like(x.c1)) for _ in range(2))
    outs = tuple(_empty(c, fhe.nlimbs(q - bits), 1 << n) for _ in range(2))

    def go():
        ctx.ct_rescale(ctx.ct_multconst(ctx.ct_add(x, y, s), k, p, logp_k=bits), bits, outs)
        return outs
    return {"go": go}


def _prepare_crypt(case, g):
    n, q, bgv = case["logN"], case["logq"], case["bgv"]
    N, L = 1 << n, fhe.nlimbs(q)
    scheme, t = (fhe.BGV, T_BGV) if bgv else (fhe.CKKS, 0)
    ctx = fhe.Context(q, q)
    pk = [_uniform(g, q, N) for _ in range(2)]
    m = torch.zeros(L, N, dtype=torch.int32, device="cuda")
    m[0] = torch.randint(0, T_BGV, (N,), dtype=torch.int32, device="cuda", generator=g)
    v, s = (torch.randint(-1, 2, (N,), dtype=torch.int8, device="cuda", generator=g) for _ in range(2))
    e0, e1 = (torch.round(3.2 * torch.randn(N, device="cuda", generator=g)).to(torch.int32) for _ in range(2))
    c0, c1 = _empty(L, N), _empty(L, N)
    out = _empty(N) if bgv else _empty(L, N)

    def go():
        ctx.encrypt(scheme, t, n, q, *pk, m, v, e0, e1, c0, c1)
        ctx.decrypt(scheme, t, 1, n, q, c0, c1, s, out)
        return c0, c1, out
    return {"go": go}


def _prepare_boot(case, g):
    n, logQ, logs, logc, degree = case["logN"], case["logq"], 2, SCALE, 11
    N, slots = 1 << n, 1 << logs
    ctx = fhe.Context(logQ, logQ)
    relin = _key(ctx, g, n, logQ, logQ)
    amounts = sorted(set(range(1, slots)) | {1 << i for i in range(logs, n - 1)})
    rot = {r: _key(ctx, g, n, logQ, logQ, galois=pow(5, r, 2 * N)) for r in amounts}
    conj = _key(ctx, g, n, logQ, logQ, galois=2 * N - 1)
    r = [pow(5, j, 4 * slots) for j in range(slots)]
    V = np.array([[np.exp(2j * np.pi * (rj * k % (4 * slots)) / (4 * slots)) for k in range(slots)] for rj in r])

    def encoded(A):
        d = [np.array([A[j][(j + i) % slots] for j in range(slots)]) for i in range(slots)]
        return fhe.to_device(np.stack([fhe.ckks_encode(x, n, logc, logQ) for x in d]))

    c2s, s2c = encoded(np.linalg.inv(V)), encoded(V / (2 * np.pi))
    k_y = round(2 * math.pi * 2.0 ** logc)
    taylor = [round((-1) ** (k // 2) / math.factorial(k) * 2.0 ** logc) for k in range(degree + 1)]
    params = dict(logN=n, logslots=logs, logq_in=SCALE, logQ=logQ, logc=logc, logT=8, degree=degree)
    x = _ct(_uniform(g, SCALE, N), _uniform(g, SCALE, N), n, SCALE, 30)
    bufs = [_empty(fhe.nlimbs(logQ) * N) for _ in range(2)]

    def go():
        o = ctx.ct_bootstrap(params, relin, rot, conj, c2s, s2c, k_y, taylor, x, bufs)
        return [b[:fhe.nlimbs(o.logq) * N] for b in bufs]
    return {"go": go}


# ------------------------------------------------------------------ floors
def _words(bits, logN, count=1):
    return 4.0 * fhe.nlimbs(bits) * (1 << logN) * count


def _transforms(logN, bits, rows):
    """Operations (a multiply-add is two) of `rows` polynomials' transforms over the primes
    of a product of `bits` bits: three multiply-adds to a butterfly."""
    return rows * math.ceil(bits / PRIME_BITS) * 6.0 * logN * (1 << logN) / 2


def _mult_work(logN, logq, cnum, bits, key_once=True):
    ins = 4 * _words(logq, logN, cnum)
    outs = 2 * _words(logq - bits, logN, cnum)
    key = 2 * _words(2 * logq, logN, 1 if key_once else cnum)
    ops = _transforms(logN, 2 * logq + logN, 7 * cnum) + _transforms(logN, 3 * logq + logN, 3 * cnum)
    return {"bytes": ins + outs + key, "flops": ops}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        each = [_mult_work(n, q, 1, SCALE, key_once=False) for n, q in _mix(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    n = case["logN"]
    if kind == "ntt":
        rows = case["primes"] * case["count"]
        return {"bytes": 8.0 * rows * (1 << n), "flops": rows * 6.0 * n * (1 << n) / 2}
    q = case["logq"]
    if kind == "mult":
        return _mult_work(n, q, case["cnum"], case["bits"])
    if kind == "ring":
        return {"bytes": 3 * _words(q, n, case["cnum"]), "flops": _transforms(n, 2 * q + n, 3 * case["cnum"])}
    if kind == "vec":
        return {"bytes": 5 * _words(q, n, case["cnum"]), "flops": _transforms(n, 2 * q + n, 5 * case["cnum"])}
    if kind == "rotate":
        return {"bytes": 4 * _words(q, n, case["cnum"]) + 2 * _words(2 * q, n),
                "flops": _transforms(n, 3 * q + n, 3 * case["cnum"])}
    if kind == "linear":
        c, bits = case["cnum"], case["bits"]
        return {"bytes": 4 * _words(q, n, c) + 2 * _words(q - bits, n, c), "flops": 6.0 * c * (1 << n)
                * fhe.nlimbs(q) * 2}
    if kind == "crypt":
        return {"bytes": 6 * _words(q, n) + 10.0 * (1 << n), "flops": _transforms(n, q + n, 6)}
    # bootstrapping reads its keys and diagonals at least once
    keys = 2 + len(set(range(1, 4)) | {1 << i for i in range(2, n - 1)})
    return {"bytes": keys * 2 * _words(2 * q, n) + 10 * _words(q, n),
            "flops": _transforms(n, 3 * q + n, 3 * (keys - 1 + 6))}


def exact(case, seed):
    """Every output is a whole number that two correct runs agree on in each bit: there is
    no error against 64 bits to state, and the multiprecision products themselves have no
    64-bit form."""
    return None
