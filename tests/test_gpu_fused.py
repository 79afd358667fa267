"""GPU: the fused kernels at the sizes where they can go wrong (edges of tiles, remainders,
the smallest and largest of their ranges), bit for bit against the oracle or against the
general path."""
import numpy as np
import pytest

import paper_2607_05920_amd as fhe
import synth
from oracle import galois, ops, scheme
from oracle import ntt as ontt
from oracle import ring
from tests.gpu_helpers import check, dev, host, ints, limbs_of, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    c = fhe.Context(1555, 1555)
    yield c
    c.close()


# (logN, primes, polynomials, natural order): one transform, counts that leave the last of
# the eight runs short, and the smallest counts that take one workgroup per transform at
# 2^15 and 2^16 points
@pytest.mark.parametrize("logN,nprimes,count,natural", [
    (10, 1, 1, True), (10, 3, 11, False), (11, 5, 3, True), (12, 3, 5, True), (13, 9, 1, False), (13, 3, 7, True),
    (14, 1, 1, True), (14, 5, 5, False), (15, 4, 8, True), (15, 5, 32, False),
    (15, 7, 32, False), (16, 4, 16, True), (16, 4, 60, False), (16, 3, 85, False)])
def test_ntt_whole(ctx, logN, nprimes, count, natural):
    say(f"ntt whole logN={logN} primes={nprimes} count={count} natural={natural}")
    prime0, N = 2, 1 << logN
    rng = np.random.default_rng(100 * logN + count)
    q = np.array([ctx.prime_info(prime0 + p)[0] for p in range(nprimes)], dtype=np.uint64)
    data = (rng.integers(0, 1 << 62, (count, nprimes, N), dtype=np.uint64) % q[:, None]).astype(np.uint32)
    data[0, 0, :7] = q[0] - 1
    t = dev(data)
    ctx.ntt(logN, nprimes, t, count=count, bitrev=not natural, prime0=prime0)
    fwd = host(t, data.shape).copy()
    rev = np.array([int(format(i, f"0{logN}b")[::-1], 2) for i in range(N)])
    for c, p in {(0, 0), (count - 1, nprimes - 1)}:
        psi = pow(ctx.prime_info(prime0 + p)[1], (1 << 16) // N, int(q[p]))
        want = ontt.ntt_fast([int(v) for v in data[c, p]], int(q[p]), psi)
        check([int(v) for v in (fwd[c, p] if natural else fwd[c, p][rev])], want, f"transform {c} prime {p}")
    if logN >= 15:  # one polynomial at a time takes the two-pass transforms
        for c in range(count):
            one = dev(data[c])
            ctx.ntt(logN, nprimes, one, count=1, bitrev=not natural, prime0=prime0)
            assert np.array_equal(host(one, data[c].shape), fwd[c]), f"polynomial {c}"
    ctx.ntt(logN, nprimes, t, count=count, inverse=True, bitrev=not natural, prime0=prime0)
    assert np.array_equal(host(t, data.shape), data)


# (logN, logq, cnum): one limb (one k-block of the lift, primes far below a step of 16 and a
# block of 32); prime counts on both sides of a block (31 and 33 primes at logN 10); the
# lift's largest fused limb count and the first that takes the separate stages; every row
# length of the middle pass, with uneven ciphertext counts
@pytest.mark.parametrize("logN,logq,cnum", [
    (10, 20, 1), (10, 430, 3), (10, 470, 1), (10, 1792, 1), (10, 1793, 2), (11, 256, 2), (12, 257, 1), (13, 100, 3),
    (14, 64, 2), (15, 33, 1), (16, 40, 1)])
def test_ring_mul_fused(ctx, logN, logq, cnum):
    say(f"ring_mul fused logN={logN} logq={logq} cnum={cnum}")
    N, L = 1 << logN, synth.nlimbs(logq)
    rng = np.random.default_rng(7 * logN + logq)
    a, b = (synth.uniform_limbs(rng, logq, N, count=cnum) for _ in range(2))
    top = limbs_of([(1 << logq) - 1], logq)[:, 0]
    a[0, :, :] = top[:, None]  # every coefficient at its largest: the products' largest value
    b[0, :, :] = top[:, None]
    out = dev(np.zeros((cnum, L, N), dtype=np.uint32))
    ctx.ring_mul(logN, logq, dev(a), dev(b), out, cnum=cnum)
    got = host(out, (cnum, L, N))
    for c in range(cnum):
        check(ints(got[c]), ring.ring_mul(ints(a[c]), ints(b[c]), 1 << logq), f"ring_mul {c}")


# one limb, a block of 16 limb rows, and one row more; the second component in m's place
@pytest.mark.parametrize("logN,logq", [(10, 20), (10, 512), (11, 513)])
def test_encrypt_fused(ctx, logN, logq):
    import torch
    say(f"encrypt fused logN={logN} logq={logq}")
    N, L = 1 << logN, synth.nlimbs(logq)
    rng = np.random.default_rng(9 * logN + logq)
    pk = synth.uniform_limbs(rng, 32 * L, N, count=2)  # bits above logq, which do not count
    m = synth.uniform_limbs(rng, logq, N)
    v = rng.integers(-1, 2, N).astype(np.int8)
    e = rng.integers(-(1 << 31), 1 << 31, (2, N)).astype(np.int32)
    v[:4], e[:, :2] = -1, [-(1 << 31), (1 << 31) - 1]
    c0, dm = dev(np.zeros((L, N), dtype=np.uint32)), dev(m)
    ctx.encrypt(fhe.CKKS, 0, logN, logq, dev(pk[0]), dev(pk[1]), dm,
                *(torch.from_numpy(x.copy()).cuda() for x in (v, *e)), c0, dm)
    for i, got in enumerate((host(c0, (L, N)), host(dm, (L, N)))):
        prod = ring.ring_mul([int(x) % (1 << logq) for x in v], [x % (1 << logq) for x in ints(pk[i])], 1 << logq)
        add = ints(m) if i == 0 else [0] * N
        check(ints(got), [(p + a + int(x)) % (1 << logq) for p, a, x in zip(prod, add, e[i])], f"component {i}")


# c1 over m or e0 (read by c0's sum), with words of other coefficients on each other, a whole
# number of rows apart, and apart; the result is that of buffers of their own
@pytest.mark.parametrize("over,shift", [("m", 64), ("m", -3), ("m", 2048), ("m", -1025), ("e0", 5), ("e0", -700),
                                        ("e0", -1024), ("m", 1 << 20)])
def test_encrypt_c1_over_inputs(ctx, over, shift):
    import torch
    logN, logq = 10, 150
    say(f"encrypt, c1 {shift} words from {over}")
    N, L = 1 << logN, synth.nlimbs(logq)
    rng = np.random.default_rng(17)
    pk = [dev(synth.uniform_limbs(rng, logq, N)) for _ in range(2)]
    m = dev(synth.uniform_limbs(rng, logq, N)).reshape(-1)
    v = torch.from_numpy(rng.integers(-1, 2, N).astype(np.int8)).cuda()
    e = [torch.from_numpy(rng.integers(-9, 10, N).astype(np.int32)).cuda() for _ in range(2)]

    def run(m, e0, c1):
        c0 = torch.empty(L * N, dtype=torch.int32, device="cuda")
        ctx.encrypt(fhe.CKKS, 0, logN, logq, *pk, m, v, e0, e[1], c0, c1)
        return host(c0, -1).copy(), host(c1, -1).copy()

    want = run(m, e[0], torch.empty(L * N, dtype=torch.int32, device="cuda"))
    src = m if over == "m" else e[0]
    at = max(0, -shift)
    room = torch.empty(at + max(shift, 0) + L * N, dtype=torch.int32, device="cuda")
    put = room[at:at + src.numel()]
    put.copy_(src)
    c1 = room[at + shift:at + shift + L * N]
    got = run(put if over == "m" else m, put if over == "e0" else e[0], c1)
    for i in (0, 1):
        assert np.array_equal(got[i], want[i]), f"component {i}"


# the ciphertext counts on both sides of the line where a row's polynomials share a wave (16
# rows of 1024 points per compute unit for the HE-mult, 12 for the ring product): one more
# than the line takes the other form for all
@pytest.mark.parametrize("logN,logq", [(13, 218), (14, 100)])
def test_rows_split(ctx, logN, logq):
    import torch
    say(f"rows split logN={logN} logq={logq}")
    N, L = 1 << logN, synth.nlimbs(logq)
    rng = np.random.default_rng(11 * logN + logq)
    per = ((2 * logq + logN) // 30 + 1) * (N >> 10)  # rows of 1024 points per ciphertext, about
    most = 16 * torch.cuda.get_device_properties(0).multi_processor_count // per + 8
    x = [synth.uniform_limbs(rng, logq, N, count=most) for _ in range(4)]
    top = limbs_of([(1 << logq) - 1], logq)[:, 0]
    for v in x:
        v[0, :, :] = top[:, None]
    key = fhe.EvalKey(ctx, fhe.CKKS, 0, logN, logq, logq, synth.uniform_limbs(rng, 2 * logq, N),
                      synth.uniform_limbs(rng, 2 * logq, N))

    def mult(n, first=0):
        out = [dev(np.zeros((n, L, N), dtype=np.uint32)) for _ in range(2)]
        ctx.mul_relin(key, logq, *(dev(v[first:first + n]) for v in x), *out, cnum=n)
        return np.stack([host(o, (n, L, N)) for o in out])

    def ring_mul(n, first=0):
        out = dev(np.zeros((n, L, N), dtype=np.uint32))
        ctx.ring_mul(logN, logq, dev(x[0][first:first + n]), dev(x[1][first:first + n]), out, cnum=n)
        return host(out, (1, n, L, N))

    try:
        for f in (mult, ring_mul):
            want = f(most)  # the other form
            for i in (0, 1, most - 1):
                assert np.array_equal(f(1, i), want[:, i:i + 1]), f"{f.__name__} {i}"
            for n in range(3, most, 4):
                assert np.array_equal(f(n), want[:, :n]), f"{f.__name__} of {n}"
    finally:
        key.close()


def test_bootstrap_same_on_used_memory():
    """The modulus raise clears the limbs above the input's in both components: repeated
    bootstraps, whose buffers hold what earlier work left there, give the same output."""
    import torch
    logN, logq_in, logQ, logc, degree = 10, 40, 840, 40, 11
    N, L = 1 << logN, synth.nlimbs(logQ)
    say("bootstrap on used memory")
    rng = np.random.default_rng(3)
    c = fhe.Context(logQ, logQ)

    def key(g=0):
        return fhe.EvalKey(c, fhe.CKKS, 0, logN, logQ, logQ, synth.uniform_limbs(rng, 2 * logQ, N),
                           synth.uniform_limbs(rng, 2 * logQ, N), g=g)

    relin, conj = key(), key(2 * N - 1)
    rot = {r: key(pow(5, r, 2 * N)) for r in [1, 2, 3] + [1 << i for i in range(2, logN - 1)]}
    diag = [dev(synth.uniform_limbs(rng, logQ, N, count=4)).reshape(-1) for _ in range(2)]
    taylor = [int(v) for v in rng.integers(1, 1 << 39, size=degree + 1)]
    params = dict(logN=logN, logslots=2, logq_in=logq_in, logQ=logQ, logc=logc, logT=8, degree=degree)
    x = fhe.Ciphertext(*(dev(synth.uniform_limbs(rng, logq_in, N)).reshape(-1) for _ in range(2)), logN, logq_in, 30,
                       fhe.CKKS, 0, 1, 1)
    first = None
    try:
        for _ in range(3):
            out = [torch.zeros(L * N, dtype=torch.int32, device="cuda") for _ in range(2)]
            o = c.ct_bootstrap(params, relin, rot, conj, *diag, 1 << 42, taylor, x, out)
            got = [host(v, -1)[:synth.nlimbs(o.logq) * N].copy() for v in out]
            first = first or got
            assert all(np.array_equal(a, b) for a, b in zip(got, first))
    finally:
        for k in [relin, conj, *rot.values()]:
            k.close()
        c.close()


# limb counts on both sides of the limb-serial kernels' blocks (of two and four rows, the next
# block in flight): the rescale by 20 or 32 bits keeps the count or lowers it by one
@pytest.mark.parametrize("logq", [33, 64, 90, 128, 129, 160, 256, 257, 288, 289])
def test_limb_blocks(ctx, logq):
    import torch
    logN, logP = 10, 70
    say(f"limb blocks logq={logq}")
    N, L = 1 << logN, synth.nlimbs(logq)
    rng = np.random.default_rng(13 * logq)
    top = limbs_of([(1 << logq) - 1], logq)[:, 0]
    osch = {fhe.CKKS: scheme.CKKS, fhe.BGV: scheme.BGV}

    def tensor(sch, t):
        c = synth.uniform_limbs(rng, logq, N, count=2)
        c[:, :, :2] = top[None, :, None]  # carries through every limb
        c[:, :, 2] = 0
        return (fhe.Ciphertext(dev(c[0]).reshape(-1), dev(c[1]).reshape(-1), logN, logq, 60, sch, t, 1, 1),
                scheme.Ciphertext(ints(c[0]), ints(c[1]), logN, logq, 60, osch[sch], t))

    def same(got, want, what):
        Lo = synth.nlimbs(got.logq)
        check(ints(host(got.c0, -1)[:Lo * N].reshape(Lo, N)), want.c0, f"{what} c0")
        check(ints(host(got.c1, -1)[:Lo * N].reshape(Lo, N)), want.c1, f"{what} c1")

    out = tuple(torch.empty(L * N, dtype=torch.int32, device="cuda") for _ in range(2))
    for sch, t in ((fhe.CKKS, 0), (fhe.BGV, 65537)):
        (x, ox), (y, oy) = tensor(sch, t), tensor(sch, t)
        same(ctx.ct_add(x, y, out), ops.add(ox, oy), "add")
        same(ctx.ct_sub(x, y, out), ops.sub(ox, oy), "sub")
        same(ctx.ct_negate(x, out), ops.negate(ox), "negate")
        k = (1 << 60) + 12345
        same(ctx.ct_multconst(x, -k, out), ops.multconst(ox, -k, 0), "multconst")
        for bits in (20, 32):
            same(ctx.ct_rescale(x, bits, out), scheme.rescale(ox, bits), f"rescale {bits}")
        inplace = fhe.Ciphertext(x.c0.clone(), x.c1.clone(), *[getattr(x, f) for f in
                                 ("logN", "logq", "logp", "scheme", "t", "gamma", "cnum")])
        same(ctx.ct_rescale(inplace, 20, (inplace.c0, inplace.c1)), scheme.rescale(ox, 20), "rescale in place")
        eb, ea = (synth.uniform_limbs(rng, logq + logP, N) for _ in range(2))
        key = fhe.EvalKey(ctx, sch, t, logN, logq, logP, eb, ea)
        okey = scheme.EvalKey(ints(eb), ints(ea), logN, logq, logP, osch[sch], t)
        try:
            same(ctx.ct_mul_relin(key, x, y, out), scheme.mult(ox, oy, okey), "mult")
            for bits in (20, 32):
                same(ctx.ct_mul_relin(key, x, y, out, bits=bits), scheme.mult_rescale(ox, oy, okey, bits),
                     f"mult, rescale {bits}")
        finally:
            key.close()
        auto = torch.empty(L * N, dtype=torch.int32, device="cuda")
        ctx.automorphism(logN, logq, 5, x.c0, auto)
        check(ints(host(auto, (L, N))), galois.automorphism(ox.c0, 5, 1 << logq), "automorphism")
