"""What a program that uses this library has it do, for timing and comparison.

Every case is one pass through the public Python entry points on buffers that
are resident on the GPU: a batched KeySwitch under the plan the shipped tuning
table gives for the set (the library's default where it holds none), HMUL,
HROT, a replayed HIP graph, and the step calls (ntt, intt, bconv, modup,
keymult, moddown) that a program strings together itself. Sizes are the
benchmark's four parameter sets, the paper's grid (N = 2^14..2^17,
L = 10, 30, 50, dnum = 2, 4, 6, 8), levels of those sets, and batches from one
ciphertext to 32, odd ones among them. Values are uniform residues modulo each
prime, which is how ciphertext components and evaluation keys are distributed.

A case: op; dnum, log_n, ell of the parameter set; level (Q limbs of the
ciphertext, ell at the top); batch; plan ("tuned": the shipped table's plan or
its nearest batch, else the default; "default": plan=None).
"""
import functools

import torch

import paper_2603_16692_amd as ks
from paper_2603_16692_amd import autotune

OPS = ("keyswitch", "hmul", "hrot", "graph", "steps", "raise")


def _case(name, op, dnum, log_n, ell, batch, level=None, plan="tuned", galois=5):
    return {"name": name, "op": op, "dnum": dnum, "log_n": log_n, "ell": ell, "level": level or ell, "batch": batch,
            "plan": plan, "galois": galois}


def listed():
    return [
        # one small ciphertext: a latency-bound call, a few microseconds a kernel
        _case("ks-d2n13l6-b1", "keyswitch", 2, 13, 6, 1),
        # one ciphertext of the mid set replayed from a graph, as a serving loop holds it
        _case("graph-d2n15l10-b1", "graph", 2, 15, 10, 1),
        # a full batch of the mid set, as the serving loop forms it
        _case("ks-d2n15l10-b32", "keyswitch", 2, 15, 10, 32),
        # a rotation of a part-filled batch at an odd level of the mid set
        _case("hrot-d2n15l9-b5", "hrot", 2, 15, 10, 5, level=9, galois=78125 % (1 << 16)),
        # the benchmark's default workload, and the same set with one ciphertext
        _case("ks-d4n16l32-b8", "keyswitch", 4, 16, 32, 8),
        _case("ks-d4n16l32-b1", "keyswitch", 4, 16, 32, 1),
        # a ciphertext that has lost limbs (short last digit), an odd batch, no plan given
        _case("ks-d4n16l32-lv13-b3", "keyswitch", 4, 16, 32, 3, level=13, plan="default"),
        # the product of two ciphertexts with relinearisation, which the paper times
        _case("hmul-d4n16l32-b8", "hmul", 4, 16, 32, 8),
        # the deep set: the largest key and footprint
        _case("ks-d8n17l56-b2", "keyswitch", 8, 17, 56, 2),
        # a set of the paper's grid with wide digits (25 primes)
        _case("ks-d2n17l50-b1", "keyswitch", 2, 17, 50, 1),
        # the KeySwitch called step by step: modup, keymult, moddown
        _case("steps-d4n16l32-b2", "steps", 4, 16, 32, 2),
        # one digit raised by hand with the transform and conversion calls: intt, bconv, ntt
        _case("raise-d4n16l32-b4", "raise", 4, 16, 32, 4),
    ]


def _cost(c):
    """Words of the raised digits: what a case's time and memory grow with."""
    alpha = -(-c["ell"] // c["dnum"])
    ndig = -(-c["level"] // alpha)
    return c["batch"] * ndig * (c["level"] + alpha) << c["log_n"]


_COST_MAX = 2 * 8 * 63 << 17  # two ciphertexts of (8, 2^17, 56)


def _log_int(rng, lo, hi):
    return min(hi, int(lo * ((hi + 1) / lo) ** rng.random()))


def draw(rng):
    while True:
        dnum, log_n = rng.randint(2, 8), rng.randint(13, 17)
        ell = max(dnum, _log_int(rng, 5, 56))
        level = ell if rng.random() < 0.6 else rng.randint(1, ell)
        op = rng.choice(("keyswitch", "keyswitch", "keyswitch", "hmul", "hrot", "graph", "steps", "raise"))
        plan = rng.choice(("tuned", "default"))
        c = _case("", op, dnum, log_n, ell, _log_int(rng, 1, 32), level, plan,
                  pow(5, rng.randint(1, 1000), 2 << log_n))
        del c["name"]
        if _cost(c) <= _COST_MAX:
            return c


@functools.lru_cache(maxsize=4)
def _handle(dnum, log_n, ell, level):
    G = ks.KsParams(dnum, log_n, ell)
    return G if level == ell else G.at_level(level)


@functools.lru_cache(maxsize=1)
def _table():
    return autotune.shipped_cache()


def _uniform(gen, shape, moduli):
    """[..., len(moduli), n] residues, uniform modulo each prime."""
    x = torch.randint(0, 1 << 62, shape, dtype=torch.int64, device="cuda", generator=gen)
    return x.remainder_(torch.tensor(moduli, dtype=torch.int64, device="cuda")[:, None])


def _inputs(case, seed, n, ndig_key, q, p, q_top):
    """The case's inputs: q the ciphertext's primes, q_top those of the key."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    b, op = case["batch"], case["op"]
    x = {}
    if op in ("hmul", "hrot"):
        x["a"] = _uniform(gen, (b, 2, len(q), n), q)
        if op == "hmul":
            x["b"] = _uniform(gen, (b, 2, len(q), n), q)
    else:
        x["d"] = _uniform(gen, (b, len(q), n), q)
    if op != "raise":
        x["evk"] = _uniform(gen, (ndig_key, 2, len(q_top) + len(p), n), q_top + p)
    return x


def prepare(case, seed):
    G = _handle(case["dnum"], case["log_n"], case["ell"], case["level"])
    top = _handle(case["dnum"], case["log_n"], case["ell"], case["ell"])
    b, sh = case["batch"], G.shapes(case["batch"])
    st = {"case": case, "G": G}
    st.update(_inputs(case, seed, G.n, sh["evk"][0], G.moduli[:G.ell], G.moduli[G.ell:], top.moduli[:top.ell]))
    empty = lambda *shape: torch.empty(shape, dtype=torch.int64, device="cuda")
    plan = autotune.plan_for(G, b, _table()) if case["plan"] == "tuned" else None
    st["plan"] = plan
    if case["op"] == "raise":
        a = min(G.alpha, G.ell)
        st["digit"], st["raised"] = empty(b, a, G.n), empty(b, G.nl - a, G.n)
        return st
    st["out"] = empty(*sh["out"])
    if case["op"] == "steps":
        st["ext"], st["acc"] = empty(*sh["ext"]), empty(*sh["acc"])
        st["ws"] = G.workspace(b, ks.make_plan(ks.STAGED))
    elif case["op"] in ("hmul", "hrot"):
        st["ws"] = G.eval_workspace(b, plan)
    else:
        st["ws"] = G.workspace(b, plan)
    if case["op"] == "graph":
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        st["graph"] = G.graph(st["d"], st["evk"], st["out"], b, st["ws"], plan, stream=s)
        s.synchronize()
    return st


def run(st):
    c, G, b = st["case"], st["G"], st["case"]["batch"]
    if c["op"] == "keyswitch":
        G.keyswitch(st["d"], st["evk"], st["out"], b, st["ws"], st["plan"])
        return st["out"]
    if c["op"] == "hmul":
        G.hmul(st["a"], st["b"], st["evk"], st["out"], b, st["ws"], st["plan"])
        return st["out"]
    if c["op"] == "hrot":
        G.hrot(st["a"], c["galois"], st["evk"], st["out"], b, st["ws"], st["plan"])
        return st["out"]
    if c["op"] == "graph":
        st["graph"].launch()
        return st["out"]
    if c["op"] == "steps":
        G.modup(st["d"], st["ext"], b, st["ws"])
        G.keymult(st["ext"], st["evk"], st["acc"], b)
        G.moddown(st["acc"], st["out"], b, st["ws"])
        return st["ext"], st["acc"], st["out"]
    # the first digit to coefficient form (on a copy: the NTT form stays in use), to the other primes, and back
    a = st["digit"].shape[1]
    st["digit"].copy_(st["d"][:, :a])
    G.intt(st["digit"], 0, a, b)
    G.bconv(st["digit"], 0, st["raised"], b)
    G.ntt(st["raised"], a, G.nl - a, b)
    return st["digit"], st["raised"]


def work(case):
    """Bytes: inputs, key rows of the level and outputs once, 8 a word.
    Operations: 4 a butterfly (a modular product as 2, an addition, a
    subtraction), 3 a multiply-add, 2 a product."""
    n, b, lv, op = 1 << case["log_n"], case["batch"], case["level"], case["op"]
    alpha = -(-case["ell"] // case["dnum"])
    nl, ndig = lv + alpha, -(-lv // alpha)
    digits = [min((j + 1) * alpha, lv) - j * alpha for j in range(ndig)]
    bfly = 4 * case["log_n"] / 2  # operations a coefficient of a transform
    if op == "raise":
        a = digits[0]
        return {"bytes": 8.0 * b * n * (2 * a + nl - a),
                "flops": float(b * n * (nl * bfly + a * 2 + a * (nl - a) * 3))}
    raised = sum(nl - a for a in digits)
    ops = (lv + raised + 2 * alpha + 2 * lv) * bfly
    ops += sum(a * 2 + a * (nl - a) * 3 for a in digits) + 2 * (alpha * 2 + alpha * lv * 3)
    ops += 2 * ndig * nl * 3 + 2 * lv * 3
    words = lv + 2 * lv
    if op == "hmul":
        words, ops = 4 * lv + 2 * lv, ops + 4 * lv * 3
    elif op == "hrot":
        words, ops = 2 * lv + 2 * lv, ops + lv
    elif op == "steps":
        words += 2 * ndig * nl + 2 * 2 * nl
    return {"bytes": 8.0 * n * (b * words + 2 * ndig * nl), "flops": float(b * n * ops)}


# ------------------------------------------- the same results in plain torch

def _mul30(a, c, q):
    """a*c mod q for 0 <= a < q < 2^60, 0 <= c <= 2^30: the quotient estimate is off by at most one."""
    k = (a.double() * c / q.double()).long()
    r = a * c - k * q
    r = torch.where(r < 0, r + q, r)
    return torch.where(r >= q, r - q, r)


def _mul(a, b, q):
    r = _mul30(_mul30(a, b >> 30, q), 1 << 30, q) + _mul30(a, b & ((1 << 30) - 1), q)
    return torch.where(r >= q, r - q, r)


def _is_prime(x):
    for s in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if x % s == 0:
            return x == s
    d, r = x - 1, 0
    while d % 2 == 0:
        d, r = d // 2, r + 1
    for a in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        y = pow(a, d, x)
        if y in (1, x - 1):
            continue
        for _ in range(r - 1):
            y = y * y % x
            if y == x - 1:
                break
        else:
            return False
    return True


@functools.lru_cache(maxsize=None)
def _primes(bits, log_n, count):
    step, out = 2 << log_n, []
    c = ((1 << bits) - 1) // step * step + 1
    if c >= 1 << bits:
        c -= step
    while len(out) < count:
        if _is_prime(c):
            out.append(c)
        c -= step
    return out


def _powers(g, q, n):
    """g^0 .. g^(n-1) mod q by doubling."""
    qt = torch.tensor(q, dtype=torch.int64, device="cuda")
    x = torch.ones(1, dtype=torch.int64, device="cuda")
    while x.numel() < n:
        f = torch.tensor(pow(g, x.numel(), q), dtype=torch.int64, device="cuda")
        x = torch.cat([x, _mul(x, f, qt)])
    return x[:n]


@functools.lru_cache(maxsize=256)
def _root(q, log_n):
    """The smallest primitive 2N-th root of unity mod q."""
    n = 1 << log_n
    g = next(c for x in range(2, 1000) for c in (pow(x, (q - 1) // (2 * n), q),) if pow(c, n, q) == q - 1)
    qt = torch.tensor(q, dtype=torch.int64, device="cuda")
    return int(_mul(_powers(g * g % q, q, n), torch.tensor(g, dtype=torch.int64, device="cuda"), qt).min())


def _brv(log_n):
    i = torch.arange(1 << log_n, device="cuda")
    r = torch.zeros_like(i)
    for b in range(log_n):
        r |= ((i >> b) & 1) << (log_n - 1 - b)
    return r


def _transform(x, primes, log_n, inverse):
    """x [items][limbs][N]: the negacyclic transform to bit-reversed order, or its inverse."""
    n, brv = 1 << log_n, _brv(log_n)
    q = torch.tensor(primes, dtype=torch.int64, device="cuda").view(1, -1, 1, 1)
    roots = [pow(_root(p, log_n), -1 if inverse else 1, p) for p in primes]
    tw = torch.stack([_powers(r, p, n)[brv] for r, p in zip(roots, primes)])[None]
    x = x.clone()
    for s in (range(log_n - 1, -1, -1) if inverse else range(log_n)):
        v = x.view(x.shape[0], x.shape[1], 1 << s, 2, n >> (s + 1))
        w = tw[:, :, 1 << s:2 << s, None]
        a, b = v[:, :, :, 0], v[:, :, :, 1]
        b = b if inverse else _mul(b, w, q)
        lo, hi = (a + b) % q, (a - b) % q
        x = torch.stack([lo, _mul(hi, w, q) if inverse else hi], 3).view(x.shape)
    if inverse:
        ninv = torch.tensor([pow(n, -1, p) for p in primes], dtype=torch.int64, device="cuda").view(1, -1, 1)
        x = _mul(x, ninv, q[..., 0])
    return x


def _col(vals):
    return torch.tensor(vals, dtype=torch.int64, device="cuda").view(1, -1, 1)


def _convert(x, src, dst):
    """Fast base conversion of x [items][src][N] (coefficients) to the primes dst."""
    hat = [functools.reduce(lambda u, v: u * v, (p for p in src if p != s), 1) for s in src]
    y = _mul(x, _col([pow(h, -1, s) for h, s in zip(hat, src)]), _col(src))
    out = []
    for t in dst:
        tt, z = _col([t]), 0
        for i, h in enumerate(hat):
            z = (z + _mul(y[:, i:i + 1] % tt, _col([h % t]), tt)) % tt
        out.append(z)
    return torch.cat(out, 1)


def exact(case, seed):
    """What run returns, from the definitions, with integer torch arithmetic."""
    n, log_n, ell, lv, op = 1 << case["log_n"], case["log_n"], case["ell"], case["level"], case["op"]
    alpha = -(-ell // case["dnum"])
    qtop, p = _primes(50, log_n, ell), _primes(60, log_n, alpha)
    q, key_digits = qtop[:lv], -(-ell // alpha)
    x = _inputs(case, seed, n, key_digits, q, p, qtop)
    basis = q + p
    digits = [(j * alpha, min((j + 1) * alpha, lv)) for j in range(-(-lv // alpha))]

    def others(lo, hi):
        return basis[:lo] + basis[hi:]

    if op == "raise":
        lo, hi = digits[0]
        c = _transform(x["d"][:, lo:hi], q[lo:hi], log_n, True)
        return c, _transform(_convert(c, q[lo:hi], others(lo, hi)), others(lo, hi), log_n, False)
    add = None
    if op == "hmul":
        a0, a1, b0, b1 = x["a"][:, 0], x["a"][:, 1], x["b"][:, 0], x["b"][:, 1]
        cq = _col(q)
        add = torch.stack([_mul(a0, b0, cq), (_mul(a0, b1, cq) + _mul(a1, b0, cq)) % cq], 1)
        d = _mul(a1, b1, cq)
    elif op == "hrot":
        brv = _brv(log_n)
        src = brv[((case["galois"] * (2 * brv + 1)) % (2 * n) - 1) // 2]
        add = torch.stack([x["a"][:, 0][..., src], torch.zeros_like(x["a"][:, 0])], 1)
        d = x["a"][:, 1][..., src]
    else:
        d = x["d"]
    coef, b, nl, cb = _transform(d, q, log_n, True), case["batch"], len(basis), _col(basis)
    rows = list(range(lv)) + list(range(ell, ell + alpha))
    ext = []
    for lo, hi in digits:
        r = _transform(_convert(coef[:, lo:hi], q[lo:hi], others(lo, hi)), others(lo, hi), log_n, False)
        ext.append(torch.cat([r[:, :lo], d[:, lo:hi], r[:, lo:]], 1))
    ext = torch.stack(ext, 1)
    acc = torch.zeros(b, 2, nl, n, dtype=torch.int64, device="cuda")
    for j in range(len(digits)):
        for c in range(2):
            acc[:, c] = (acc[:, c] + _mul(ext[:, j], x["evk"][j, c][rows][None], cb)) % cb
    ap = _transform(acc[:, :, lv:].reshape(2 * b, alpha, n), p, log_n, True)
    conv = _transform(_convert(ap, p, q), q, log_n, False).view(b, 2, lv, n)
    big = functools.reduce(lambda u, v: u * v, p, 1)
    cq, pinv = _col(q)[None], _col([pow(big, -1, t) for t in q])[None]
    out = _mul((acc[:, :, :lv] - conv) % cq, pinv, cq)
    if add is not None:
        out = (out + add) % cq
    return (ext, acc, out) if op == "steps" else out
