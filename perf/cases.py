"""The calls this library is measured on, from one small HMult to a 64-job batch.

Every case is a dict of plain values:

* ``kind``: what one pass calls (below);
* ``chain``: the prime chain, ``"Q+P"`` (number of ciphertext and of special
  primes); ``logN``: the ring degree; ``L``: the level (Q limbs) of the inputs;
* ``n``, ``giant``: how many rotations, jobs or multiplications the pass holds,
  where the kind has such a count.

Kinds:

* ``hmult``, ``hrot``: one homomorphic product / rotation;
* ``step``: HMult, rescale of its result, HRot of the first input;
* ``hoisted``: n rotations of one ciphertext that share its ModUp;
* ``lintrans``: one level of a linear transform in baby-step giant-step form
  (n hoisted rotations, ``giant`` plaintext sums, their rotations, the sum and
  a rescale);
* ``chain``: n squarings, each with its rescale;
* ``batch``: one launch of a captured batch: n HMults at level L under one key,
  or with ``mixed`` HMults, rotations and rescales at levels 4..L;
* ``staged``: a key-switch put together from its stages (ModUp, inner product,
  ModDown of both components);
* ``ntt``: a forward transform of one polynomial and an inverse one of another,
  all Q and P rows.

Residues are uniform below each row's prime: what ciphertexts and keys hold.
"""
from __future__ import annotations

import functools
import math
import random

import torch

import ckks_inputs as ci
import paper_2512_18345_amd as P

# prime chains: Q primes + P primes -> digits of the key (dnum)
DNUM = {"4+1": 4, "6+2": 3, "24+1": 24, "36+12": 3}


def listed():
    def case(name, kind, chain, logN, L, **more):
        return dict(name=name, kind=kind, chain=chain, logN=logN, L=L, **more)

    return [
        # the smallest call: one product on a small ring, launch and latency bound
        case("hmult_n12_l4", "hmult", "4+1", 12, 4),
        # the smallest ring with many small requests gathered into one launch
        case("batch16_n12_l4", "batch", "4+1", 12, 4, n=16, mixed=False),
        # a middle ring, a level that leaves the last digit almost empty (12 + 1 limbs)
        case("hmult_n14_l13", "hmult", "36+12", 14, 13),
        # a rotation on the serving ring, last digit partial
        case("hrot_n15_l25", "hrot", "36+12", 15, 25),
        # a rotation late in a computation, where few limbs are left
        case("hrot_n16_l7", "hrot", "36+12", 16, 7),
        # the benchmark's step at the full level
        case("step_n16_l36", "step", "36+12", 16, 36),
        # the baby steps of a linear transform
        case("hoisted16_n16_l36", "hoisted", "36+12", 16, 36, n=16),
        # a whole level of bootstrapping's linear transforms, second level down
        case("lintrans_n16_l35", "lintrans", "36+12", 16, 35, n=16, giant=4),
        # the multiplication chain between two transforms
        case("chain12_n16_l33", "chain", "36+12", 16, 33, n=12),
        # the mixed batch of requests at uneven levels
        case("batch64_n16", "batch", "36+12", 16, 36, n=64, mixed=True),
        # the stages of a key-switch as separate calls
        case("staged_n16_l36", "staged", "36+12", 16, 36),
        # the transforms as calls of their own (encoding, plaintext products)
        case("ntt_n16_l36", "ntt", "36+12", 16, 36),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    taken = [{k: v for k, v in c.items() if k != "name"} for c in listed()]
    c = _draw(rng)
    while c in taken:
        c = _draw(rng)
    return c


def _draw(rng):
    kind = rng.choice(["hmult", "hrot", "step", "hoisted", "lintrans", "chain", "batch", "staged", "ntt"])
    chain = rng.choice(["4+1", "6+2", "24+1"] + ["36+12"] * 5)
    logN = rng.choice([12, 13, 14, 15, 16, 16, 16]) if chain == "36+12" else 12
    top = int(chain.split("+")[0])
    c = dict(kind=kind, chain=chain, logN=logN, L=_log_int(rng, 2, top))
    if kind == "hoisted":
        c["n"] = _log_int(rng, 2, 17)
    elif kind == "lintrans":
        c.update(n=rng.randint(2, 16), giant=rng.randint(1, 4))
    elif kind == "chain":
        c["n"] = rng.randint(1, min(12, c["L"] - 1))
    elif kind == "batch":
        c["mixed"] = rng.random() < 0.5
        c["n"] = _log_int(rng, 2, 48 if c["mixed"] else 16)
        c["L"] = max(c["L"], 4)
    return c


def _spec(c):
    q, p = (int(x) for x in c["chain"].split("+"))
    return ci.chain_spec(c["chain"], c["logN"], q, p, DNUM[c["chain"]], 0, logN_max=16 if q == 36 else c["logN"])


def _jobs(c):
    """(op, L, rotation) of a batch's jobs: the same for every seed."""
    if not c["mixed"]:
        return [("HMULT", c["L"], 0)] * c["n"]
    rng = random.Random(c["n"])
    jobs = []
    for _ in range(c["n"]):
        op = rng.choices(["HMULT", "HROT", "RESCALE"], [4, 4, 2])[0]
        jobs.append((op, rng.randint(4, c["L"]), rng.randint(1, 8)))
    return jobs


class State:
    """Inputs, outputs and workspaces of a case, and its batch if it has one."""

    batch = None

    def __del__(self):
        if self.batch is not None:
            P.ckks_batch_destroy(self.batch)


@functools.lru_cache(maxsize=None)
def _context(chain, logN):
    return P.Context.from_spec(_spec(dict(chain=chain, logN=logN)))


class _Inputs:
    """Uniform residues of a spec's primes, drawn in order from one seed."""

    def __init__(self, spec, seed):
        self.spec = spec
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def rows(self, primes, *lead):
        q = torch.tensor(primes, dtype=torch.int64, device="cuda")[:, None]
        x = torch.randint(0, 1 << 62, (*lead, len(primes), self.spec.N), generator=self.g, device="cuda")
        return x.remainder_(q).to(torch.int32)

    def poly(self, L):
        return self.rows(self.spec.q[:L])

    def ct(self, L):
        return self.rows(self.spec.q[:L], 2)

    def key(self):
        return self.rows(self.spec.q + self.spec.p, self.spec.beta(self.spec.L_max), 2)


def _inputs(c, seed):
    """The inputs of a case by name: the same for a run and for its exact value."""
    spec, kind, L = _spec(c), c["kind"], c["L"]
    src, rng, half = _Inputs(spec, seed), random.Random(seed), 1 << (c["logN"] - 1)
    if kind == "hmult":
        return dict(ct1=src.ct(L), ct2=src.ct(L), rlk=src.key())
    if kind == "hrot":
        return dict(ct=src.ct(L), rot=rng.randrange(1, half), rotk=src.key())
    if kind == "step":
        return dict(ct1=src.ct(L), ct2=src.ct(L), rlk=src.key(), rot=rng.randrange(1, half), rotk=src.key())
    if kind == "hoisted":
        return dict(ct=src.ct(L), rots=list(range(1, c["n"] + 1)), keys=[src.key() for _ in range(c["n"])])
    if kind == "lintrans":
        n, g = c["n"], c["giant"]
        return dict(ct=src.ct(L), rots=list(range(1, n + 1)), keys=[src.key() for _ in range(n)],
                    pts=[[src.poly(L) for _ in range(n)] for _ in range(g)],
                    grots=[n * (i + 1) for i in range(g)], gkeys=[src.key() for _ in range(g)])
    if kind == "chain":
        return dict(ct=src.ct(L), rlk=src.key())
    if kind == "batch":
        keys = [src.key() for _ in range(9 if c["mixed"] else 1)]  # the last one relinearises, the others rotate
        jobs = [dict(op=op, L=l, rot=r, in0=src.ct(l), in1=src.ct(l) if op == "HMULT" else None,
                     key=keys[-1] if op == "HMULT" else keys[r - 1] if op == "HROT" else None)
                for op, l, r in _jobs(c)]
        return dict(jobs=jobs)
    if kind == "staged":
        return dict(d=src.poly(L), evk=src.key())
    return dict(a=src.rows(spec.q[:L] + spec.p), b=src.rows(spec.q[:L] + spec.p))


def prepare(case, seed):
    c, L, kind = case, case["L"], case["kind"]
    s = State()
    s.case, s.ctx = c, _context(c["chain"], c["logN"])
    s.h = s.ctx.handle
    s.__dict__.update(_inputs(c, seed))
    N, k, beta = s.ctx.N, s.ctx.k, s.ctx.beta(L)

    def empty(*shape):
        return torch.empty(shape, dtype=torch.int32, device="cuda")

    if kind in ("hmult", "hrot", "step", "chain"):
        s.ws = s.ctx.workspace("HMULT", L)
    if kind in ("hmult", "hrot"):
        s.out = empty(2, L, N)
    elif kind == "step":
        s.ws_rs = s.ctx.workspace("RESCALE", L)
        s.prod, s.scaled, s.rotated = empty(2, L, N), empty(2, L - 1, N), empty(2, L, N)
    elif kind in ("hoisted", "lintrans"):
        s.ws = s.ctx.workspace("HROT_HOISTED", L)
        s.outs = [empty(2, L, N) for _ in s.rots]
        if kind == "lintrans":
            s.ws_many = s.ctx.workspace("HROT", L, c["giant"])
            s.ws_rs = s.ctx.workspace("RESCALE", L)
            s.sums, s.turned = ([empty(2, L, N) for _ in s.grots] for _ in range(2))
            s.acc, s.out = empty(2, L, N), empty(2, L - 1, N)
    elif kind == "chain":
        s.ws_rs = s.ctx.workspace("RESCALE", L)
        s.prods = [empty(2, L - i, N) for i in range(c["n"])]
        s.cts = [empty(2, L - i - 1, N) for i in range(c["n"])]
    elif kind == "batch":
        for j in s.jobs:
            j["out"] = empty(2, j["L"] - (j["op"] == "RESCALE"), N)
        s.batch = P.ckks_batch_create(s.h, [dict(j, op=P.JOB[j["op"]]) for j in s.jobs], use_graph=True)
    elif kind == "staged":
        s.ws_up, s.ws_down = s.ctx.workspace("MODUP", L), s.ctx.workspace("MODDOWN", L)
        s.M, s.acc, s.out = empty(beta, L + k, N), empty(2, L + k, N), empty(2, L, N)
    return s


def run(s):
    c, h, L, kind = s.case, s.h, s.case["L"], s.case["kind"]
    if kind == "hmult":
        P.ckks_hmult(h, s.ct1, s.ct2, L, s.rlk, s.out, s.ws)
        return s.out
    if kind == "hrot":
        P.ckks_hrot(h, s.ct, L, s.rot, s.rotk, s.out, s.ws)
        return s.out
    if kind == "step":
        P.ckks_hmult(h, s.ct1, s.ct2, L, s.rlk, s.prod, s.ws)
        P.ckks_rescale(h, s.prod, L, s.scaled, s.ws_rs)
        P.ckks_hrot(h, s.ct1, L, s.rot, s.rotk, s.rotated, s.ws)
        return s.prod, s.scaled, s.rotated
    if kind == "hoisted":
        P.ckks_hrot_hoisted(h, s.ct, L, s.rots, s.keys, s.outs, s.ws)
        return s.outs
    if kind == "lintrans":
        P.ckks_hrot_hoisted(h, s.ct, L, s.rots, s.keys, s.outs, s.ws)
        P.ckks_pmult_sums(h, s.outs, s.pts, L, s.sums)
        P.ckks_hrot_many(h, s.sums, L, s.grots, s.gkeys, s.turned, s.ws_many)
        total = s.turned[0]
        for t in s.turned[1:]:
            P.ckks_add(h, total, t, L, s.acc)
            total = s.acc
        P.ckks_rescale(h, total, L, s.out, s.ws_rs)
        return [s.out, *s.sums]
    if kind == "chain":
        ct = s.ct
        for i in range(c["n"]):
            P.ckks_hmult(h, ct, ct, L - i, s.rlk, s.prods[i], s.ws)
            P.ckks_rescale(h, s.prods[i], L - i, s.cts[i], s.ws_rs)
            ct = s.cts[i]
        return ct
    if kind == "batch":
        P.ckks_batch_launch(s.batch)
        return [j["out"] for j in s.jobs]
    if kind == "staged":
        P.ckks_modup(h, s.d, L, s.M, s.ws_up)
        P.ckks_inner_product(h, s.M, L, s.evk, s.acc)
        for i in range(2):
            P.ckks_moddown(h, s.acc[i], L, s.out[i], s.ws_down)
        return s.out
    P.ckks_ntt(h, s.a, L, True)
    P.ckks_intt(h, s.b, L, True)
    return s.a, s.b


def work(case):
    """Words in and out once, and the additions and multiplications of residues."""
    c, spec, L, kind = case, _spec(case), case["L"], case["kind"]
    N, k, alpha = spec.N, spec.k, spec.alpha
    fly = 3 * N // 2 * c["logN"]  # a transform: one product and two sums a butterfly

    def key(l):
        return 2 * spec.beta(l) * (l + k)

    def up(l):  # ModUp: transforms back and forth, base conversion
        b = spec.beta(l)
        return (b * (l + k)) * fly + 2 * N * l * (l + k - alpha)

    def down(l):  # inner product and ModDown of both components
        return 2 * (k + l) * fly + 4 * N * k * l + 2 * N * key(l) + 2 * 3 * N * l

    def rescale(l):
        return 2 * l * fly + 2 * 2 * N * l

    limbs, ops = 0, 0
    if kind in ("hmult", "step"):
        limbs, ops = 4 * L + key(L) + 2 * L, up(L) + down(L) + 5 * N * L
    if kind == "step":  # the first input and the product are there already
        limbs, ops = limbs + 2 * (L - 1) + key(L) + 2 * L, 2 * ops + rescale(L)
    elif kind == "hrot":
        limbs, ops = 2 * L + key(L) + 2 * L, up(L) + down(L)
    elif kind == "hoisted":
        limbs, ops = 2 * L + c["n"] * (key(L) + 2 * L), up(L) + c["n"] * down(L)
    elif kind == "lintrans":
        n, g = c["n"], c["giant"]
        limbs = 2 * L + (n + g) * key(L) + n * g * L + 2 * (L - 1)
        ops = (1 + g) * up(L) + (n + g) * down(L) + 4 * N * L * n * g + rescale(L)
    elif kind == "chain":
        limbs = 2 * L + key(L) + 2 * (L - c["n"])
        ops = sum(up(l) + down(l) + 5 * N * l + rescale(l) for l in range(L, L - c["n"], -1))
    elif kind == "batch":
        rows = {}  # rows of each key that some job reads
        for op, l, r in _jobs(c):
            if op == "RESCALE":
                limbs, ops = limbs + 2 * l + 2 * (l - 1), ops + rescale(l)
                continue
            which = r if op == "HROT" else 0
            rows[which] = max(rows.get(which, 0), key(l))
            limbs += (4 if op == "HMULT" else 2) * l + 2 * l
            ops += up(l) + down(l)
        limbs += sum(rows.values())
    elif kind == "staged":
        limbs, ops = L + key(L) + 2 * L, up(L) + down(L)
    elif kind == "ntt":
        limbs, ops = 4 * (L + k), 2 * (L + k) * fly
    return {"bytes": 4 * N * limbs, "flops": ops}


# ----- the same values in plain 64-bit arithmetic -----------------------------

@functools.lru_cache(maxsize=None)
def _powers(q, logN):
    """psi^e, e < 2N, of the smallest primitive 2N-th root of unity mod q."""
    N, x = 1 << logN, 2
    while pow(x, (q - 1) // 2, q) == 1:
        x += 1
    pw = torch.ones(1, dtype=torch.int64)
    step = pow(x, (q - 1) // (2 * N), q)
    root = step
    for _ in range(logN + 1):
        pw = torch.cat([pw, pw * step % q])
        step = step * step % q
    psi = int(pw[1::2].min())
    e = int((pw == psi).nonzero()[0])
    return pw[torch.arange(2 * N) * e % (2 * N)] if psi != root else pw


@functools.lru_cache(maxsize=None)
def _brv(logN):
    i, out = torch.arange(1 << logN), torch.zeros(1 << logN, dtype=torch.int64)
    for b in range(logN):
        out |= ((i >> b) & 1) << (logN - 1 - b)
    return out


class _Exact:
    def __init__(self, c):
        self.spec, self.logN = _spec(c), c["logN"]
        self.N, self.k, self.alpha = self.spec.N, self.spec.k, self.spec.alpha
        self.q, self.p = list(self.spec.q), list(self.spec.p)

    @staticmethod
    def col(primes):
        return torch.tensor(primes, dtype=torch.int64, device="cuda")[:, None]

    def twiddles(self, primes, sign):
        at = (sign * _brv(self.logN)) % (2 * self.N)
        return torch.stack([_powers(q, self.logN)[at] for q in primes]).cuda()

    def ntt(self, a, primes):
        q, w, n = self.col(primes)[:, :, None], self.twiddles(primes, 1), len(primes)
        m = 1
        while m < self.N:
            a = a.view(n, m, 2, -1)
            t = a[:, :, 1] * w[:, m:2 * m, None] % q
            a = torch.stack([(a[:, :, 0] + t) % q, (a[:, :, 0] - t) % q], 2)
            m *= 2
        return a.reshape(n, self.N)

    def intt(self, a, primes):
        q, w, n = self.col(primes)[:, :, None], self.twiddles(primes, -1), len(primes)
        m = self.N // 2
        while m:
            a = a.reshape(n, m, 2, -1)
            x, y = a[:, :, 0], a[:, :, 1]
            a = torch.stack([(x + y) % q, (x - y) % q * w[:, m:2 * m, None] % q], 2)
            m //= 2
        return a.reshape(n, self.N) * self.col([pow(self.N, -1, v) for v in primes]) % self.col(primes)

    def bconv(self, x, src, dst):
        x = x * self.col([pow(math.prod(src) // v, -1, v) for v in src]) % self.col(src)
        rows = [sum(x[i] * (math.prod(src) // v % t) % t for i, v in enumerate(src)) % t for t in dst]
        return torch.stack(rows)

    def modup(self, d, L):
        rows, out = self.q[:L] + self.p, []
        for lo in range(0, L, self.alpha):
            src = self.q[lo:min(lo + self.alpha, L)]
            dst = rows[:lo] + rows[lo + len(src):]
            z = self.ntt(self.bconv(self.intt(d[lo:lo + len(src)], src), src, dst), dst)
            out.append(torch.cat([z[:lo], d[lo:lo + len(src)], z[lo:]]))
        return out

    def inner(self, M, key, L):
        at = list(range(L)) + list(range(len(self.q), len(self.q) + self.k))
        q = self.col(self.q[:L] + self.p)
        return [sum(m * key[j, c, at].long() % q for j, m in enumerate(M)) % q for c in range(2)]

    def moddown(self, a, L):
        Q = self.q[:L]
        z = self.ntt(self.bconv(self.intt(a[L:], self.p), self.p, Q), Q)
        return (a[:L] - z) % self.col(Q) * self.col([pow(math.prod(self.p), -1, v) for v in Q]) % self.col(Q)

    def keyswitch(self, M, key, L):
        return torch.stack([self.moddown(a, L) for a in self.inner(M, key, L)])

    def hmult(self, a, b, L, key):
        a, b, q = a.long(), b.long(), self.col(self.q[:L])
        ks = self.keyswitch(self.modup(a[1] * b[1] % q, L), key, L)
        return (ks + torch.stack([a[0] * b[0] % q, (a[0] * b[1] % q + a[1] * b[0]) % q])) % q

    def turn(self, a, rot):
        g, brv = pow(5, rot % (self.N // 2), 2 * self.N), _brv(self.logN)
        return a[..., brv[(g * (2 * brv + 1) % (2 * self.N) - 1) // 2].cuda()]

    def hrot(self, ct, L, rot, key, M=None):
        ct = ct.long()
        M = self.modup(self.turn(ct[1], rot), L) if M is None else [self.turn(m, rot) for m in M]
        ks = self.keyswitch(M, key, L)
        return torch.stack([(ks[0] + self.turn(ct[0], rot)) % self.col(self.q[:L]), ks[1]])

    def rescale(self, ct, L):
        Q, top, ct = self.q[:L - 1], self.q[L - 1], ct.long()
        inv = self.col([pow(top, -1, v) for v in Q])
        t = [self.ntt(self.intt(x[L - 1:], [top]) % self.col(Q), Q) for x in ct]
        return (ct[:, :L - 1] - torch.stack(t)) % self.col(Q) * inv % self.col(Q)


def exact(case, seed):
    c, L, kind = case, case["L"], case["kind"]
    E, i = _Exact(c), _inputs(c, seed)
    out = None
    if kind == "hmult":
        out = E.hmult(i["ct1"], i["ct2"], L, i["rlk"])
    elif kind == "hrot":
        out = E.hrot(i["ct"], L, i["rot"], i["rotk"])
    elif kind == "step":
        prod = E.hmult(i["ct1"], i["ct2"], L, i["rlk"])
        out = prod, E.rescale(prod, L), E.hrot(i["ct1"], L, i["rot"], i["rotk"])
    elif kind in ("hoisted", "lintrans"):
        M = E.modup(i["ct"][1].long(), L)
        out = [E.hrot(i["ct"], L, r, k, M) for r, k in zip(i["rots"], i["keys"])]
        if kind == "lintrans":
            q = E.col(E.q[:L])
            sums = [sum(x * p.long() % q for x, p in zip(out, pts)) % q for pts in i["pts"]]
            total = sum(E.hrot(x, L, r, k) for x, r, k in zip(sums, i["grots"], i["gkeys"])) % q
            out = [E.rescale(total, L), *sums]
    elif kind == "chain":
        out = i["ct"]
        for l in range(L, L - c["n"], -1):
            out = E.rescale(E.hmult(out, out, l, i["rlk"]), l)
    elif kind == "batch":
        out = [E.hmult(j["in0"], j["in1"], j["L"], j["key"]) if j["op"] == "HMULT" else
               E.hrot(j["in0"], j["L"], j["rot"], j["key"]) if j["op"] == "HROT" else
               E.rescale(j["in0"], j["L"]) for j in i["jobs"]]
    elif kind == "staged":
        out = E.keyswitch(E.modup(i["d"].long(), L), i["evk"], L)
    else:
        primes = E.q[:L] + E.p
        out = E.ntt(i["a"].long(), primes), E.intt(i["b"].long(), primes)
    if isinstance(out, (list, tuple)):
        return [x.to(torch.int32) for x in out]
    return out.to(torch.int32)
