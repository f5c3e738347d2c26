"""GPU parity of key-switches of more than four digits that are not hoisted: the
inner product takes such digits in turn (the pipeline's general kernel, P rows and
Q rows with ModDown's combine; at N = 2^12 the whole-limb kernel's group of several
digits), folding its 64-bit sums after every eighth digit.  Levels on both sides of
a step of the digit count: five digits, eight, nine, a partial last one, all.

Bit-exact against the oracle on every residue (tolerance 0)."""
import pytest
import torch

import ckks_inputs as ci
import oracle as O
import paper_2512_18345_amd as P
from gpu_helpers import dev, empty, first_mismatch, host

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# logN, Q primes, digit size (= P primes), schedule bit 8 or the pipeline, levels
CASES = [(12, 24, 1, 0, (5, 9, 24)), (12, 10, 2, 0, (9, 10)), (13, 20, 2, 0, (9, 16, 17, 20)), (13, 21, 4, 0, (17, 21)),
         (14, 9, 1, 0, (5, 8, 9)), (15, 6, 1, 0, (5, 6)), (16, 25, 5, 0, (21, 25)),
         (12, 10, 2, 8, (9, 10)), (12, 36, 1, 8, (29, 32, 36)), (12, 36, 2, 8, (17, 35))]


@pytest.mark.parametrize("logN,primes,alpha,shape,levels", CASES)
def test_many_digits(logN, primes, alpha, shape, levels):
    spec = ci.chain_spec("many", logN, primes, alpha, -(-primes // alpha), 900 + primes)
    par, ctx, rng = O.Params.from_spec(spec), P.Context.from_spec(spec), ci.Rng(spec.seed)
    h, N = ctx.handle, spec.N
    P.ckks_ctx_set_schedule(h, 12, 6, 128, shape)
    key = rng.evk(spec)
    d_key = dev(key)
    for L in levels:
        assert spec.beta(L) > 4
        ct1, ct2, rot = rng.polys(2, spec.q[:L], N), rng.polys(2, spec.q[:L], N), rng.rotation(N)
        out = empty(2, L, N)
        P.ckks_keyswitch(h, dev(ct1[0]), L, d_key, out, ctx.workspace("KEYSWITCH", L))
        msg = first_mismatch(host(out), O.keyswitch(par, ct1[0], L, key))
        assert not msg, f"keyswitch L={L}: {msg}"
        P.ckks_hmult(h, dev(ct1), dev(ct2), L, d_key, out, ctx.workspace("HMULT", L))
        msg = first_mismatch(host(out), O.hmult(par, ct1, ct2, L, key))
        assert not msg, f"hmult L={L}: {msg}"
        P.ckks_hrot(h, dev(ct1), L, rot, d_key, out, ctx.workspace("HROT", L))
        msg = first_mismatch(host(out), O.hrot(par, ct1, L, rot, key))
        assert not msg, f"hrot L={L}: {msg}"


@pytest.mark.parametrize("shape", [0, 8])
@pytest.mark.parametrize("kind", ["max", "one_hot"])
def test_many_digits_of_extreme_words(kind, shape):
    """36 digits of one limb, every input and key word the largest there is (or
    all but one zero): the largest sums between two folds."""
    spec = ci.chain_spec("extreme", 12, 36, 1, 36, 11)
    par, ctx = O.Params.from_spec(spec), P.Context.from_spec(spec)
    h, N, L = ctx.handle, spec.N, spec.L_max
    P.ckks_ctx_set_schedule(h, 12, 6, 128, shape)
    d, key = ci.edge_residues(kind, spec.q, N, 5), ci.edge_evk("max", spec)
    out = empty(2, L, N)
    P.ckks_keyswitch(h, dev(d), L, dev(key), out, ctx.workspace("KEYSWITCH", L))
    msg = first_mismatch(host(out), O.keyswitch(par, d, L, key))
    assert not msg, msg


@pytest.mark.parametrize("use_graph", [True, False])
def test_split_batch_of_many_digits(use_graph):
    """Jobs of 5 to 24 digits in one launch of the general kernel, each against the
    same job alone through the whole-limb kernels, one against the oracle."""
    spec = ci.get("n12_l24_k1")
    par, ctx, rng = O.Params.from_spec(spec), P.Context.from_spec(spec), ci.Rng(spec.seed + 600)
    h, N = ctx.handle, spec.N
    key = rng.evk(spec)
    d_key = dev(key)
    jobs, want = [], []
    for i, L in enumerate([24, 5, 9, 3, 16, 17]):
        ct1, ct2 = dev(rng.polys(2, spec.q[:L], N)), dev(rng.polys(2, spec.q[:L], N))
        ref = empty(2, L, N)
        op = ["HMULT", "HROT", "KEYSWITCH"][i % 3]
        if op == "HMULT":
            P.ckks_hmult(h, ct1, ct2, L, d_key, ref, ctx.workspace("HMULT", L))
        elif op == "HROT":
            P.ckks_hrot(h, ct1, L, 7, d_key, ref, ctx.workspace("HROT", L))
        else:
            P.ckks_keyswitch(h, ct1[0].contiguous(), L, d_key, ref, ctx.workspace("KEYSWITCH", L))
        want.append(host(ref))
        jobs.append(dict(op=P.JOB[op], L=L, rot=7, in0=ct1[0].contiguous() if op == "KEYSWITCH" else ct1,
                         in1=ct2 if op == "HMULT" else None, key=d_key, out=empty(2, L, N)))
    msg = first_mismatch(want[0], O.hmult(par, host(jobs[0]["in0"]), host(jobs[0]["in1"]), 24, key))
    assert not msg, msg
    b = P.ckks_batch_create(h, jobs, use_graph=use_graph)
    try:
        P.ckks_batch_set_plan(b, 0, 1, 1)
        for rep in range(3):  # graph replays with eager work and syncs in between
            for j in jobs:
                j["out"].fill_(-1)
            P.ckks_batch_launch(b)
            torch.cuda.synchronize()
            for i, j in enumerate(jobs):
                msg = first_mismatch(host(j["out"]), want[i])
                assert not msg, f"replay {rep}, job {i} (L={j['L']}): {msg}"
    finally:
        P.ckks_batch_destroy(b)
