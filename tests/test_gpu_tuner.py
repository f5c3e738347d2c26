"""The tuners choose among launches that differ: they reach every pipeline a
call can take, whatever plan and schedule they start from."""
import pytest
import torch

import ckks_inputs as ci
import paper_2512_18345_amd as P
from gpu_helpers import dev, empty, first_mismatch, host

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("use_graph", [True, False])
@pytest.mark.parametrize("shape", [0, 8])
def test_batch_tuner_reaches_the_whole_limb_kernels(shape, use_graph):
    """Eight HMults at N = 2^12, digit size 1, take the whole-limb kernels about
    20 us and the pipeline 34, so the tuner must end with split 0 and ntt_shape
    bit 8 also for a batch created without that bit (whose plan is split)."""
    spec = ci.get("n12_l4")
    ctx = P.Context.from_spec(spec)
    h, N, L = ctx.handle, spec.N, spec.L_max
    rng = ci.Rng(spec.seed + 500)
    key = dev(rng.evk(spec))
    ins = [dev(rng.polys(2, spec.q, N)) for _ in range(9)]
    want = empty(2, L, N)
    jobs = [dict(op=P.JOB["HMULT"], L=L, in0=ins[i], in1=ins[i + 1], key=key, out=empty(2, L, N)) for i in range(8)]
    P.ckks_ctx_set_schedule(h, 12, 6, 128, shape)
    b = P.ckks_batch_create(h, jobs, use_graph=use_graph)
    try:
        assert P.ckks_batch_get_plan(b)["split"] == (0 if shape else 1)
        plan, us = P.ckks_batch_tune(b, reps=20)
        assert plan == P.ckks_batch_get_plan(b) and plan in [p for p, _ in P.ckks_batch_tune_log(b)]
        assert plan["split"] == 0 and P.ckks_batch_get_schedule(b)["ntt_shape"] == 8, (plan, us)
        assert P.ckks_ctx_get_schedule(h)["ntt_shape"] == shape
        for rep in range(3):  # graph replays with eager work and syncs in between
            for j in jobs:
                j["out"].fill_(-1)
            P.ckks_batch_launch(b)
            for i, j in enumerate(jobs):
                P.ckks_hmult(h, ins[i], ins[i + 1], L, key, want, ctx.workspace("HMULT", L))
                msg = first_mismatch(host(j["out"]), host(want))
                assert not msg, f"replay {rep}, job {i}: {msg}"
    finally:
        P.ckks_batch_destroy(b)


def test_schedule_tuner_keeps_the_default_among_equals():
    """At N = 2^12, digit size 1, every candidate with bit 8 is one launch
    sequence (the whole-limb kernels, 19 us against the pipeline's 31): the tuner
    must not choose among its names, but keep the default's."""
    spec = ci.get("n12_l4")
    ctx = P.Context.from_spec(spec)
    default = P.ckks_ctx_get_schedule(ctx.handle)
    assert default == dict(bconv_up_rows=12, bconv_down_rows=6, small_grid=128, ntt_shape=8)
    for start in (default, dict(bconv_up_rows=2, bconv_down_rows=2, small_grid=0, ntt_shape=0)):
        P.ckks_ctx_set_schedule(ctx.handle, **start)
        best, us = P.ckks_ctx_tune(ctx.handle, spec.L_max, reps=20)
        assert us > 0 and best == default, best


@pytest.mark.parametrize("logN,L", [(12, 13), (16, 36)])
def test_tuners_time_a_launch_sequence_once(logN, L):
    """With 36 + 12 primes at most 47 rows make one row group under a cap of 8 x 12
    or 8 x 6 rows, the grids pass 128 work-groups or none of them does, and at
    N = 2^12 digits of 12 limbs have no whole-limb kernels: the candidates that
    differ in such a field alone launch the same, and only the first may be chosen."""
    base = ci.get("n16_l36")
    spec = ci.ChainSpec(base.name, logN, base.q, base.p, base.dnum, base.seed)
    ctx = P.Context.from_spec(spec)
    h, N = ctx.handle, spec.N
    shape = 8 if logN == 12 else 0
    best, _ = P.ckks_ctx_tune(h, L, reps=2)
    assert best["ntt_shape"] == shape, best
    if logN == 16:
        assert best["bconv_up_rows"] != 6 and best["bconv_down_rows"] != 12 and best["small_grid"] != 0, best
    P.ckks_ctx_set_schedule(h, 12, 6, 128, shape)
    ct = torch.zeros(2, L, N, dtype=torch.int32, device="cuda")
    key = torch.zeros(spec.beta(spec.L_max), 2, spec.L_max + spec.k, N, dtype=torch.int32, device="cuda")
    jobs = [dict(op=P.JOB["HMULT"], L=L, in0=ct, in1=ct, key=key, out=empty(2, L, N)) for _ in range(3)]
    b = P.ckks_batch_create(h, jobs, use_graph=False)
    try:
        P.ckks_batch_tune(b, reps=2)
        s = P.ckks_batch_get_schedule(b)
        assert s["ntt_shape"] == shape and (s["bconv_up_rows"], s["bconv_down_rows"]) != (12, 12), s
    finally:
        P.ckks_batch_destroy(b)
