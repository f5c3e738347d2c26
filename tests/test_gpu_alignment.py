"""Every pointer of a call at a 4-byte offset: inputs, keys, outputs and the
workspace are read and written in 16-byte quads, but need only be 4-byte aligned.

Bit-exact against the oracle on every residue (tolerance 0), and the words on
both sides of an output are left alone."""
import pytest
import torch

import ckks_inputs as ci
import oracle as O
import paper_2512_18345_amd as P
from gpu_helpers import dev, first_mismatch, host

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


class Room:
    """An output of the given shape one word past a 16-byte boundary, a word of room on each side."""

    def __init__(self, *shape):
        n = 1
        for s in shape:
            n *= s
        self.all = torch.full((n + 8,), -1, dtype=torch.int32, device="cuda")
        self.t = self.all[1:n + 1].view(shape)
        assert self.t.data_ptr() % 16 == 4

    def check(self, want, what):
        got = host(self.all)
        n = want.size
        msg = first_mismatch(got[1:n + 1].reshape(want.shape), want)
        assert not msg, f"{what}: {msg}"
        assert got[0] == 0xffffffff and (got[n + 1:] == 0xffffffff).all(), f"{what}: a word beside the output changed"


def shifted(a):
    r = Room(*a.shape)
    r.t.copy_(dev(a))
    return r.t


@pytest.mark.parametrize("name,logN,shape", [("n12_l4", 12, 8), ("toy_n12", 12, 0), ("n12_l24_k1", 12, 0),
                                             ("n16_l36", 13, 0), ("n16_l36", 16, 0)])
def test_pointers_at_a_four_byte_offset(name, logN, shape):
    base = ci.get(name)
    spec = ci.ChainSpec(base.name, logN, base.q, base.p, base.dnum, base.seed)
    par, ctx, rng = O.Params.from_spec(spec), P.Context.from_spec(spec), ci.Rng(spec.seed + 700)
    h, N, k = ctx.handle, spec.N, spec.k
    P.ckks_ctx_set_schedule(h, 12, 6, 128, shape)
    L = min(spec.L_max, 13)
    R = L + k
    q, beta = spec.q[:L], spec.beta(L)

    def ws(op):
        return Room(P.ckks_workspace_bytes(h, P.OP[op], L) // 4).t

    a = rng.polys(1, list(q) + list(spec.p), N)[0]
    r = Room(R, N)
    r.t.copy_(dev(a))
    P.ckks_ntt(h, r.t, L, with_P=True)
    r.check(O.ntt(par, a, list(q) + list(spec.p)), "ntt")
    r.t.copy_(dev(a))
    P.ckks_intt(h, r.t, L, with_P=True)
    r.check(O.intt(par, a, list(q) + list(spec.p)), "intt")

    ct1, ct2 = rng.polys(2, q, N), rng.polys(2, q, N)
    r = Room(2, L - 1, N)
    P.ckks_rescale(h, shifted(ct1), L, r.t, ws("RESCALE"))
    r.check(O.rescale(par, ct1, L), "rescale")
    r = Room(beta, R, N)
    P.ckks_modup(h, shifted(ct1[0]), L, r.t, ws("MODUP"))
    r.check(O.modup(par, ct1[0], L), "modup")
    r = Room(L, N)
    P.ckks_moddown(h, shifted(a), L, r.t, ws("MODDOWN"))
    r.check(O.moddown(par, a, L), "moddown")

    key = rng.evk(spec)
    d_key = shifted(key)
    r = Room(2, L, N)
    P.ckks_keyswitch(h, shifted(ct1[0]), L, d_key, r.t, ws("KEYSWITCH"))
    r.check(O.keyswitch(par, ct1[0], L, key), "keyswitch")
    r = Room(2, L, N)
    P.ckks_hmult(h, shifted(ct1), shifted(ct2), L, d_key, r.t, ws("HMULT"))
    r.check(O.hmult(par, ct1, ct2, L, key), "hmult")
    r = Room(2, L, N)
    P.ckks_hrot(h, shifted(ct1), L, 3, d_key, r.t, ws("HROT"))
    r.check(O.hrot(par, ct1, L, 3, key), "hrot")
    outs = [Room(2, L, N) for _ in range(2)]
    P.ckks_hrot_hoisted(h, shifted(ct1), L, [1, 3], [d_key, d_key], [o.t for o in outs], ws("HROT_HOISTED"))
    for o, w in zip(outs, O.hrot_hoisted(par, ct1, L, [1, 3], [key, key])):
        o.check(w, "hoisted")
