"""GPU parity of the fused column kernels (INTT columns, base conversion, NTT
columns of ModUp and ModDown) at the sizes where their split can go wrong:
digit sizes on both sides of a step of four limbs, of an even count and of the
12 past which the sum takes one more correction; one limb, a full digit, one
limb past it and every limb; every ring degree's tile width.

Bit-exact against the oracle on every residue (tolerance 0)."""
import numpy as np
import pytest
import torch

import ckks_inputs as ci
import oracle as O
import paper_2512_18345_amd as P
from gpu_helpers import dev, empty, first_mismatch, host

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("logN,alpha", [(12, 1), (12, 3), (12, 16), (13, 2), (13, 5), (13, 13),
                                        (14, 4), (14, 12), (15, 9), (16, 1), (16, 7)])
def test_column_kernels_at_every_digit_size(logN, alpha):
    spec = ci.chain_spec(f"a{alpha}", logN, 2 * alpha, alpha, 2, 100 + alpha)
    par, ctx, rng = O.Params.from_spec(spec), P.Context.from_spec(spec), ci.Rng(spec.seed)
    h, N = ctx.handle, spec.N
    P.ckks_ctx_set_schedule(h)  # the pipeline at N = 2^12 too, not the whole-limb kernels
    key = rng.evk(spec)
    d_key = dev(key)
    for L in sorted({1, alpha, alpha + 1, 2 * alpha}):
        ct1, ct2 = rng.polys(2, spec.q[:L], N), rng.polys(2, spec.q[:L], N)
        rot = rng.rotation(N)
        out = empty(2, L, N)
        P.ckks_hmult(h, dev(ct1), dev(ct2), L, d_key, out, ctx.workspace("HMULT", L))
        msg = first_mismatch(host(out), O.hmult(par, ct1, ct2, L, key))
        assert not msg, f"hmult N=2^{logN} digit {alpha} L={L}: {msg}"
        P.ckks_hrot(h, dev(ct1), L, rot, d_key, out, ctx.workspace("HROT", L))
        msg = first_mismatch(host(out), O.hrot(par, ct1, L, rot, key))
        assert not msg, f"hrot N=2^{logN} digit {alpha} L={L}: {msg}"
        outs = [empty(2, L, N) for _ in range(2)]
        P.ckks_hrot_hoisted(h, dev(ct1), L, [rot, 1], [d_key, d_key], outs, ctx.workspace("HROT_HOISTED", L))
        for o, w in zip(outs, O.hrot_hoisted(par, ct1, L, [rot, 1], [key, key])):
            msg = first_mismatch(host(o), w)
            assert not msg, f"hoisted N=2^{logN} digit {alpha} L={L}: {msg}"


@pytest.mark.parametrize("name,L", [("n12_l4", 4), ("toy_n12", 5), ("n16_l36", 13)])
def test_rotations_of_a_ciphertext_at_a_four_byte_offset(name, L):
    """The automorphism reads and the outputs are written as 16-byte quads;
    ciphertexts need only be 4-byte aligned."""
    spec = ci.get(name)
    par, ctx, rng = O.Params.from_spec(spec), P.Context.from_spec(spec), ci.Rng(77)
    h, N = ctx.handle, spec.N
    ct, key = rng.polys(2, spec.q[:L], N), rng.evk(spec)
    room = torch.empty(1 + ct.size, dtype=torch.int32, device="cuda")
    shifted = room[1:].view(2, L, N)
    shifted.copy_(dev(ct))
    assert shifted.data_ptr() % 16 == 4
    out = torch.empty(1 + ct.size, dtype=torch.int32, device="cuda")[1:].view(2, L, N)
    for rot in (0, 1, 2, 3, N // 2 - 1):
        P.ckks_hrot(h, shifted, L, rot, dev(key), out, ctx.workspace("HROT", L))
        msg = first_mismatch(host(out), O.hrot(par, ct, L, rot, key))
        assert not msg, f"hrot by {rot}: {msg}"
        P.ckks_hrot_hoisted(h, shifted, L, [rot], [dev(key)], [out], ctx.workspace("HROT_HOISTED", L))
        msg = first_mismatch(host(out), O.hrot_hoisted(par, ct, L, [rot], [key])[0])
        assert not msg, f"hoisted rotation by {rot}: {msg}"


@pytest.mark.parametrize("alpha", [4, 5, 11, 16])
def test_conversions_of_extreme_words(alpha):
    """Scaled inputs whose words, or every byte of them, are the largest and the
    smallest there are, over all limbs at once: the largest sums."""
    spec = ci.chain_spec(f"x{alpha}", 13, 2 * alpha, alpha, 2, 7)
    par, ctx = O.Params.from_spec(spec), P.Context.from_spec(spec)
    h, N, L = ctx.handle, spec.N, alpha + 2
    low = 128 * (1 + (1 << 8) + (1 << 16))

    def words(primes):  # coefficients that the pre-multiplier turns into these words
        rows = []
        for q in primes:
            rest = 1
            for t in primes:
                rest = rest * (t if t != q else 1) % q
            y = [q - 1, 0, (63 << 24) - low, (63 << 24) + 127 * (low >> 7), 1, (q - 1) // 2, low, 128]
            rows.append([w % q * rest % q for w in y])
        return np.tile(np.array(rows, dtype=np.uint32), (1, N // 8))

    d = np.concatenate([words(spec.q[r.start:r.stop]) for r in par.digits(L)])
    d = O.ntt(par, d, spec.q[:L])
    out = empty(par.beta(L), L + alpha, N)
    P.ckks_modup(h, dev(d), L, out, ctx.workspace("MODUP", L))
    msg = first_mismatch(host(out), O.modup(par, d, L))
    assert not msg, f"ModUp, digits of {alpha}: {msg}"
    a = np.concatenate([d, O.ntt(par, words(spec.p), spec.p)])
    out = empty(L, N)
    P.ckks_moddown(h, dev(a), L, out, ctx.workspace("MODDOWN", L))
    msg = first_mismatch(host(out), O.moddown(par, a, L))
    assert not msg, f"ModDown, {alpha} special primes: {msg}"
