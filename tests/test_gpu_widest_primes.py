"""GPU parity where the lazy ranges are fullest: the largest primes below 2^54 (narrow forward, wide inverse), 2^55 (the last whose
ModDown takes unreduced transforms), 2^57 (wide in both directions) and 2^60 (the widest class), residues at their top or at zero.
Transforms, a key switch of every kind, rescale, and the sums of plaintext products that fill their split accumulators - against
the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams, is_prime

pytestmark = pytest.mark.gpu


def primes_below(top, two_n, count):
    c, out = top - two_n + 1, []
    while len(out) < count:
        if is_prime(c):
            out.append(c)
        c -= two_n
    return out


def _setup(logN, bits, nq, np_, dnum):
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    m = primes_below(1 << bits, 2 << logN, nq + np_)
    prm = HEParams(logN=logN, q=m[np_:], p=m[:np_], dnum=dnum, scale=2.0 ** 40, hamming=64, name="widest")
    rng = S.make_rng(1000 + 64 * logN + bits)

    def residues(moduli, n, fill):
        if fill == "uniform":
            return S.uniform_limbs(rng, moduli, prm.N, n)
        top = np.broadcast_to(np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1), (n, len(moduli), prm.N)).copy()
        if fill == "mixed":
            top[rng.integers(0, 2, size=top.shape) == 1] = 0
        return top

    return prm, Oracle.from_params(prm), HEContext.from_params(prm), residues


@pytest.mark.parametrize("logN", [12, 13, 14, 15, 16, 17])
@pytest.mark.parametrize("bits", [54, 55, 57, 60])
def test_transforms_and_key_switches(logN, bits):
    from gpu_util import dev, host, zeros
    prm, orc, ctx, residues = _setup(logN, bits, 4, 2, 2)
    N, level, step = prm.N, 3, 3
    g = orc.galois_elt(step)
    idx = [0, 1, 2, 3] * 2
    for fill in ("top", "mixed"):
        a = residues(prm.q, 2, fill).reshape(8, N)
        d = dev(a)
        ctx.he_ntt(d, idx)
        assert (host(d) == orc.ntt(a, idx)).all(), fill
        d = dev(a)
        ctx.he_intt(d, idx)
        assert (host(d) == orc.intt(a, idx)).all(), fill
        key = residues(prm.moduli, 4, fill).reshape(2, 2, -1, N)
        ctx.he_evk_register(g, dev(key))
        cts = [residues(prm.q, 2, fill) for _ in range(2)]
        d_cts, out = [dev(c) for c in cts], zeros(2, 4, N)
        for c, dc in zip(cts, d_cts):
            ctx.he_rotate(dc, level, step, out)
            assert (host(out) == orc.rotate(c, level, g, key)).all(), fill
        ctx.he_rotate_sum(d_cts + d_cts, level, [step, 0, step, step], out, deferred=True)
        assert (host(out) == orc.rotate_sum_deferred(cts + cts, level, [g, 1, g, g], [key, None, key, key])).all(), fill
        ctx.he_evk_register(0, dev(key))
        ctx.he_mulct(d_cts[0], d_cts[1], level, out)
        assert (host(out) == orc.mulct(cts[0], cts[1], level, key)).all(), fill
        down = zeros(2, 3, N)
        ctx.he_rescale(d_cts[0], level, down)
        assert (host(down) == orc.rescale(cts[0], level)).all(), fill


# a launch takes 16 terms; 8 products of 60 bits fill a split sum, 16 below 60 bits
@pytest.mark.parametrize("n", [1, 6, 7, 8, 9, 10, 14, 15, 16, 17, 33])
@pytest.mark.parametrize("logN,bits", [(8, 60), (9, 59), (13, 60)])
def test_plaintext_sums(logN, bits, n):
    """he_raconv with one tap (the sum over its inputs, rescaled) and he_ptct_mac_rot, all residues at their top."""
    from gpu_util import dev, host, zeros
    from oracle import prcr as PR
    prm, orc, ctx, residues = _setup(logN, bits, 3, 1, 3)
    N, level = prm.N, 2
    for fill in ("top", "mixed"):
        cts, pts = [residues(prm.q, 2, fill) for _ in range(n)], [residues(prm.q, 1, fill)[0] for _ in range(n)]
        d_cts, d_pts = [dev(c) for c in cts], [dev(p) for p in pts]
        want = PR.mac_rotated_plaintexts(orc, cts, pts, [1] * n, level)
        out = ctx.he_raconv(8, 1, 1, level, d_pts, d_cts, zeros(2, level, N))
        assert (host(out) == orc.rescale(want, level)).all(), fill
        gs = [orc.galois_elt(i) if i else 1 for i in range(n)]
        acc = ctx.he_ptct_mac_rot(zeros(2, level + 1, N), d_cts, d_pts, gs, level)
        want = PR.mac_rotated_plaintexts(orc, cts, pts, gs, level)
        assert (host(acc) == want).all(), fill
        ctx.he_ptct_mac_rot(acc, d_cts, d_pts, gs, level, init=False)
        assert (host(acc) == orc.add(want, want, level)).all(), fill


@pytest.mark.parametrize("logN", [9, 13, 16])
@pytest.mark.parametrize("bits", [54, 55, 60])
def test_hoisted_sums(logN, bits):
    """The rotate-and-sum of he_conv2d as one hoisted sum: 15 terms of 3 digits, more than one fold of its split accumulators at
    either width, keys at their top; it is the rotation sum of the rescaled output, repeated."""
    from gpu_util import dev, host, zeros
    prm, orc, ctx, residues = _setup(logN, bits, 4, 1, 4)
    N, level, C_a = prm.N, 3, 16
    block = N // 2 // C_a
    gs = [orc.galois_elt(block * i) for i in range(1, C_a)]
    for fill in ("top", "mixed"):
        keys = [residues(prm.moduli, 8, fill).reshape(4, 2, -1, N) for _ in gs]
        d_keys = [dev(k) for k in keys]
        for g, k in zip(gs, d_keys):
            ctx.he_evk_register(g, k)
        ct, pts = residues(prm.q, 2, "uniform"), [residues(prm.q, 1, f)[0] for f in (fill, "uniform", "mixed")]
        outs = ctx.he_conv2d(C_a, 1, block, 1, 1, level, [dev(p) for p in pts], dev(ct), [zeros(2, level, N) for _ in pts], hoisted_ras=True)
        for p, o in zip(pts, outs):
            x = orc.rescale(orc.ptct_mac(None, ct, p, level, init=True), level)
            assert (host(o) == orc.rotate_sum_deferred([x] * C_a, level - 1, [1] + gs, [None] + keys)).all(), fill
