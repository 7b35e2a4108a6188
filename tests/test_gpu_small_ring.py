"""GPU parity: key switches and rescales of rings up to 2^12 whose primes reach the widest that FP64 carries exactly (the
largest below 2^45), every register-block split of the transforms, 1 to 4 limbs per digit and special primes, 1 to 8 digits, uniform
and extreme residues - against the oracle, bit for bit."""
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


@pytest.mark.parametrize("logN,bits,nq,np_,dnum,levels", [
    (8, 45, 8, 1, 8, (7, 3)),       # eight digits of one limb; four
    (9, 45, 7, 4, 2, (6, 4, 1)),    # four sources and four special primes; partial digits
    (10, 45, 6, 3, 2, (5, 2)),
    (11, 45, 4, 2, 2, (3, 1)),
    (12, 45, 5, 2, 3, (4, 1)),
    (12, 46, 3, 1, 3, (2, 1)),      # one bit more: the integer kernels
    (12, 30, 3, 1, 3, (2, 1)),      # special prime wider than the others by half
])
@pytest.mark.parametrize("fill", ["uniform", "extreme"])
def test_small_ring_edges(logN, bits, nq, np_, dnum, levels, fill):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    q = primes_below(1 << bits, 2 << logN, nq + np_)
    p = q[:np_] if bits != 30 else primes_below(1 << 45, 2 << logN, np_)
    prm = HEParams(logN=logN, q=q[np_:], p=p, dnum=dnum, scale=2.0 ** 20, hamming=64, name="small")
    rng, orc, ctx = S.make_rng(900 + logN + bits), Oracle.from_params(prm), HEContext.from_params(prm)
    N, step, n_ct = prm.N, 3, 3

    def residues(moduli, n):
        if fill == "uniform":
            return S.uniform_limbs(rng, moduli, N, n)
        top = np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1)
        return np.where(rng.integers(0, 2, size=(n, len(moduli), N)) == 1, top, np.uint64(0))

    key = residues(prm.moduli, 2 * dnum).reshape(dnum, 2, len(prm.moduli), N)
    ctx.he_evk_register(ctx.galois_elt(step), dev(key))
    for level in levels:
        cts = [residues(prm.q[:level + 1], 2) for _ in range(n_ct)]
        outs = [zeros(2, level + 1, N) for _ in range(n_ct)]
        ctx.he_rotate_batch([dev(c) for c in cts], level, [step], outs, hoisted=False)
        for c, o in zip(cts, outs):
            assert (host(o) == orc.rotate(c, level, orc.galois_elt(step), key)).all(), level
        down = zeros(2, level, N)
        ctx.he_rescale(dev(cts[0]), level, down)
        assert (host(down) == orc.rescale(cts[0], level)).all(), level
