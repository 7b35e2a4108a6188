"""GPU parity on both sides of every line between the classes of moduli (he_internal.h): the products' operands are fullest just below a
line, and just above it other code runs.  Transforms, key switches of every kind and rescale against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams, is_prime

pytestmark = pytest.mark.gpu

LINES = {"inverse": (1 << 63) // 640, "forward": (1 << 63) // 96, "widest": (1 << 63) // 13}


def primes_from(start, step, count):
    """primes = 1 mod |step| going down (step < 0) or up from start"""
    n = abs(step)
    c, out = start - (start - 1) % n + (n if step > 0 else 0), []
    while len(out) < count:
        if is_prime(c):
            out.append(c)
        c += step
    return out


@pytest.mark.parametrize("logN", [13, 14, 15, 16, 17])
@pytest.mark.parametrize("line", sorted(LINES))
@pytest.mark.parametrize("side", ["below", "above"])
def test_both_sides_of_a_line(logN, line, side):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    m = primes_from(LINES[line], (2 << logN) * (1 if side == "above" else -1), 6)
    assert all((x > LINES[line]) == (side == "above") for x in m)
    prm = HEParams(logN=logN, q=m[2:], p=m[:2], dnum=2, scale=2.0 ** 40, hamming=64, name="line")
    orc, ctx, N, level, step = Oracle.from_params(prm), HEContext.from_params(prm), prm.N, 3, 3
    rng, g, idx = S.make_rng(77 + logN), orc.galois_elt(step), [0, 1, 2, 3] * 2

    def top(moduli, n):
        return np.broadcast_to(np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1), (n, len(moduli), N)).copy()

    for fill in (top, lambda moduli, n: S.uniform_limbs(rng, moduli, N, n)):
        a = fill(prm.q, 2).reshape(8, N)
        d = dev(a)
        ctx.he_ntt(d, idx)
        assert (host(d) == orc.ntt(a, idx)).all()
        d = dev(a)
        ctx.he_intt(d, idx)
        assert (host(d) == orc.intt(a, idx)).all()
        key, ct = fill(prm.moduli, 4).reshape(2, 2, -1, N), fill(prm.q, 2)
        ctx.he_evk_register(g, dev(key))
        d_ct, out, down = dev(ct), zeros(2, 4, N), zeros(2, 3, N)
        ctx.he_rotate(d_ct, level, step, out)
        assert (host(out) == orc.rotate(ct, level, g, key)).all()
        ctx.he_rotate_sum([d_ct, d_ct, d_ct], level, [step, 0, step], out, deferred=True)
        assert (host(out) == orc.rotate_sum_deferred([ct, ct, ct], level, [g, 1, g], [key, None, key])).all()
        ctx.he_rescale(d_ct, level, down)
        assert (host(down) == orc.rescale(ct, level)).all()
