"""GPU parity of key switches of seven and eight digits whose special primes are at the top of the class near a multiple of 2^32 (just below 2^59 +
2^50): their rows enter the products below 2q, so the split sums hold the largest values that class gives them.  Ciphertext primes of
the same size beside narrow ones; keys and sources at the top of their range and random; one source, batches (a wavefront to a row, more
digits than a sum takes), complete digits and sums of rotations - against the oracle, bit for bit."""
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_modulus_classes import primes_from, tops
from test_gpu_near_moduli import near_primes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,digits,cts", [(13, 7, 1), (13, 8, 1), (14, 7, 9), (14, 8, 9), (16, 8, 2)])
def test_digits_at_the_top(logN, digits, cts):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    two_n = 2 << logN
    top = near_primes("centred top", two_n, 2 + digits // 2)
    assert all((1 << 59) < p <= (1 << 59) + (1 << 50) for p in top)
    q = top[2:] + primes_from(1 << 53, two_n, digits - len(top) + 2)
    prm = HEParams(logN=logN, q=q, p=top[:2], dnum=digits, scale=2.0 ** 20, hamming=64, name="digits")
    rng, orc, ctx, N, level = S.make_rng(8800 + logN + digits), Oracle.from_params(prm), HEContext.from_params(prm), prm.N, digits - 1
    keys = [tops(prm.moduli, 2 * digits, N).reshape(digits, 2, -1, N), S.uniform_limbs(rng, prm.moduli, N, 2 * digits).reshape(digits, 2, -1, N)]
    d_keys, steps = [dev(k) for k in keys], [1, 2]
    gs = [orc.galois_elt(s) for s in steps]
    for g, k in zip(gs, d_keys):
        ctx.he_evk_register(g, k)
    x = [tops(q, 2, N) if i == 0 else S.uniform_limbs(rng, q, N, 2) for i in range(cts)]
    d_x = [dev(c) for c in x]
    for hoisted in (False, True):
        outs = [zeros(2, level + 1, N) for _ in x for _ in steps]
        ctx.he_rotate_batch(d_x, level, steps, outs, hoisted=hoisted)
        for i, o in enumerate(outs):
            assert (host(o) == orc.rotate(x[i // 2], level, gs[i % 2], keys[i % 2])).all(), (hoisted, i)
    out, terms = zeros(2, level + 1, N), [i % 2 for i in range(max(cts, 3))]
    src = [i % cts for i in range(len(terms))]
    ctx.he_rotate_sum([d_x[i] for i in src], level, [steps[t] for t in terms], out, deferred=True)
    assert (host(out) == orc.rotate_sum_deferred([x[i] for i in src], level, [gs[t] for t in terms], [keys[t] for t in terms])).all()
