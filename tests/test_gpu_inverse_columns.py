"""GPU parity of the inverse column passes at N = 2^17 on both sides of the number of work groups from which a form of fewer registers runs: moduli of
every class side by side, plain (he_intt) and with the scaling of a key switch's sources, whole residues at the top of their range among
the inputs - against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_modulus_classes import LINES, primes_from

pytestmark = pytest.mark.gpu

LOGN, N = 17, 1 << 17
Q = [primes_from(s, d * 2 * N, 1)[0] for s, d in ((1 << 53, 1), (LINES["inverse"], -1), (LINES["inverse"], 1), ((1 << 53) - (1 << 40), -1), (LINES["widest"], -1),
                                                  ((1 << 60) - (1 << 31), -1), (LINES["forward"], 1), (1 << 52, 1))]


@pytest.mark.parametrize("limbs", [1, 31, 32, 33])
def test_plain(limbs):
    from gpu_util import dev, host
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    orc, ctx, rng = Oracle(LOGN, Q, [], 1), HEContext(LOGN, Q, [], 1), S.make_rng(17 + limbs)
    idx = [(3 * i) % len(Q) for i in range(limbs)]
    a = np.stack([S.uniform_limbs(rng, [Q[i]], N)[0][0] for i in idx])
    a[::3] = np.array([Q[i] - 1 for i in idx[::3]], dtype=np.uint64)[:, None]
    d = dev(a)
    ctx.he_intt(d, idx)
    assert (host(d) == orc.intt(a, idx)).all()


@pytest.mark.parametrize("cts", [3, 4])
def test_sources_of_key_switches(cts):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    prm = HEParams(logN=LOGN, q=Q, p=primes_from(1 << 59, 2 * N, 1), dnum=8, scale=2.0 ** 20, hamming=64, name="columns")
    orc, ctx, rng, level = Oracle.from_params(prm), HEContext.from_params(prm), S.make_rng(27 + cts), len(Q) - 1
    key = S.uniform_limbs(rng, prm.moduli, N, 16).reshape(8, 2, -1, N)
    d_key = dev(key)
    ctx.he_evk_register(orc.galois_elt(5), d_key)
    x = [S.uniform_limbs(rng, Q, N, 2) for _ in range(cts)]
    outs = [zeros(2, level + 1, N) for _ in x]
    ctx.he_rotate_batch([dev(c) for c in x], level, [5], outs, hoisted=False)
    for c, o in zip(x, outs):
        assert (host(o) == orc.rotate(c, level, orc.galois_elt(5), key)).all()
