"""GPU parity: Rescale whose two column passes are one launch, on every ring that has them, with primes at the top of every width the
kernels tell apart, moduli that do not divide evenly among a tile's work groups, and rounding at both ends of the dropped modulus -
against the oracle, bit for bit."""
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


@pytest.mark.parametrize("logN,widths,levels", [
    (13, [30, 54, 57, 58, 60], (1, 4)),
    (14, [60, 31, 55, 60], (1, 2, 3)),
    (15, [57, 60, 54, 60, 57, 55, 58, 60], (3, 7)),
    (16, [58, 54, 60, 57, 60, 54, 60, 58, 57, 54, 60, 59, 60], (5, 12)),     # moduli by threes
    (17, [60, 57, 54, 60, 57, 60, 54, 60], (1, 4, 7)),
])
def test_rescale(logN, widths, levels):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    pool = {w: primes_below(1 << w, 2 << logN, widths.count(w) + 1) for w in set(widths)}
    q = [pool[w].pop() for w in widths]
    prm = HEParams(logN=logN, q=q, p=[pool[60].pop()], dnum=len(q), scale=2.0 ** 20, hamming=64, name="rescale")
    rng, orc, ctx = S.make_rng(900 + logN), Oracle.from_params(prm), HEContext.from_params(prm)
    N = prm.N
    for level in levels:
        ct = S.uniform_limbs(rng, prm.q[:level + 1], N, 2)
        ql, top = prm.q[level], np.array(prm.q[:level + 1], dtype=np.uint64)[:, None] - np.uint64(1)
        ct[0, :, ::3] = top                              # the largest residues
        ct[1, :, 1::5] = 0
        # coefficients of the dropped limb on both sides of the rounding boundary
        edge = np.array([(ql >> 1) + d for d in (-1, 0, 1, 2)] + [0, 1, ql - 1, ql - 2], dtype=np.uint64)
        ct[1, level] = orc.ntt(np.tile(edge, N // 8), [level]).reshape(N)
        out = zeros(2, level, N)
        ctx.he_rescale(dev(ct), level, out)
        assert (host(out) == orc.rescale(ct, level)).all(), level
