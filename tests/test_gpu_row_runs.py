"""GPU parity: transforms of launches whose row passes go by runs of one modulus (at least three limbs of every four lane
quarters in use), at the edges of a run: 3 to 17 limbs of a modulus, narrow and wide moduli, extreme values - against the oracle."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import ntt_primes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,counts", [
    (13, (4, 3, 3)),            # exactly three of four lanes
    (13, (17, 16, 3)),          # one limb more than a run holds
    (14, (8, 7, 5)),
    (16, (1, 4, 16)),           # a lone limb among full runs
    (17, (4, 4, 4)),
])
def test_row_runs(logN, counts):
    from gpu_util import dev, host
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    two_n, N = 2 << logN, 1 << logN
    q, p = ntt_primes(54, two_n, 1) + ntt_primes(58, two_n, 1), ntt_primes(60, two_n, 1)
    orc, ctx, rng = Oracle(logN, q, p, 2), HEContext(logN, q, p, 2), S.make_rng(logN + sum(counts))
    idx = [m for m, n in enumerate(counts) for _ in range(n)]
    rng.shuffle(idx)
    a = np.stack([S.uniform_limbs(rng, [(q + p)[i]], N)[0][0] for i in idx])
    a[0, :] = (q + p)[idx[0]] - 1
    d = dev(a)
    ctx.he_ntt(d, idx)
    assert (host(d) == orc.ntt(a, idx)).all()
    d = dev(a)
    ctx.he_intt(d, idx)
    assert (host(d) == orc.intt(a, idx)).all()
