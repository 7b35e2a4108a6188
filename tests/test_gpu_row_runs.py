"""GPU parity: transforms on both sides of the row passes' rules - rows of 64 threads for small launches, runs of one modulus
for large ones - at the edges of a run, for narrow and wide moduli and extreme values, against the oracle."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import ntt_primes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,counts", [
    (13, (2, 1, 3)),            # few limbs: rows of 64 threads, the smallest ring
    (14, (90, 91, 76)),         # one limb more than those take: runs of 4 with 2, 3 and none left over
    (16, (21, 21, 22)),         # the last launch of 64 threads to a row ...
    (16, (17, 16, 32)),         # ... and the first of runs, one limb more than a run holds
    (16, (1, 34, 32)),          # a lone limb among full runs
    (17, (12, 12, 9)),          # one limb in the last run of its modulus
    (16, (133, 134, 135)),      # runs of 8, two rounds of four: 5, 6 and 7 left over
    (16, (129, 130, 131)),      # ... and 1, 2 and 3
    (17, (130, 135, 141)),      # runs of 16: 2, 7 and 13 left over
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
