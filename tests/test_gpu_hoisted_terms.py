"""GPU parity of hoisted sums of 31 terms by how many products a sum takes: all in one launch up to 512 (with digits below 2q up to 256), more in
launches that continue, on rings with and without rows of their own, moduli of 54 and 60 bits side by side, keys at the top of their
range - against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_modulus_classes import primes_from, tops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,digits,outs", [(13, 8, 3), (13, 9, 2), (13, 16, 1), (13, 17, 1), (14, 24, 1), (12, 3, 5), (12, 16, 2), (11, 17, 1), (10, 24, 1)])
def test_terms_and_digits(logN, digits, outs):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    C_a, two_n, nq = 32, 2 << logN, digits + 1
    q = [m for pair in zip(primes_from(1 << 54, -two_n, (nq + 1) // 2), primes_from(1 << 60, -two_n, (nq + 1) // 2)) for m in pair][:nq]
    prm = HEParams(logN=logN, q=q, p=primes_from(1 << 59, two_n, 1), dnum=nq, scale=2.0 ** 20, hamming=64, name="terms")
    rng, orc, ctx, N, level = S.make_rng(7200 + logN + digits), Oracle.from_params(prm), HEContext.from_params(prm), prm.N, nq - 1
    block = N // 2 // C_a
    gs = [orc.galois_elt(block * i) for i in range(1, C_a)]
    keys = [S.uniform_limbs(rng, prm.moduli, N, 2 * nq).reshape(nq, 2, -1, N), tops(prm.moduli, 2 * nq, N).reshape(nq, 2, -1, N)]
    d_keys = [dev(k) for k in keys]
    for i, g in enumerate(gs):
        ctx.he_evk_register(g, d_keys[i % 3 == 0])
    ct, pts = S.uniform_limbs(rng, q, N, 2), [S.uniform_limbs(rng, q, N)[0] for _ in range(outs)]
    got = ctx.he_conv2d(C_a, 1, block, 1, 1, level, [dev(p) for p in pts], dev(ct), [zeros(2, level, N) for _ in pts], hoisted_ras=True)
    for p, o in zip(pts, got):
        x = orc.rescale(orc.ptct_mac(None, ct, p, level, init=True), level)
        want = orc.rotate_sum_deferred([x] * C_a, level - 1, [1] + gs, [None] + [keys[i % 3 == 0] for i in range(len(gs))])
        assert (np.asarray(host(o)) == want).all()
