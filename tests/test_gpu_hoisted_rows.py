"""GPU parity of hoisted sums whose kernel takes the digits through their rows and the special primes' sums through their inverse rows itself:
moduli of every class side by side in one launch, 1 to 8 outputs of a launch's tile and one beyond it (rows that two and four wavefronts
share unevenly), up to 31 terms, one digit (tiles of LDS for the rows alone) and
several, on rings with and without the conversion with its columns - against the oracle, bit for bit."""
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_modulus_classes import LINES, primes_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,C_a,outs,dnum", [(13, 8, 1, 4), (13, 32, 2, 2), (13, 8, 3, 1), (14, 16, 5, 1), (14, 32, 8, 2), (13, 4, 9, 4), (16, 8, 8, 1),
                                                  (17, 4, 2, 2)])
def test_moduli_of_every_class(logN, C_a, outs, dnum):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    two_n = 2 << logN
    # near a multiple of 2^32; narrow; wide on both sides of a line; the widest
    special = [primes_from(s, d * two_n, 1)[0] for s, d in ((1 << 53, 1), (LINES["inverse"] - (1 << 31), -1), (LINES["inverse"], 1), (LINES["widest"], -1), (1 << 60, -1))]
    q = [primes_from(s, d * two_n, 1)[0] for s, d in (((1 << 60) - (1 << 31), -1), ((1 << 54) + (1 << 31), -1), (LINES["forward"], 1), (1 << 54, -1))]
    if outs % 2:                                         # the near and the narrow one among the limbs that are left at the end
        q.reverse()
    prm = HEParams(logN=logN, q=q, p=special, dnum=dnum, scale=2.0 ** 20, hamming=64, name="rows")
    rng, orc, ctx, N, level = S.make_rng(3100 + logN + outs), Oracle.from_params(prm), HEContext.from_params(prm), prm.N, 3
    block = N // 2 // C_a
    gs = [orc.galois_elt(block * i) for i in range(1, C_a)]
    keys = [S.uniform_limbs(rng, prm.moduli, N, 2 * dnum).reshape(dnum, 2, -1, N) for _ in gs[:3]]
    keys = [keys[i % len(keys)] for i in range(len(gs))]
    d_keys = [dev(k) for k in keys[:3]]
    for i, g in enumerate(gs):
        ctx.he_evk_register(g, d_keys[i % len(d_keys)])
    ct, pts = S.uniform_limbs(rng, q, N, 2), [S.uniform_limbs(rng, q, N)[0] for _ in range(outs)]
    ctx.he_counters_reset()
    beta = -(-level // -(-len(q) // dnum))
    got = ctx.he_conv2d(C_a, 1, block, 1, 1, level, [dev(p) for p in pts], dev(ct), [zeros(2, level, N) for _ in pts], hoisted_ras=True)
    assert ctx.he_counters()["intt_limbs"] == outs * (2 + level + 2 * len(special))
    assert ctx.he_counters()["ntt_limbs"] == outs * (2 * level + beta * (level + len(special)) - level + 2 * level)
    for p, o in zip(pts, got):
        x = orc.rescale(orc.ptct_mac(None, ct, p, level, init=True), level)
        assert (host(o) == orc.rotate_sum_deferred([x] * C_a, level - 1, [1] + gs, [None] + keys)).all()
