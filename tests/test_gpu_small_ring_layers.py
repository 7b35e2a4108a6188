"""GPU parity of rotate-and-sum layers on small rings, where the rescale raises what the first step rotates and a step what the next one does: 1 to 4 limbs per digit and special primes, 1 to 8 digits, primes at the widest that FP64 carries, every register-block split of the transforms, no step, one
and several, one output and as many as a launch takes and more, uniform and extreme residues - against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_small_ring import primes_below

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,bits,nq,np_,dnum,levels,C_a,outs", [
    (8, 45, 9, 1, 9, (8, 1), 8, 2),     # eight digits of one limb; one
    (9, 45, 8, 4, 2, (7, 5, 1), 16, 1),  # four sources and four special primes; partial digits
    (10, 45, 6, 3, 2, (5, 3), 4, 16),
    (11, 45, 5, 2, 3, (4, 3), 4, 17),   # more outputs than a launch takes
    (12, 45, 5, 2, 3, (4, 1), 2, 3),
    (12, 40, 4, 1, 4, (3, 2), 8, 4),
    (11, 45, 9, 1, 3, (8, 4), 8, 2),    # three limbs a digit and one special prime, the most that a step raises; a partial digit
    (10, 45, 4, 3, 4, (3,), 16, 1),     # one and three
    (9, 45, 6, 2, 3, (5, 4), 4, 3),     # two and two
    (12, 40, 3, 1, 3, (2,), 1, 2),      # no step
    (12, 46, 4, 1, 4, (3,), 4, 2),      # one bit more: the integer kernels, a launch each
])
@pytest.mark.parametrize("fill", ["uniform", "extreme"])
def test_rotate_and_sum(logN, bits, nq, np_, dnum, levels, C_a, outs, fill):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    m = primes_below(1 << bits, 2 << logN, nq + np_)
    prm = HEParams(logN=logN, q=m[np_:], p=m[:np_], dnum=dnum, scale=2.0 ** 20, hamming=64, name="small")
    rng, orc, ctx, N = S.make_rng(950 + logN + bits), Oracle.from_params(prm), HEContext.from_params(prm), prm.N

    def residues(moduli, n):
        if fill == "uniform":
            return S.uniform_limbs(rng, moduli, N, n)
        top = np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1)
        return np.where(rng.integers(0, 2, size=(n, len(moduli), N)) == 1, top, np.uint64(0))

    block = N // 2 // C_a
    steps = [block << t for t in range(C_a.bit_length() - 1)]
    keys = {s: residues(prm.moduli, 2 * dnum).reshape(dnum, 2, -1, N) for s in steps}
    for s, k in keys.items():
        ctx.he_evk_register(ctx.galois_elt(s), dev(k))
    for level in levels:
        q = prm.q[:level + 1]
        ct, pts = residues(q, 2), [residues(q, 1)[0] for _ in range(outs)]
        ctx.he_counters_reset()
        got = ctx.he_conv2d(C_a, 1, block, 1, 1, level, [dev(p) for p in pts], dev(ct), [zeros(2, level, N) for _ in pts])
        cnt = ctx.he_counters()
        assert cnt["modup"] == cnt["moddown"] == cnt["keyswitch"] == outs * len(steps) and cnt["rescale"] == outs
        beta, R = -(-level // -(-nq // dnum)), level + np_
        assert cnt["intt_limbs"] == outs * (2 + len(steps) * (level + 2 * np_))
        assert cnt["ntt_limbs"] == outs * (2 * level + len(steps) * (beta * R - level + 2 * level))
        for p, o in zip(pts, got):
            x = orc.rescale(orc.ptct_mac(None, ct, p, level, init=True), level)
            for s in steps:
                x = orc.add(x, orc.rotate(x, level - 1, orc.galois_elt(s), keys[s]), level - 1)
            assert (host(o) == x).all(), level
