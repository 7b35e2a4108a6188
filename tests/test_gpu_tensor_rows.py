"""GPU parity of products whose last part goes through the inverse rows of its key switch in the launch that forms it: moduli of every class
side by side, the smallest and largest rings that take this form, one that does not, partial digits, residues at their top, products in
place, and the squares of a fused block in groups - against the oracle, bit for bit."""
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_modulus_classes import LINES, primes_from, tops

pytestmark = pytest.mark.gpu


def every_class(logN):
    two_n = 2 << logN
    q = [primes_from(s, d * two_n, 1)[0] for s, d in ((1 << 53, 1), ((1 << 54) + (1 << 31), -1), (LINES["widest"], -1), ((1 << 60) - (1 << 31), -1), (1 << 54, -1))]
    return HEParams(logN=logN, q=q, p=primes_from(1 << 60, -two_n, 2), dnum=3, scale=2.0 ** 20, hamming=64, name="products")


@pytest.mark.parametrize("logN,level", [(13, 4), (13, 0), (14, 3), (15, 1), (16, 4), (17, 4)])
def test_products_of_every_class(logN, level):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    prm = every_class(logN)
    rng, orc, ctx, N = S.make_rng(4100 + logN), Oracle.from_params(prm), HEContext.from_params(prm), prm.N
    rlk = S.uniform_limbs(rng, prm.moduli, N, 6).reshape(3, 2, -1, N)
    ctx.he_evk_register(0, dev(rlk))
    a, b, t = S.uniform_limbs(rng, prm.q[:level + 1], N, 2), S.uniform_limbs(rng, prm.q[:level + 1], N, 2), tops(prm.q[:level + 1], 2, N)
    out = zeros(2, level + 1, N)
    for x, y in ((a, b), (t, t), (a, t)):
        ctx.he_mulct(dev(x), dev(y), level, out)
        assert (host(out) == orc.mulct(x, y, level, rlk)).all()
    d = dev(b)
    ctx.he_mulct(d, d, level, d)
    assert (host(d) == orc.mulct(b, b, level, rlk)).all()


@pytest.mark.parametrize("hoisted", [False, True])
def test_squares_of_a_block(hoisted):
    from gpu_util import dev, host, zeros
    from oracle import block as OB
    from oracle import conv2d as CV
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    prm, level, C_a, H, W, n_ra, k_in = every_class(13), 4, 4, 32, 32, 5, (1 << 53) + 12345
    rng, orc, ctx, N = S.make_rng(4200), Oracle.from_params(prm), HEContext.from_params(prm), prm.N
    g_ca, g_ra = CV.ConvGeometry(N, C_a, H, W, n_ra, f=3), CV.RAGeometry(N, C_a, H, W, n_ra, f=3)
    steps = set(s for s in g_ca.tap_steps if s) | set(s for s in g_ra.tap_steps if s) | set(g_ca.ras_steps) | {H * W * g_ca.R * i for i in range(1, C_a)}
    evks = {st: S.uniform_limbs(rng, prm.moduli, N, 6).reshape(3, 2, -1, N) for st in sorted(steps)}
    rlk = S.uniform_limbs(rng, prm.moduli, N, 6).reshape(3, 2, -1, N)
    for st, k in evks.items():
        ctx.he_evk_register(ctx.galois_elt(st), dev(k))
    ctx.he_evk_register(0, dev(rlk))
    p_ca = [[S.uniform_limbs(rng, prm.q[:level + 1], N, 9)] for _ in range(n_ra)]
    p_ra = [[S.uniform_limbs(rng, prm.q[:level - 1], N, 9) for _ in range(n_ra)]]
    ct = S.uniform_limbs(rng, prm.q[:level + 1], N, 2)
    want = OB.ca_ra_block(orc, g_ca, g_ra, [ct], level, p_ca, p_ra, evks, rlk, k_in, hoisted_ras=hoisted)
    w_ca, w_ra = [dev(p_ca[j][0][t]) for j in range(n_ra) for t in range(9)], [dev(p_ra[0][j][t]) for j in range(n_ra) for t in range(9)]
    for group in (1, 3, 0):
        out = zeros(2, level - 2, N)
        ctx.he_ca_ra_block(C_a, H, W, g_ca.R, 3, level, k_in, w_ca, w_ra, [dev(ct)], [out], group=group, hoisted_ras=hoisted)
        assert (host(out) == want[0]).all(), group
