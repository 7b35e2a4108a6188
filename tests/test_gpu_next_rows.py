"""GPU parity of rotate-and-sum stages whose steps leave the inverse rows of what the next step raises: moduli of every class side by side, work
groups and wavefronts to a row, eight digits, more outputs than are raised at once (which keep the launch of their own), a ring without this
form, taps with a ModDown each and with one - against the oracle, bit for bit."""
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_modulus_classes import LINES, primes_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,C_a,H,W,n_out,f,level,dnum,deferred", [
    (13, 16, 16, 16, 1, 3, 3, 2, False), (13, 4, 32, 32, 5, 1, 4, 3, False), (14, 16, 16, 16, 12, 3, 4, 3, False), (14, 8, 32, 16, 9, 3, 2, 2, True),
    (13, 4, 16, 16, 9, 1, 7, 8, False), (14, 4, 32, 64, 17, 1, 7, 8, False), (13, 8, 16, 16, 17, 1, 4, 3, False), (16, 4, 64, 64, 2, 1, 4, 3, False), (17, 4, 64, 64, 2, 1, 3, 2, False)])
def test_steps_of_every_class(logN, C_a, H, W, n_out, f, level, dnum, deferred):
    from gpu_util import dev, host, zeros
    from oracle import conv2d as CV
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    two_n = 2 << logN
    lines = ((1 << 53, 1), ((1 << 54) + (1 << 31), -1), (LINES["widest"], -1), ((1 << 60) - (1 << 31), -1), (1 << 54, -1), (1 << 52, 1), (1 << 51, 1), (1 << 50, 1))
    q = [primes_from(s, d * two_n, 1)[0] for s, d in lines[:level + 1]]
    prm = HEParams(logN=logN, q=q, p=primes_from(1 << 60, -two_n, 2), dnum=dnum, scale=2.0 ** 20, hamming=64, name="next")
    rng, orc, ctx, N = S.make_rng(5100 + logN + n_out), Oracle.from_params(prm), HEContext.from_params(prm), prm.N
    R = N // 2 // (C_a * H * W)
    geo = CV.ConvGeometry(N, C_a, H, W, n_out * R, f=f)
    assert geo.n_out == n_out and geo.R == R
    evks = {st: S.uniform_limbs(rng, prm.moduli, N, 2 * dnum).reshape(dnum, 2, -1, N) for st in sorted(set(s for s in geo.tap_steps if s) | set(geo.ras_steps))}
    for st, k in evks.items():
        ctx.he_evk_register(ctx.galois_elt(st), dev(k))
    ct = S.uniform_limbs(rng, q, N, 2)
    pts = S.uniform_limbs(rng, prm.moduli if deferred else q, N, n_out * f * f).reshape(n_out, f * f, -1, N)
    want = CV.caconv(orc, geo, ct, level, pts, evks, deferred_taps=deferred)
    outs = [zeros(2, level, N) for _ in range(n_out)]
    ctx.he_conv2d(C_a, H, W, geo.R, f, level, [dev(pts[o, t]) for o in range(n_out) for t in range(f * f)], dev(ct), outs, deferred_taps=deferred)
    for o in range(n_out):
        assert (host(outs[o]) == want[o]).all(), o
