"""GPU parity of replication-aligned convolutions whose plaintext sums go through the inverse rows of the key switches behind them in the same
launch: moduli of every class side by side, 1 to 17 inputs (one launch of every kind of kernel, and two of which only the last goes on), more
taps than are raised at once, a ring whose conversions are launches of their own, each with one ModDown and with one per rotation - against the oracle, bit for bit."""
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams
from test_gpu_modulus_classes import LINES, primes_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,C_a,H,W,n_in,f,level", [(13, 16, 16, 16, 1, 3, 3), (13, 16, 16, 16, 9, 3, 2), (13, 4, 32, 32, 17, 3, 3), (14, 16, 16, 16, 16, 3, 1),
                                                       (13, 8, 1, 128, 3, 3, 3), (13, 16, 16, 16, 2, 5, 3), (17, 16, 64, 64, 2, 3, 3)])
@pytest.mark.parametrize("deferred", [False, True])
def test_sums_of_every_class(logN, C_a, H, W, n_in, f, level, deferred):
    from gpu_util import dev, host, zeros
    from oracle import conv2d as CV
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    two_n = 2 << logN
    q = [primes_from(s, d * two_n, 1)[0] for s, d in ((1 << 53, 1), ((1 << 54) + (1 << 31), -1), (LINES["widest"], -1), ((1 << 60) - (1 << 31), -1))]
    prm = HEParams(logN=logN, q=q, p=primes_from(1 << 60, -two_n, 2), dnum=2, scale=2.0 ** 20, hamming=64, name="rows")
    rng, orc, ctx, N = S.make_rng(3300 + logN + n_in), Oracle.from_params(prm), HEContext.from_params(prm), prm.N
    R = N // 2 // (C_a * H * W)
    geo = CV.RAGeometry(N, C_a, H, W, n_in * R, f=f)
    assert geo.n_in == n_in and geo.R == R
    steps = sorted(set(s for s in geo.tap_steps if s))
    key = S.uniform_limbs(rng, prm.moduli, N, 4).reshape(2, 2, -1, N)
    evks = {st: (key if i % 2 else key[::-1].copy()) for i, st in enumerate(steps)}
    for st, k in evks.items():
        ctx.he_evk_register(ctx.galois_elt(st), dev(k))
    cts = [S.uniform_limbs(rng, q[:level + 1], N, 2) for _ in range(n_in)]
    pts = S.uniform_limbs(rng, q[:level + 1], N, n_in * f * f).reshape(n_in, f * f, level + 1, N)
    want = CV.raconv(orc, geo, cts, level, pts, evks, deferred=deferred)
    out = zeros(2, level, N)
    ctx.he_raconv(W, geo.R, f, level, [dev(pts[i, t]) for i in range(n_in) for t in range(f * f)], [dev(c) for c in cts], out, deferred=deferred)
    assert (host(out) == want).all()
