"""GPU parity of the sums' kernels at the edges of how they share out work, on the largest primes below 2^60: the rotated c0 parts of hoisted
sums (four limbs of the outputs to a work group, sums brought down every eight terms, sixteen terms to a launch), and the plaintext sums
of a layer with one ModDown per output (only one tap has a second component, nine products of residues of 60 bits at their top).  And, on the
largest primes below 2^54, hoisted sums of as many products as their sums take."""
import numpy as np
import pytest

from test_gpu_widest_primes import _setup

pytestmark = pytest.mark.gpu


# outputs x limbs = 1, 2, 3, 4, 9 of four to a work group; 1, 3, 7, 15, 31 terms
@pytest.mark.parametrize("C_a,outs,level", [(2, 1, 1), (4, 1, 2), (8, 1, 3), (16, 2, 2), (32, 3, 3)])
@pytest.mark.parametrize("logN", [9, 13])
def test_hoisted_sum_shapes(logN, C_a, outs, level):
    from gpu_util import dev, host, zeros
    prm, orc, ctx, residues = _setup(logN, 60, 4, 1, 4)
    block = prm.N // 2 // C_a
    gs = [orc.galois_elt(block * i) for i in range(1, C_a)]
    keys = [residues(prm.moduli, 8, "mixed").reshape(4, 2, -1, prm.N) for _ in gs]
    for g, k in zip(gs, keys):
        ctx.he_evk_register(g, dev(k))
    q = prm.q[:level + 1]
    ct, pts = residues(q, 2, "uniform"), [residues(q, 1, f)[0] for f in ("top", "uniform", "mixed")[:outs]]
    got = ctx.he_conv2d(C_a, 1, block, 1, 1, level, [dev(p) for p in pts], dev(ct), [zeros(2, level, prm.N) for _ in pts], hoisted_ras=True)
    for p, o in zip(pts, got):
        x = orc.rescale(orc.ptct_mac(None, ct, p, level, init=True), level)
        assert (host(o) == orc.rotate_sum_deferred([x] * C_a, level - 1, [1] + gs, [None] + keys)).all()


@pytest.mark.parametrize("logN", [10, 13])
def test_sums_with_one_second_component(logN):
    from gpu_util import dev, host, zeros
    from oracle import conv2d as CV
    prm, orc, ctx, residues = _setup(logN, 60, 3, 1, 3)
    level, C_a = 2, 4
    side = 1 << (logN - 4) // 2                             # C_a images with at least one replica fill the slots
    geo = CV.ConvGeometry(prm.N, C_a, side, side, C_a * (prm.N // 2 // (C_a * side * side)))
    evks = {st: residues(prm.moduli, 6, "mixed").reshape(3, 2, -1, prm.N) for st in sorted(set(s for s in geo.tap_steps if s) | set(geo.ras_steps))}
    for st, k in evks.items():
        ctx.he_evk_register(ctx.galois_elt(st), dev(k))
    ct = residues(prm.q, 2, "top")
    pts = np.stack([np.stack([residues(prm.moduli, 1, "top")[0] for _ in geo.taps]) for _ in range(geo.n_out)])
    want = CV.caconv(orc, geo, ct, level, pts, evks, deferred_taps=True)
    outs = [zeros(2, level, prm.N) for _ in range(geo.n_out)]
    ctx.he_conv2d(C_a, side, side, geo.R, 3, level, [dev(pts[o, t]) for o in range(geo.n_out) for t in range(len(geo.taps))], dev(ct), outs, deferred_taps=True)
    for o in range(geo.n_out):
        assert (host(outs[o]) == want[o]).all(), o


# 16 terms in the first of two launches: 16 digits make 256 products, as many as the sums take of digits below 2q; from 17 on digits are
# brought below q first
@pytest.mark.parametrize("digits", [16, 17])
def test_hoisted_sum_of_many_digits(digits):
    from gpu_util import dev, host, zeros
    logN, C_a, level = 13, 32, digits
    prm, orc, ctx, residues = _setup(logN, 54, level + 1, 1, level + 1)
    block = prm.N // 2 // C_a
    gs = [orc.galois_elt(block * i) for i in range(1, C_a)]
    key = residues(prm.moduli, 2 * (level + 1), "top").reshape(level + 1, 2, -1, prm.N)
    d_key = dev(key)
    for g in gs:
        ctx.he_evk_register(g, d_key)
    ct, pt = residues(prm.q, 2, "uniform"), residues(prm.q, 1, "mixed")[0]
    got, = ctx.he_conv2d(C_a, 1, block, 1, 1, level, [dev(pt)], dev(ct), [zeros(2, level, prm.N)], hoisted_ras=True)
    x = orc.rescale(orc.ptct_mac(None, ct, pt, level, init=True), level)
    assert (host(got) == orc.rotate_sum_deferred([x] * C_a, level - 1, [1] + gs, [None] + [key] * len(gs))).all()
