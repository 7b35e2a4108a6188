"""GPU parity for he_conv2d with deferred_taps (Slide_f and MulFilter&Sum_f of Algorithm 1 sharing one ModDown per
output): every output ciphertext equals the oracle's bit for bit, decrypts to the float64 convolution, differs in
bits from the tap-by-tap order while agreeing with it far below the tolerance, and the operation counts show
n_out ModDowns in place of f^2-1."""
import sys

import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import config_params, toy_params

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, file=sys.__stdout__, flush=True)


def _run(prm, C_a, H, W, c_out, level, w_std, tol, f=3, seed=None):
    from gpu_util import dev, host, zeros
    from oracle import ckks_client as K
    from oracle import conv2d as CV
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    rng = S.make_rng(prm.seed if seed is None else seed)
    orc, ctx = Oracle.from_params(prm), HEContext.from_params(prm)
    cl = K.Client(orc, S.ternary_secret(rng, prm.N, prm.hamming))
    geo = CV.ConvGeometry(prm.N, C_a, H, W, c_out, f=f)
    x, wt = S.conv_tensors(rng, C_a, c_out, H, W, f, w_std)
    steps = sorted(set(s for s in geo.tap_steps if s) | set(geo.ras_steps))
    evks = {st: cl.rotation_key(orc.galois_elt(st), S.uniform_limbs(rng, prm.moduli, prm.N, prm.dnum),
                                S.gaussian_error(rng, prm.N, prm.sigma, prm.dnum)) for st in steps}
    ct = cl.encrypt(geo.pack_input(x).astype(np.complex128), prm.scale, level,
                    S.uniform_limbs(rng, prm.q[:level + 1], prm.N)[0], S.gaussian_error(rng, prm.N, prm.sigma)[0])
    pts = CV.encode_weights_raised(orc, geo, wt, level, float(prm.q[level]))
    _say("deferred-tap conv parity: inputs ready (N=%d, f=%d, %d keys), running the oracle" % (prm.N, f, len(evks)))
    want = CV.caconv(orc, geo, ct, level, pts, evks, progress=_say, deferred_taps=True)

    for st, k in evks.items():
        ctx.he_evk_register(ctx.galois_elt(st), dev(k))
    weights = [dev(pts[o, t]) for o in range(geo.n_out) for t in range(len(geo.taps))]
    outs = [zeros(2, level, prm.N) for _ in range(geo.n_out)]
    d_ct = dev(ct)
    ctx.he_ws_reserve(ctx.he_ws_query_conv2d(geo.C_a, geo.H, geo.W, geo.R, f, level, geo.n_out, deferred_taps=True))
    ws = ctx.he_ws_bytes()
    ctx.he_counters_reset()
    _say("deferred-tap conv parity: GPU call")
    ctx.he_conv2d(geo.C_a, geo.H, geo.W, geo.R, f, level, weights, d_ct, outs, deferred_taps=True)
    cnt = ctx.he_counters()
    assert ctx.he_ws_bytes() == ws                                  # the reserved workspace was enough
    got = [host(o) for o in outs]
    for o in range(geo.n_out):
        assert (got[o] == want[o]).all(), o
    n_ras, n_rot = len(geo.ras_steps), len([s for s in geo.tap_steps if s])
    assert cnt["keyswitch"] == n_rot + geo.n_out * n_ras
    assert cnt["modup"] == 1 + geo.n_out * n_ras
    assert cnt["moddown"] == geo.n_out + geo.n_out * n_ras          # one per output instead of one per rotated tap
    assert cnt["mac"] == f * f * geo.n_out and cnt["rescale"] == geo.n_out
    dec, spread = geo.unpack_output([cl.decrypt(g, level - 1, prm.scale) for g in got])
    assert np.max(np.abs(dec - CV.conv2d_float(x, wt))) < tol
    assert spread < tol
    # against the tap-by-tap order on the GPU: other bits, the same values
    w_q = [dev(np.ascontiguousarray(pts[o, t, :level + 1])) for o in range(geo.n_out) for t in range(len(geo.taps))]
    ref = [zeros(2, level, prm.N) for _ in range(geo.n_out)]
    ctx.he_conv2d(geo.C_a, geo.H, geo.W, geo.R, f, level, w_q, d_ct, ref)
    ref = [host(r) for r in ref]
    assert any((a != b).any() for a, b in zip(got, ref))
    gap = max(np.max(np.abs(np.asarray(cl.decrypt(a, level - 1, prm.scale)) - np.asarray(cl.decrypt(b, level - 1, prm.scale))))
              for a, b in zip(got, ref))
    assert gap < tol, gap


def test_small_ring_two_outputs():
    prm = toy_params(logN=10, q_bits=40, nq=3, p_bits=41, np_=1, dnum=3, scale=2.0 ** 30, hamming=32, seed=80)
    _run(prm, C_a=4, H=4, W=4, c_out=16, level=2, w_std=0.1, tol=1e-3)


def test_config0():
    _run(config_params(0), C_a=4, H=8, W=8, c_out=4, level=2, w_std=0.1, tol=1e-3)


def test_five_by_five_filter_two_special_primes():
    # 25 taps (the any-number-of-taps kernels), two special primes, a partial last digit, 12 outputs (two chunks of ModDowns)
    prm = toy_params(logN=10, q_bits=40, nq=5, p_bits=45, np_=2, dnum=3, scale=2.0 ** 30, hamming=32, seed=81)
    _run(prm, C_a=2, H=4, W=4, c_out=192, level=4, w_std=0.05, tol=1e-3, f=5)


def test_two_pass_ring():
    prm = toy_params(logN=13, q_bits=40, nq=4, p_bits=50, np_=2, dnum=2, scale=2.0 ** 30, hamming=32, seed=82)
    _run(prm, C_a=4, H=8, W=8, c_out=16, level=3, w_std=0.1, tol=1e-3)


@pytest.mark.timeout(900)
def test_config3_resnet20_layer():
    _run(config_params(3), C_a=16, H=32, W=32, c_out=16, level=23, w_std=(2.0 / (9 * 16)) ** 0.5, tol=1e-3)


def test_more_outputs_than_one_set_of_moddowns():
    """12 outputs of 25 limbs: both components are more limbs than one launch lists.  Uniform residues; every output is the one
    that a call for it alone gives."""
    from gpu_util import dev, host, zeros
    from paper_2302_02407_amd.binding import HEContext
    prm = toy_params(logN=9, q_bits=40, nq=25, p_bits=41, np_=1, dnum=25, hamming=16, seed=83)
    rng, ctx, N, level, n_out = S.make_rng(83), HEContext.from_params(prm), prm.N, 24, 12
    C_a, H, W, R, f = 2, 8, 16, 1, 3
    steps = {((dy * W + dx) * R) % (N // 2) for dy in (-1, 0, 1) for dx in (-1, 0, 1)} - {0} | {H * W * R}
    for s in sorted(steps):
        ctx.he_evk_register(ctx.galois_elt(s), dev(S.uniform_limbs(rng, prm.moduli, N, 2 * prm.dnum).reshape(prm.dnum, 2, -1, N)))
    w = [dev(x) for x in S.uniform_limbs(rng, prm.moduli, N, n_out * f * f)]
    ct = dev(S.uniform_limbs(rng, prm.q, N, 2))
    outs = ctx.he_conv2d(C_a, H, W, R, f, level, w, ct, [zeros(2, level, N) for _ in range(n_out)], deferred_taps=True)
    for o in range(n_out):
        one, = ctx.he_conv2d(C_a, H, W, R, f, level, w[o * f * f:(o + 1) * f * f], ct, [zeros(2, level, N)], deferred_taps=True)
        assert (host(outs[o]) == host(one)).all(), o
