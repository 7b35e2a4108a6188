"""GPU parity on both sides of every line between the classes of moduli (he_internal.h): the products' operands are fullest just below a
line, and just above it other code runs.  Transforms in every form of the passes, key switches singly, in batches, of shared sources and
as sums, a ciphertext product, hoisted sums and rescale against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams, is_prime

pytestmark = pytest.mark.gpu

LINES = {"inverse": (1 << 63) // 640, "forward": (1 << 63) // 96, "widest": (1 << 63) // 13}


SIDES = [(line, side) for line in sorted(LINES) for side in ("below", "above")]


def primes_at(line, side, logN, count):
    m = primes_from(LINES[line], (2 << logN) * (1 if side == "above" else -1), count)
    assert all((x > LINES[line]) == (side == "above") for x in m)
    return m


def tops(moduli, n, N):
    return np.broadcast_to(np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1), (n, len(moduli), N)).copy()


def primes_from(start, step, count):
    """primes = 1 mod |step| going down (step < 0) or up from start"""
    n = abs(step)
    c, out = start - (start - 1) % n + (n if step > 0 else 0), []
    while len(out) < count:
        if is_prime(c):
            out.append(c)
        c += step
    return out


@pytest.mark.parametrize("logN", [13, 14, 15, 16, 17])
@pytest.mark.parametrize("line", sorted(LINES))
@pytest.mark.parametrize("side", ["below", "above"])
def test_both_sides_of_a_line(logN, line, side):
    check_single_calls(logN, primes_at(line, side, logN, 6))


def check_single_calls(logN, m):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    prm = HEParams(logN=logN, q=m[2:], p=m[:2], dnum=2, scale=2.0 ** 40, hamming=64, name="line")
    orc, ctx, N, level, step = Oracle.from_params(prm), HEContext.from_params(prm), prm.N, 3, 3
    rng, g, idx = S.make_rng(77 + logN), orc.galois_elt(step), [0, 1, 2, 3] * 2

    def top(moduli, n):
        return np.broadcast_to(np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1), (n, len(moduli), N)).copy()

    for fill in (top, lambda moduli, n: S.uniform_limbs(rng, moduli, N, n)):
        a = fill(prm.q, 2).reshape(8, N)
        d = dev(a)
        ctx.he_ntt(d, idx)
        assert (host(d) == orc.ntt(a, idx)).all()
        d = dev(a)
        ctx.he_intt(d, idx)
        assert (host(d) == orc.intt(a, idx)).all()
        key, ct = fill(prm.moduli, 4).reshape(2, 2, -1, N), fill(prm.q, 2)
        ctx.he_evk_register(g, dev(key))
        d_ct, out, down = dev(ct), zeros(2, 4, N), zeros(2, 3, N)
        ctx.he_rotate(d_ct, level, step, out)
        assert (host(out) == orc.rotate(ct, level, g, key)).all()
        ctx.he_rotate_sum([d_ct, d_ct, d_ct], level, [step, 0, step], out, deferred=True)
        assert (host(out) == orc.rotate_sum_deferred([ct, ct, ct], level, [g, 1, g], [key, None, key])).all()
        ctx.he_rescale(d_ct, level, down)
        assert (host(down) == orc.rescale(ct, level)).all()


# Limbs of each modulus whose launches leave the 64 threads to a row (more than 4096 wavefronts of the 16-thread form): runs of 4 with one and
# none left over, two rounds of a run with one limb in the last; and 5 limbs of each modulus, runs too poorly filled, a row per 16 lanes.
@pytest.mark.parametrize("line,side", SIDES)
@pytest.mark.parametrize("logN,counts", [(14, (85, 88, 85)), (16, (17, 16, 32)), (16, (133, 130, 129)), (16, (5,) * 13), (17, (5,) * 7)])
def test_rows_of_large_launches(line, side, logN, counts):
    check_large_launches(logN, counts, primes_at(line, side, logN, len(counts)))


def check_large_launches(logN, counts, m):
    from gpu_util import dev, host
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    N = 1 << logN
    assert sum(counts) * (N >> 10) > 4096
    orc, ctx, rng = Oracle(logN, m[1:], m[:1], 2), HEContext(logN, m[1:], m[:1], 2), S.make_rng(177 + logN + len(counts))
    moduli, idx = m[1:] + m[:1], [i for i, n in enumerate(counts) for _ in range(n)]
    rng.shuffle(idx)
    a = np.stack([S.uniform_limbs(rng, [moduli[i]], N)[0][0] for i in idx])
    for i in range(0, len(idx), 3):
        a[i] = moduli[idx[i]] - 1
    d = dev(a)
    ctx.he_ntt(d, idx)
    assert (host(d) == orc.ntt(a, idx)).all()
    d = dev(a)
    ctx.he_intt(d, idx)
    assert (host(d) == orc.intt(a, idx)).all()


@pytest.mark.parametrize("logN", [13, 15])
@pytest.mark.parametrize("line,side", SIDES)
def test_batches_of_key_switches(line, side, logN):
    check_batches(logN, primes_at(line, side, logN, 9))


def check_batches(logN, m):
    """Nine ciphertexts: conversions in tiles of 1024 points and key-switch rows of a wavefront each, where the tests above have too few (at
    2^13 complete digits still give each component a wavefront); every step on its own and sharing a decomposition, sums of both
    kinds, a product, a hoisted sum."""
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    C_a = 16
    prm = HEParams(logN=logN, q=m[3:], p=m[:3], dnum=3, scale=2.0 ** 40, hamming=64, name="line")
    orc, ctx, N, level = Oracle.from_params(prm), HEContext.from_params(prm), prm.N, 5
    rng, block, steps = S.make_rng(277), N // 2 // C_a, [1, 2, 300]
    keys = [tops(prm.moduli, 6, N).reshape(3, 2, -1, N), S.uniform_limbs(rng, prm.moduli, N, 6).reshape(3, 2, -1, N)]
    d_keys, key_of = [dev(k) for k in keys], {}
    for n, step in enumerate(steps + [block * i for i in range(1, C_a)]):
        key_of[step] = keys[n % 2]
        ctx.he_evk_register(ctx.galois_elt(step), d_keys[n % 2])
    ctx.he_evk_register(0, d_keys[0])
    cts = [tops(prm.q, 2, N)] + [S.uniform_limbs(rng, prm.q, N, 2) for _ in range(8)]
    d_cts = [dev(c) for c in cts]
    want = [orc.rotate(c, level, orc.galois_elt(s), key_of[s]) for c in cts for s in steps]
    for hoisted in (False, True):
        outs = [zeros(2, level + 1, N) for _ in want]
        ctx.he_rotate_batch(d_cts, level, steps, outs, hoisted=hoisted)
        assert all((host(o) == w).all() for o, w in zip(outs, want)), hoisted
    out, turns = zeros(2, level + 1, N), (steps * 3)[:9]
    ctx.he_rotate_sum(d_cts, level, turns, out, deferred=True)
    assert (host(out) == orc.rotate_sum_deferred(cts, level, [orc.galois_elt(s) for s in turns], [key_of[s] for s in turns])).all()
    ctx.he_rotate_sum([d_cts[0]] * 3, level, steps, out, deferred=True)
    assert (host(out) == orc.rotate_sum_deferred([cts[0]] * 3, level, [orc.galois_elt(s) for s in steps], [key_of[s] for s in steps])).all()
    ctx.he_mulct(d_cts[0], d_cts[1], level, out)
    assert (host(out) == orc.mulct(cts[0], cts[1], level, keys[0])).all()
    gs, pts = [orc.galois_elt(block * i) for i in range(1, C_a)], [tops(prm.q, 1, N)[0], S.uniform_limbs(rng, prm.q, N, 1)[0]]
    got = ctx.he_conv2d(C_a, 1, block, 1, 1, level, [dev(p) for p in pts], d_cts[1], [zeros(2, level, N) for _ in pts], hoisted_ras=True)
    for p, o in zip(pts, got):
        x = orc.rescale(orc.ptct_mac(None, cts[1], p, level, init=True), level)
        assert (host(o) == orc.rotate_sum_deferred([x] * C_a, level - 1, [1] + gs, [None] + [key_of[block * i] for i in range(1, C_a)])).all()
