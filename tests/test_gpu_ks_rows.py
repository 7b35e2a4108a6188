"""GPU parity: key switches whose sources serve one job each and sums of rotations of different ciphertexts, whose digits are
transformed inside the row kernels - in both forms (a row to a wavefront, a row to a work group), with 1 to 8 digits, primes at the
top of every width the kernels tell apart, uniform and extreme residues - against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import HEParams, is_prime

pytestmark = pytest.mark.gpu


def primes_below(top, two_n, count, skip=()):
    c, out = top - two_n + 1, []
    while len(out) < count:
        if c not in skip and is_prime(c):
            out.append(c)
        c -= two_n
    return out


@pytest.mark.parametrize("logN,q_bits,p_bits,nq,np_,dnum,levels,n_ct", [
    (13, 30, 31, 4, 1, 4, (3, 0), 3),        # primes below 2^32: sums put together in 128 bits
    (13, 54, 60, 8, 1, 8, (7, 4), 16),       # eight digits: special primes by work groups, the others by wavefronts
    (13, 40, 41, 20, 4, 5, (19,), 16),       # sixteen jobs a set, more limbs than one transform launch lists
    (13, 55, 54, 5, 2, 3, (4, 1), 2),        # two digits of two and one of one
    (14, 57, 58, 6, 2, 3, (5, 2), 7),
    (15, 60, 60, 8, 1, 8, (7,), 9),          # more products than one sum holds, in both launches
    (16, 54, 54, 2, 1, 2, (1, 0), 5),        # narrow special primes
    (16, 60, 59, 3, 2, 1, (2,), 1),          # one digit
    (17, 55, 57, 3, 1, 3, (2, 1), 2),
])
@pytest.mark.parametrize("fill", ["uniform", "extreme"])
def test_one_job_sources(logN, q_bits, p_bits, nq, np_, dnum, levels, n_ct, fill):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    q = primes_below(1 << q_bits, 2 << logN, nq)
    p = primes_below(1 << p_bits, 2 << logN, np_, skip=q)
    prm = HEParams(logN=logN, q=q, p=p, dnum=dnum, scale=2.0 ** 20, hamming=64, name="rows")
    rng, orc, ctx = S.make_rng(500 + logN + q_bits), Oracle.from_params(prm), HEContext.from_params(prm)
    N = prm.N
    steps = [3, N // 2 - 5]

    def residues(moduli, n):
        if fill == "uniform":
            return S.uniform_limbs(rng, moduli, N, n)
        top = np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1)
        return np.where(rng.integers(0, 4, size=(n, len(moduli), N)) > 0, top, np.uint64(0))

    keys = {s: residues(prm.moduli, 2 * dnum).reshape(dnum, 2, len(prm.moduli), N) for s in steps}
    for s, k in keys.items():
        ctx.he_evk_register(ctx.galois_elt(s), dev(k))
    rot = lambda c, level, s: orc.rotate(c, level, orc.galois_elt(s), keys[s])
    for level in levels:
        cts = [residues(prm.q[:level + 1], 2) for _ in range(n_ct)]
        d_cts = [dev(c) for c in cts]
        outs = [zeros(2, level + 1, N) for _ in range(2 * n_ct)]
        ctx.he_rotate_batch(d_cts, level, steps, outs, hoisted=False)
        for i in {0, n_ct // 2, n_ct - 1}:
            for j, s in enumerate(steps):
                assert (host(outs[2 * i + j]) == rot(cts[i], level, s)).all(), ("batch", level, i, s)
        o0, o1 = zeros(level + 1, N), zeros(level + 1, N)
        ctx.he_keyswitch(d_cts[0][1], level, ctx.galois_elt(steps[0]), o0, o1)
        w0, w1 = orc.keyswitch(cts[0][1], level, keys[steps[0]])
        assert (host(o0) == w0).all() and (host(o1) == w1).all(), ("keyswitch", level)
        for n in {1, min(n_ct, 3), n_ct}:                # terms spread over the wavefronts of a work group
            ts = [steps[i % 2] for i in range(n)] + [0]
            out = zeros(2, level + 1, N)
            ctx.he_rotate_sum(d_cts[:n] + [d_cts[0]], level, ts, out, deferred=True)
            want = orc.rotate_sum_deferred(cts[:n] + [cts[0]], level, [orc.galois_elt(s) for s in ts], [keys.get(s) for s in ts])
            assert (host(out) == want).all(), ("sum", level, n)


@pytest.mark.parametrize("logN,q_bits,p_bits,nq,np_,dnum,levels,n_ct", [
    (13, 30, 31, 4, 1, 4, (3, 0), 1),        # a wavefront to a component
    (13, 40, 41, 20, 4, 5, (19,), 6),        # a set of sixteen jobs and one of two
    (13, 54, 60, 8, 1, 8, (7, 4), 3),        # eight digits and five
    (14, 58, 57, 6, 2, 3, (5, 2), 5),
    (16, 54, 54, 3, 3, 2, (2,), 4),          # 9216 rows: a wavefront to both components
    (16, 57, 55, 3, 3, 1, (2, 1), 4),
    (16, 60, 60, 3, 3, 2, (2,), 4),
    (17, 55, 58, 2, 2, 2, (1,), 4),
])
@pytest.mark.parametrize("fill", ["uniform", "extreme"])
def test_shared_sources(logN, q_bits, p_bits, nq, np_, dnum, levels, n_ct, fill):
    """Sources that serve three jobs, or several terms of one sum: the row kernels take digits that are transformed already."""
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    q = primes_below(1 << q_bits, 2 << logN, nq)
    p = primes_below(1 << p_bits, 2 << logN, np_, skip=q)
    prm = HEParams(logN=logN, q=q, p=p, dnum=dnum, scale=2.0 ** 20, hamming=64, name="rows")
    rng, orc, ctx = S.make_rng(700 + logN + q_bits), Oracle.from_params(prm), HEContext.from_params(prm)
    N = prm.N
    steps = [1, N // 4 + 3, N // 2 - 6]

    def residues(moduli, n):
        if fill == "uniform":
            return S.uniform_limbs(rng, moduli, N, n)
        top = np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1)
        return np.where(rng.integers(0, 4, size=(n, len(moduli), N)) > 0, top, np.uint64(0))

    keys = {s: residues(prm.moduli, 2 * dnum).reshape(dnum, 2, len(prm.moduli), N) for s in steps}
    for s, k in keys.items():
        ctx.he_evk_register(ctx.galois_elt(s), dev(k))
    rot = lambda c, level, s: orc.rotate_from_raised(c, orc.modup(c[1], level), level, orc.galois_elt(s), keys[s])
    for level in levels:
        cts = [residues(prm.q[:level + 1], 2) for _ in range(n_ct)]
        d_cts = [dev(c) for c in cts]
        outs = [zeros(2, level + 1, N) for _ in range(3 * n_ct)]
        ctx.he_rotate_batch(d_cts, level, steps, outs, hoisted=True)
        for i in {0, n_ct - 1}:
            for j, s in enumerate(steps):
                assert (host(outs[3 * i + j]) == rot(cts[i], level, s)).all(), ("batch", level, i, s)
        for n in {2, 3 * n_ct - 1}:
            src, ts = [i // 3 for i in range(n)], [steps[i % 3] for i in range(n)]
            out = zeros(2, level + 1, N)
            ctx.he_rotate_sum([d_cts[i] for i in src], level, ts, out, deferred=True)
            want = orc.rotate_sum_deferred([cts[i] for i in src], level, [orc.galois_elt(s) for s in ts], [keys[s] for s in ts])
            assert (host(out) == want).all(), ("sum", level, n)
