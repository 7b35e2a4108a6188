"""GPU parity: the basis conversion fused with its column passes (matrix-core contraction) at the edges of its range -
1 to 8 sources, target counts that leave rounds of eight and groups of four partly empty, the smallest and widest moduli it
takes, uniform and extreme residues - against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import toy_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,q_bits,nq,p_bits,np_,dnum,levels", [
    (13, 36, 9, 37, 1, 9, (8, 4)),       # one source; more sets than one launch takes (9 digits) and exactly 5
    (13, 60, 5, 59, 5, 1, (4, 0)),       # only wide moduli, five sources; a single source limb
    (14, 54, 16, 60, 8, 2, (15, 9)),     # eight sources, sixteen targets; a partial second digit of two
    (15, 50, 7, 51, 4, 2, (6, 2)),       # moduli on both sides of the quotient's shift rule; a digit of four and one of three
    (16, 54, 11, 60, 3, 2, (10, 5)),     # six and five sources, eight and nine targets
])
@pytest.mark.parametrize("fill", ["uniform", "extreme"])
@pytest.mark.parametrize("n_ct", [1, 3])         # small tiles for the lowest level of one ciphertext, large ones otherwise
def test_conversion_edges(logN, q_bits, nq, p_bits, np_, dnum, levels, n_ct, fill):
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    prm = toy_params(logN=logN, q_bits=q_bits, nq=nq, p_bits=p_bits, np_=np_, dnum=dnum, hamming=64, seed=700 + logN)
    rng, orc, ctx = S.make_rng(700 + logN), Oracle.from_params(prm), HEContext.from_params(prm)
    N, step = prm.N, 3

    def residues(moduli, n):
        if fill == "uniform":
            return S.uniform_limbs(rng, moduli, N, n)
        top = np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1)
        return np.where(rng.integers(0, 2, size=(n, len(moduli), N)) == 1, top, np.uint64(0))

    key = residues(prm.moduli, 2 * dnum).reshape(dnum, 2, len(prm.moduli), N)
    ctx.he_evk_register(ctx.galois_elt(step), dev(key))
    for level in levels:
        cts = [residues(prm.q[:level + 1], 2) for _ in range(n_ct)]
        outs = [zeros(2, level + 1, N) for _ in range(n_ct)]
        ctx.he_rotate_batch([dev(c) for c in cts], level, [step], outs, hoisted=False)
        for c, o in zip(cts, outs):
            assert (host(o) == orc.rotate(c, level, orc.galois_elt(step), key)).all(), level


@pytest.mark.parametrize("logN,bits,n_ct", [(13, 60, 6), (13, 36, 6), (15, 60, 2), (16, 36, 1)])
@pytest.mark.parametrize("fill", ["top", "mixed"])
def test_full_contraction_of_the_widest_primes(logN, bits, n_ct, fill):
    """Eight sources and sixteen targets in tiles of 1024 points (the smallest ring among them, whose small batches all take the
    small tiles), primes just below 2^60 and 2^36, every residue at its top or at zero."""
    from gpu_util import dev, host, zeros
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    from test_gpu_widest_primes import primes_below
    m = primes_below(1 << bits, 2 << logN, 24)
    q, p, dnum, level, step = m[8:], m[:8], 2, 15, 5
    rng, orc, ctx, N = S.make_rng(800 + logN + bits), Oracle(logN, q, p, dnum), HEContext(logN, q, p, dnum), 1 << logN

    def residues(moduli, n):
        top = np.broadcast_to(np.array(moduli, dtype=np.uint64)[None, :, None] - np.uint64(1), (n, len(moduli), N)).copy()
        if fill == "mixed":
            top[rng.integers(0, 2, size=top.shape) == 1] = 0
        return top

    key = residues(q + p, 2 * dnum).reshape(dnum, 2, 24, N)
    ctx.he_evk_register(ctx.galois_elt(step), dev(key))
    cts = [residues(q, 2) for _ in range(n_ct)]
    outs = [zeros(2, level + 1, N) for _ in cts]
    ctx.he_rotate_batch([dev(c) for c in cts], level, [step], outs, hoisted=False)
    for c, o in zip(cts, outs):
        assert (host(o) == orc.rotate(c, level, orc.galois_elt(step), key)).all()
