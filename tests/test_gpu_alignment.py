"""GPU: every buffer a caller gives - ciphertexts, plaintexts, keys, outputs - may start at any multiple of 8 bytes.  The calls
whose kernels take two residues per access, on buffers that lie 8 bytes past a multiple of 16, against the same calls on
aligned ones (which the oracle tests cover)."""
import pytest

from he_inputs import sampling as S
from he_inputs.params import toy_params

pytestmark = pytest.mark.gpu


def _past16(t):
    """A copy of t that starts 8 bytes past a multiple of 16."""
    import torch
    v = torch.empty(t.numel() + 1, dtype=torch.int64, device="cuda")[1:].view(t.shape)
    assert v.data_ptr() % 16 == 8
    return v.copy_(t)


def _as_is(t):
    assert t.data_ptr() % 16 == 0
    return t.clone()


@pytest.mark.parametrize("logN,bits,n_polys", [
    (11, 40, 2),      # FP64 kernels
    (12, 54, 2),      # integer kernels of the small rings
    (13, 54, 2),      # rows of 64 threads
    (13, 60, 2),      # their wide form
    (14, 54, 60),     # runs of one modulus, rows of 16 threads
])
def test_buffers_off_by_eight_bytes(logN, bits, n_polys):
    import torch
    from gpu_util import dev
    from paper_2302_02407_amd.binding import HEContext
    prm = toy_params(logN=logN, q_bits=bits, nq=4, p_bits=bits - 1, np_=2, dnum=2, hamming=16, seed=40 + logN)
    rng, N, level = S.make_rng(40 + logN), prm.N, 3
    draw = lambda n, lv: [dev(a).view(torch.int64) for a in S.uniform_limbs(rng, prm.q[:lv + 1], N, n)]
    key = lambda: dev(S.uniform_limbs(rng, prm.moduli, N, 2 * prm.dnum).reshape(prm.dnum, 2, -1, N)).view(torch.int64)
    C_a, W, R, f = 4, 4, 2, 3
    H = N // 2 // (C_a * W * R)
    taps = sorted({((dy * W + dx) * R) % (N // 2) for dy in (-1, 0, 1) for dx in (-1, 0, 1)} - {0})
    ras = [H * W * R * i for i in range(1, C_a)]
    cts = [torch.stack(draw(2, level)) for _ in range(9)]
    pts, polys = draw(18, level), torch.stack(draw(n_polys, level))
    ctx = HEContext.from_params(prm)
    elts = [0] + [ctx.galois_elt(s) for s in sorted(set(taps + ras))]
    keys = {g: key() for g in elts}
    idx = [i % 4 for i in range(4 * n_polys)]

    def run(put):
        res = lambda lv, *lead: put(torch.zeros(lead + (2, lv + 1, N), dtype=torch.int64, device="cuda"))
        for g in elts:
            ctx.he_evk_register(g, put(keys[g]))
        c, p = [put(x) for x in cts], [put(x) for x in pts]
        got = [ctx.he_ntt(put(polys), idx), ctx.he_intt(put(polys), idx)]
        got += ctx.he_rotate_batch(c, level, ras, [res(level) for _ in range(27)], hoisted=False)        # many limbs ...
        got += ctx.he_rotate_batch(c[:2], level, ras[:1], [res(level) for _ in range(2)], hoisted=True)  # ... and few
        got.append(ctx.he_mulct(c[0], c[1], level, res(level)))
        got.append(ctx.he_rescale(c[0], level, res(level - 1)))
        got.append(ctx.he_rotate_sum(c[:3], level, [0] + taps[:2], res(level), deferred=True))
        acc = ctx.he_ptct_mac_rot(res(level), c, p[:9], [1, 5] + [ctx.galois_elt(s) for s in range(3, 10)], level)
        got.append(ctx.he_ptct_mac_rot(acc, c[:2], p[:2], [1, 1], level, init=False))
        for hoisted in (False, True):
            got += ctx.he_conv2d(C_a, H, W, R, f, level, p, c[0], [res(level - 1) for _ in range(2)], hoisted_ras=hoisted)
        got.append(ctx.he_raconv(W, R, f, level, p, c[:2], res(level - 1), deferred=True))
        got.append(ctx.he_raconv(W, R, f, level, p, c[:2], res(level - 1)))
        ctx.he_sync()
        return got

    for i, (a, b) in enumerate(zip(run(_as_is), run(_past16))):
        assert (a == b).all(), i
