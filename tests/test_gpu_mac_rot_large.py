"""GPU parity: he_ptct_mac_rot whose operands exceed the size from which ciphertexts are read past the caches - whole fours of terms
and a remainder, a second launch below that size, operands at odd residues of a buffer - against the oracle, bit for bit."""
import numpy as np
import pytest

from he_inputs import sampling as S
from he_inputs.params import config_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,level,shift", [(16, 8, 0), (15, 9, 1), (18, 8, 0)])
def test_large_sum(n, level, shift):
    import torch

    from gpu_util import dev, host, zeros
    from oracle import prcr as PR
    from oracle.he_oracle import Oracle
    from paper_2302_02407_amd.binding import HEContext
    prm = config_params(2)
    assert min(n, 16) * 3 * (level + 1) * prm.N * 8 > 192 << 20
    rng, orc, ctx = S.make_rng(60 + n), Oracle.from_params(prm), HEContext.from_params(prm)
    N, qs = prm.N, prm.q[:level + 1]
    cts = [S.uniform_limbs(rng, qs, N, 2) for _ in range(n)]
    pts = [S.uniform_limbs(rng, qs, N)[0] for _ in range(n)]
    cts[0][:] = np.array(qs, dtype=np.uint64)[None, :, None] - np.uint64(1)
    gs = [1 if i == 1 else orc.galois_elt(int(rng.integers(1, N // 2))) for i in range(n)]

    def put(a):
        buf = torch.empty(a.size + shift, dtype=dev(a[..., :1]).dtype, device="cuda")
        buf[shift:].copy_(dev(a).reshape(-1))
        return buf[shift:].reshape(a.shape)

    acc = zeros(2, level + 1, N)
    ctx.he_ptct_mac_rot(acc, [put(c) for c in cts], [put(p) for p in pts], gs, level, init=True)
    assert (host(acc) == PR.mac_rotated_plaintexts(orc, cts, pts, gs, level)).all()
