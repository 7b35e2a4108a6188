"""What a butterfly costs is its instructions (ntt_blocks.h): forward eight multiply-adds, the difference, and one addition and one minimum
for every conditional subtraction; of moduli near a multiple of 2^32 (class 3, both directions) seven multiply-adds, one product, one addition,
no conditional subtraction and no second words of factors - counted in the compiler's output for four stages on 16 points, of every class of
moduli."""
import collections
import os
import subprocess

import pytest

from paper_2302_02407_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
STAGES = """#include "ntt_blocks.h"
__global__ __launch_bounds__(256) void stages_kernel(unsigned long long* a, ulonglong2* tw, u64 q) {
    u64 x[16];
    ulonglong2 w[15];
    int b = w_lim(%d);
    for (int k = 0; k < 16; k++) x[k] = a[256 * k + threadIdx.x];
    const ctw_t c = (ctw_t)(uintptr_t)tw;
    for (int k = 0; k < 15; k++) %s;
    %s_stages<%d, 0, 4, %s>(x, w, q, b);
    for (int k = 0; k < 16; k++) a[256 * k + threadIdx.x] = x[k];
}
"""
BUTTERFLIES, FACTORS = 32, 15


def counted(tmp_path, W, uniform, direction="fwd"):
    src, u = tmp_path / "k.hip", "true" if uniform else "false"
    src.write_text(STAGES % (W, "w[k].x = c[k].x, w[k].y = c[k].y" if uniform else "w[k] = tw[256 * k + threadIdx.x]", direction, W, u))
    flags = [f for f in build.FLAGS if not f.startswith("-Rpass")]
    out = subprocess.run([HIPCC] + flags + ["-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", "-"], capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    return collections.Counter(l.split()[0] for l in out.stdout.splitlines() if l.startswith("\tv_"))


@pytest.mark.parametrize("uniform", [False, True])
@pytest.mark.parametrize("W", [0, 1, 2])
def test_forward_butterflies(tmp_path, W, uniform):
    n = counted(tmp_path, W, uniform)
    # halvings: X before every stage but where the sum stays in range, twice for the widest
    halvings = n["v_min_f64_e64"] + n["v_min_f64"]
    assert halvings == (0 if W == 0 else BUTTERFLIES * W)
    assert n["v_mad_u64_u32"] == BUTTERFLIES * 8 + (0 if uniform else 2 * FACTORS)
    # 2X + 5q, and the difference of every conditional subtraction; two for addresses
    assert n["v_lshl_add_u64"] <= BUTTERFLIES + halvings + 2


@pytest.mark.parametrize("uniform", [False, True])
@pytest.mark.parametrize("direction", ["fwd", "inv"])
def test_near_butterflies(tmp_path, direction, uniform):
    n = counted(tmp_path, 3, uniform, direction)
    assert n["v_mad_i64_i32"] == 7 * BUTTERFLIES and n["v_mul_lo_u32"] == BUTTERFLIES
    assert n["v_min_f64_e64"] + n["v_min_f64"] + n["v_mad_u64_u32"] == 0
    # an operand's rounded upper word, inverse also the sum of the points; two for addresses
    assert n["v_lshl_add_u64"] <= BUTTERFLIES * (1 if direction == "fwd" else 2) + 2
    # the difference: 2X (forward) and two with a borrow
    assert n["v_lshlrev_b64"] == (BUTTERFLIES if direction == "fwd" else 0)
    assert sum(v for k, v in n.items() if k.startswith("v_sub")) == 2 * BUTTERFLIES
