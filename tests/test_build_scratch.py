"""The build refuses a kernel that uses scratch memory and leaves no object of it behind."""
import os

import pytest

from paper_2302_02407_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARRAY = """#include <hip/hip_runtime.h>
__global__ void table_kernel(int* a, int n) {
    int t[64];
    for (int i = 0; i < 64; i++) t[(a[i] + n) & 63] = a[i];
    a[threadIdx.x] = t[a[threadIdx.x] & 63];
}
"""
# sixty-four values a lane that all have to be there at once, in the 64 registers that 8 wavefronts to a SIMD leave each
SPILL = """#include <hip/hip_runtime.h>
__global__ __launch_bounds__(256, 8) void wide_kernel(unsigned long long* a, int n) {
    unsigned long long v[64];
#pragma unroll
    for (int i = 0; i < 64; i++) v[i] = a[threadIdx.x + 256 * i];
    for (int r = 0; r < n; r++) {
#pragma unroll
        for (int i = 0; i < 64; i++) v[i] += v[(i + 17) & 63] * v[(i + 5) & 63];
    }
#pragma unroll
    for (int i = 0; i < 64; i++) a[threadIdx.x + 256 * i] = v[i];
}
"""
PLAIN = """#include <hip/hip_runtime.h>
__global__ void plain_kernel(int* a) { a[threadIdx.x] += 1; }
"""


def sources(tmp_path, text):
    src, obj = tmp_path / "k.hip", tmp_path / "k.o"
    src.write_text(text)
    return str(src), str(obj)


@pytest.mark.parametrize("text,kernel", [(ARRAY, "table_kernel"), (SPILL, "wide_kernel"), (PLAIN + SPILL.split("\n", 1)[1], "wide_kernel")])
def test_scratch_is_refused(tmp_path, text, kernel):
    src, obj = sources(tmp_path, text)
    with pytest.raises(RuntimeError, match=kernel) as e:
        build.compile_object(HIPCC, src, obj)
    assert "plain_kernel" not in str(e.value) and not os.path.exists(obj)


def test_a_kernel_without_is_built(tmp_path):
    src, obj = sources(tmp_path, PLAIN)
    build.compile_object(HIPCC, src, obj)
    assert os.path.exists(obj)


def test_every_kernel_is_reported(tmp_path):
    """The refusal rests on the compiler's report: it has to be there, with the amount under the name that is looked for."""
    src, obj = sources(tmp_path, PLAIN)
    fields = [build.FIELD.search(l) for l in build._run([HIPCC] + build.FLAGS + ["-c", src, "-o", obj], False)]
    got = {m.group(1): m.group(2) for m in fields if m}
    assert "plain_kernel" in got["Function Name"] and got["ScratchSize [bytes/lane]"] == "0" and got["Dynamic Stack"] == "False"
