"""The build refuses a kernel whose conditional subtractions (csub_min) run in a mode in which they are wrong, and leaves no object of it
behind."""
import os

import pytest

from paper_2302_02407_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
INCLUDE = '#include "modarith.h"\n'
KERNEL = """__global__ void halved_kernel(u64* a, u64 q, int n) {
    %s
    a[threadIdx.x] = csub_min(a[threadIdx.x], q);
}
"""
SET, UNSET, SOMETIMES = "ieee_off();", "", "if (n & 1) { ieee_off(); a[64 + threadIdx.x] = n; }"
OTHER = KERNEL.replace("halved_kernel", "other_kernel")


def compiled(tmp_path, text):
    src, obj = tmp_path / "k.hip", tmp_path / "k.o"
    src.write_text(INCLUDE + text)
    build.compile_object(HIPCC, str(src), str(obj), ["-I", build.CSRC])
    return str(obj)


@pytest.mark.parametrize("text", [KERNEL % UNSET, KERNEL % SOMETIMES, OTHER % SET + KERNEL % UNSET, KERNEL % UNSET + OTHER % SET],
                         ids=["never", "behind a branch", "after one that does", "before one that does"])
def test_a_kernel_in_the_wrong_mode_is_refused(tmp_path, text):
    with pytest.raises(RuntimeError, match="halved_kernel") as e:
        compiled(tmp_path, text)
    assert "other_kernel" not in str(e.value) and not (tmp_path / "k.o").exists()


def test_a_kernel_that_sets_it_is_built(tmp_path):
    listing = build.device_listing(HIPCC, compiled(tmp_path, KERNEL % SET))
    assert any("v_min_f64" in l for l in listing)           # the refusal rests on the instruction's name


def test_every_object_of_the_library_is_looked_at():
    """`build_library` compiles by `compile_object`; what it made holds such kernels, all of them in the right mode."""
    objs = [os.path.join(build.OBJ, s + ".o") for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        pytest.skip("the library was built elsewhere")
    listings = [build.device_listing(HIPCC, o) for o in objs]
    assert sum(any("v_min_f64" in l for l in x) for x in listings) >= 4
    assert [k for x in listings for k in build.ieee_kernels(x)] == []
