"""The list that places the step's kernels in the code object names kernels that are there: a stale name would silently leave its
kernel where chance puts it."""
import pytest

from paper_2503_00784_amd import binding, build


def _listed():
    with open(build.KERNEL_ORDER) as f:
        return [line.strip() for line in f if line.strip() and not line.startswith("#")]


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_every_listed_kernel_is_in_the_library(dtype):
    names = _listed()
    assert len(names) > 50 and len(set(names)) == len(names)
    with open(binding.LIB_PATHS[dtype], "rb") as f:
        image = f.read()
    missing = [n for n in names if n.encode() + b"\0" not in image]
    assert not missing
