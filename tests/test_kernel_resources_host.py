"""The compiler's registers and LDS leave the waves per SIMD that the launches count on (compiled here, no GPU)."""
import os

import pytest

from paper_2605_03109_amd import build


@pytest.mark.parametrize("name", sorted(set(build.MIN_WAVES) | set(build.NO_SCRATCH)))
def test_kernel_resources(name, tmp_path):
    try:
        build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc is not installed")
    assert os.path.exists(build._compile(os.path.join(build.HERE, "csrc", name), str(tmp_path / "o")))


def test_too_few_waves_are_refused():
    remark = "remark: Function Name: _Z10proj_stagev\nremark:     Occupancy [waves/SIMD]: {}\n"
    assert build.check_resources("gsi_stage.hip", remark.format(5)) == 1
    with pytest.raises(RuntimeError, match="4 waves"):
        build.check_resources("gsi_stage.hip", remark.format(4))
