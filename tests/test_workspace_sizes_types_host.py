"""Scratch sizes: a size that is no integer is refused, whatever was asked before."""
import pytest

pytest.importorskip("torch")


def test_no_float_sizes_after_equal_integers():
    from paper_2605_03109_amd import gsi

    which = gsi.CALL_BUILD_IMAGE
    have = gsi.workspace_bytes(which, 4096, 2048, 64, 0)
    for args in ((which, 4096.0, 2048, 64, 0), (which, 4096, 2048, 64.0, 0), (float(which), 4096, 2048, 64, 0)):
        with pytest.raises(Exception, match="wrong type|cannot be interpreted"):
            gsi.workspace_bytes(*args)
    assert gsi.workspace_bytes(which, 4096, 2048, 64, 0) == have
