"""The Python binding's own bookkeeping on a GPU: what names a device, and whose stream a workspace belongs to."""
import pytest

import paper_2311_09550_amd as w4a8

pytestmark = pytest.mark.gpu


def test_workspace_takes_every_name_of_the_current_device(gpu):
    """No device, "cuda", its ordinal and "cuda:0" are one device: one workspace per stream of it, another on another stream."""
    t = gpu
    first = w4a8.workspace(4, 64, 256)
    for name in ("cuda", t.device("cuda"), "cuda:0", t.device("cuda", 0), 0):
        assert w4a8.workspace(4, 64, 256, device=name) is first, name
    assert first.device == t.device("cuda", 0) and first.dtype == t.uint8 and not bool(first.any())
    with t.cuda.stream(t.cuda.Stream()):
        assert w4a8.workspace(4, 64, 256, device="cuda") is not first
    for name in ("cpu", "cpu:0"):
        with pytest.raises(ValueError):
            w4a8.workspace(4, 64, 256, device=name)
