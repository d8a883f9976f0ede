"""The binding's use of the torch node without a GPU."""
import os
import sys

import pytest
import torch

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14669_amd", "libquartet.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="HIP library not built (run __graft_entry__.build())")
NODE = "paper_2505_14669_amd._nn_native"


class Broken:
    """finder under which the torch node exists and does not load"""

    @staticmethod
    def find_spec(name, path=None, target=None):
        if name == NODE:
            raise ImportError("_nn_native.so: undefined symbol: quartet_linear_fwd")


@pytest.mark.parametrize("broken", [False, True])
def test_calls_without_the_torch_node_say_so(monkeypatch, broken):
    import paper_2505_14669_amd as package
    from paper_2505_14669_amd import binding as q
    for name in ("_native", "_current_device", "_current_raw_stream"):
        monkeypatch.setattr(q, name, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: None)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0, raising=False)
    monkeypatch.delattr(package, "_nn_native", raising=False)
    if broken:
        monkeypatch.delitem(sys.modules, NODE, raising=False)
        monkeypatch.setattr(sys, "meta_path", [Broken, *sys.meta_path])
    else:
        monkeypatch.setitem(sys.modules, NODE, None)
    with pytest.warns(RuntimeWarning, match="undefined symbol" if broken else "not available"):
        assert q.quartet_quant_fwd(0x10000, 0, 64, 64, 0, 0x10000, 0x10000, 0x10000) == q.QUARTET_OK      # empty: no launch
    assert q._native is None
