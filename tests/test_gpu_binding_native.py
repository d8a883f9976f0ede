"""The binding's calls without ctypes: the same results and the same refusals as the conversion in Python."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture()
def q():
    from paper_2505_14669_amd import binding
    torch.zeros(1, device="cuda")
    binding._stream(None)
    assert binding._native is not None
    return binding


class Sub(torch.Tensor):
    pass


def buffers(q, rows, k):
    return (torch.zeros((rows, k // 2), dtype=torch.uint8, device="cuda"), torch.zeros(q.quartet_scale_bytes(rows, k), dtype=torch.uint8, device="cuda"),
            torch.zeros((rows, k // 32), dtype=torch.int32, device="cuda"))


def test_same_bytes_and_same_refusals(q, monkeypatch):
    rows, k = 40, 96
    x = torch.randn((rows, k), device="cuda").to(torch.bfloat16)
    want = buffers(q, rows, k)
    with monkeypatch.context() as m:
        m.setattr(q, "_native", None)
        q.check(q.quartet_quant_fwd(x, rows, k, k, 0, *want))
    side = torch.cuda.Stream()
    for tensor, sizes, stream in ((x, (rows, k, k, False), None), (torch.nn.Parameter(x), (rows, k, k, 0), torch.cuda.current_stream().cuda_stream),
                                  (x.as_subclass(Sub), (rows, k, k, 0), None), (x.data_ptr(), (rows, k, k, 0), None),
                                  (x, tuple(np.int64(v).item() for v in (rows, k, k, 0)), side)):
        got = buffers(q, rows, k)
        torch.cuda.synchronize()
        q.check(q.quartet_quant_fwd(tensor, *sizes, *got, stream))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    for bad, error in ((x.cpu(), q.QuartetError), (x.t(), q.QuartetError), (x.to("meta"), q.QuartetError), ("x", AttributeError)):
        with pytest.raises(error):
            q.quartet_quant_fwd(bad, rows, k, k, 0, *want)
    with pytest.raises(Exception):
        q.quartet_quant_fwd(x, 40.0, k, k, 0, *want)
    assert q.quartet_quant_fwd(None, rows, k, k, 0, *want) == q.QUARTET_EINVAL
    assert q.quartet_quant_fwd(x, -1, k, k, 0, *want) == q.QUARTET_EINVAL


def test_current_stream_of_each_thread(q):
    a = torch.randn((512, 1024), device="cuda").to(torch.bfloat16)
    want = buffers(q, 512, 1024)
    q.check(q.quartet_quant_fwd(a, 512, 1024, 1024, 0, *want))
    torch.cuda.synchronize()
    results = [buffers(q, 512, 1024) for _ in range(4)]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                q.check(q.quartet_quant_fwd(a, 512, 1024, 1024, 0, *results[i]))
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(torch.equal(x, y) for r in results for x, y in zip(r, want))
