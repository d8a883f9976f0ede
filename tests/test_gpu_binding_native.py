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


class NoCtypes:
    """in the library's place: a call that is not native ends here"""

    def __getattr__(self, name):
        raise AssertionError(f"{name} went through ctypes")


def layer(q, block):
    """name -> (arguments with outputs of their own, the outputs) of the eight calls on one small layer"""
    t, i, o = (512, 256, 256) if block == 256 else (288, 320, 352)
    gen = torch.Generator(device="cuda").manual_seed(block)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    x, w, dy = rand(t, i), rand(o, i), rand(t, o)
    xq, wq = buffers(q, t, i), buffers(q, o, i)
    q.check(q.quartet_linear_fwd_block(x, w, t, i, o, block, torch.empty((t, o), device="cuda"), 0, *xq, *wq))
    ws_bytes = q.quartet_linear_workspace_bytes_block(t, i, o, block)
    f32 = lambda *s: torch.zeros(s, device="cuda")

    def make():
        y, dx, dw, cx, cw, cg, ws = f32(t, o), f32(t, i), f32(o, i), buffers(q, t, i), buffers(q, o, i), buffers(q, t, o), torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda")
        both = (*xq, *wq)
        calls = {"quartet_quant_fwd": ((x, t, i, i, False, *cx), cx),
                 "quartet_quant_bwd_sr": ((dy, t, o, o, 0, q.quartet_sign_word(9), 2 ** 64 - 9, 3, 0, *cg[:2]), cg[:2]),
                 "quartet_mxfp4_gemm": ((*xq[:2], *wq[:2], t, o, i, 0.75, y, 0, o), (y,)),
                 "quartet_mxfp4_gemm_grad": ((*xq[:2], *wq[:2], t, o, i, None, 1.5, y, 0, o), (y,)),
                 "quartet_linear_fwd": ((x, w, t, i, o, y, 0, *cx, *cw), (y, *cx, *cw)),
                 "quartet_linear_bwd": ((dy, t, i, o, *both, 2 ** 63 + 5, 0, dx, dw, 0, ws, ws_bytes), (dx, dw)),
                 "quartet_linear_fwd_block": ((x, w, t, i, o, block, y, 0, *cx, *cw), (y, *cx, *cw)),
                 "quartet_linear_bwd_block": ((dy, t, i, o, block, *both, 7, 1, dx, dw, 0, ws, ws_bytes), (dx, dw))}
        return calls
    return make


NAMES = ("quartet_quant_fwd", "quartet_quant_bwd_sr", "quartet_mxfp4_gemm", "quartet_mxfp4_gemm_grad", "quartet_linear_fwd", "quartet_linear_bwd",
         "quartet_linear_fwd_block", "quartet_linear_bwd_block")


@pytest.mark.parametrize("block", [32, 256])
@pytest.mark.parametrize("name", NAMES)
def test_both_conversions_give_the_same(q, monkeypatch, name, block):
    make, call = layer(q, block), getattr(q, name)
    (args, native), (cargs, ctyped) = make()[name], make()[name]
    with monkeypatch.context() as m:
        m.setattr(q, "_lib", NoCtypes())
        assert call(*args) == q.QUARTET_OK
    with monkeypatch.context() as m:
        m.setattr(q, "_native", None)
        assert call(*cargs) == q.QUARTET_OK
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) and bool(a.any()) for a, b in zip(native, ctyped))
    # one argument at a time that is refused: the same refusal, before anything has run
    for n, arg in enumerate(args):
        worse = [None, "x", 1.5j] if not isinstance(arg, torch.Tensor) else [arg.cpu(), arg.reshape(1, -1).expand(2, -1), "x"]
        for bad in worse:
            if bad is None and arg is None:
                continue
            outcome = []
            for conversion in (q._native, None):
                with monkeypatch.context() as m:
                    m.setattr(q, "_native", conversion)
                    try:
                        outcome.append(call(*args[:n], bad, *args[n + 1:]))
                    except Exception as e:
                        outcome.append((type(e), str(e)))
            assert outcome[0] == outcome[1] and outcome[0] != q.QUARTET_OK, (name, n, bad if not isinstance(bad, torch.Tensor) else bad.shape)


def test_current_stream_of_each_thread(q, monkeypatch):
    # On each thread's stream: a delay, the thread's own values into its input, the call, a copy of the result.  A launch on any other
    # stream would not wait for the values.
    rows, k, threads = 512, 1024, 4
    data = [torch.randn((rows, k), device="cuda").to(torch.bfloat16) for _ in range(threads)]
    want, results, errors = [buffers(q, rows, k) for _ in data], [None] * threads, []
    for x, out in zip(data, want):
        q.check(q.quartet_quant_fwd(x, rows, k, k, 0, *out))
    inputs, outputs, streams = [torch.zeros_like(x) for x in data], [buffers(q, rows, k) for _ in data], [torch.cuda.Stream() for _ in data]
    torch.cuda.synchronize()
    monkeypatch.setattr(q, "_lib", NoCtypes())

    def work(n):
        try:
            with torch.cuda.stream(streams[n]):
                torch.cuda._sleep(4_000_000)               # 2 to 40 ms
                inputs[n].copy_(data[n])
                q.check(q.quartet_quant_fwd(inputs[n], rows, k, k, 0, *outputs[n]))
                results[n] = [t.clone() for t in outputs[n]]
                streams[n].synchronize()
        except Exception as e:
            errors.append(e)

    workers = [threading.Thread(target=work, args=(n,)) for n in range(threads)]
    for t in workers:
        t.start()
    for t in workers:
        t.join()
    assert not errors
    assert all(torch.equal(a, b) for got, ref in zip(results, want) for a, b in zip(got, ref))
