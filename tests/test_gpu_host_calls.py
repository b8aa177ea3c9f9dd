"""The binding's host code: what it takes it answers as the Python code behind it does, and what it does not take is refused as before."""
import numpy as np
import pytest

import synthetic_inputs as syn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch

    from tests import gpu_util as gpu
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    layer = syn.make_layer(96, 1024, seed=(970, 0))
    return gpu, gpu.DeviceLayer(layer), gpu.to_dev(syn.make_x(5, 1024, seed=(970, 1)))


@pytest.fixture
def python_only(monkeypatch):
    """The Python code alone: the host code declines every call."""
    from paper_2510_10467_amd import binding
    binding.lib()

    class Declines:
        gemv = gemv_multi = gemm_mixed = staticmethod(lambda *a: None)

    def switch(on):
        monkeypatch.setattr(binding, "_host", Declines if on else original)
    original = binding._host
    yield switch
    switch(False)


def _calls(torch, bcq, dl, x):
    z = {q: torch.randn(96, 8, device="cuda").half() for q in (2, 3)}
    p_req = torch.tensor([1, 2, 3, 4, 2], dtype=torch.int32, device="cuda")
    y = torch.empty((5, 96), dtype=torch.float16, device="cuda")
    return [lambda: bcq.bcq_gemv(dl.planes, dl.scales[3], 3, x),
            lambda: bcq.bcq_gemv(dl.planes, dl.scales[3], 3, x, y=y),
            lambda: bcq.bcq_gemv(dl.planes, dl.scales[2], 2, x, offsets=z[2]),
            lambda: bcq.bcq_gemv(dl.planes, dl.scales[2], np.int64(2), x),                  # not a plain int: the Python way
            lambda: bcq.bcq_gemv(torch.nn.Parameter(dl.planes, requires_grad=False), dl.scales[2], 2, x),
            lambda: torch.cat(bcq.bcq_gemv_multi([dl.planes, dl.planes], [dl.scales[4], dl.scales[4]], 4, x)),
            lambda: torch.cat(bcq.bcq_gemv_multi((dl.planes,), (dl.scales[1],), 1, x, ys=[y])),
            lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req, x),
            lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req, x, y=y, offsets_by_p={}),
            lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req, x, offsets_by_p=z),
            lambda: bcq.bcq_gemv(dl.planes, dl.scales[3], 3, x[:0])]


def _refused(torch, bcq, dl, x):
    s, p_req = dl.scales[2], torch.full((5,), 2, dtype=torch.int32, device="cuda")
    wide = torch.zeros((5, 2048), dtype=torch.float16, device="cuda")
    return [lambda: bcq.bcq_gemv(dl.planes, s, 2, x.cpu()),
            lambda: bcq.bcq_gemv(dl.planes, s, 2, x.float()),
            lambda: bcq.bcq_gemv(dl.planes, s, 2, wide[:, ::2]),                            # a stride
            lambda: bcq.bcq_gemv(dl.planes, s, 2, wide),
            lambda: bcq.bcq_gemv(dl.planes, s, 3, x),
            lambda: bcq.bcq_gemv(dl.planes[:1], s, 2, x),
            lambda: bcq.bcq_gemv(dl.planes, s, 2, x, y=torch.empty((5, 95), dtype=torch.float16, device="cuda")),
            lambda: bcq.bcq_gemv(dl.planes, s, 2, x, offsets=torch.zeros((96, 9), dtype=torch.float16, device="cuda")),
            lambda: bcq.bcq_gemv(dl.planes, s, 2, x, group=0),
            lambda: bcq.bcq_gemv(dl.planes, s[:0], 0, x),                                   # a precision that the library refuses
            lambda: bcq.bcq_gemv(dl.planes, s, 2, wide.view(-1)[1:1 + 5 * 1024].view(5, 1024)),     # not aligned
            lambda: bcq.bcq_gemv_multi([dl.planes], [s, s], 2, x),
            lambda: bcq.bcq_gemv_multi([dl.planes] * 5, [s] * 5, 2, x),
            lambda: bcq.bcq_gemv_multi([], [], 2, x),
            lambda: bcq.bcq_gemm_mixed(dl.planes, {5: s}, p_req, x),
            lambda: bcq.bcq_gemm_mixed(dl.planes, {}, p_req, x),
            lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req[:4], x),
            lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req.long(), x)]


def test_the_same_answers_and_the_same_refusals(setup, python_only):
    import torch

    import paper_2510_10467_amd as bcq
    gpu, dl, x = setup

    def outcome(call):
        try:
            return call().clone()
        except Exception as e:                  # noqa: BLE001  (whatever it is: it has to be the same)
            return type(e), str(e)
    for made, some_answer in ((_calls, True), (_refused, False)):
        for k, call in enumerate(made(torch, bcq, dl, x)):
            python_only(True)
            expected = outcome(call)
            python_only(False)
            got = outcome(call)
            if isinstance(expected, torch.Tensor):
                assert some_answer and torch.equal(got, expected) and got.dtype == expected.dtype, (made.__name__, k)
            else:
                assert got == expected, (made.__name__, k, got, expected)
            assert some_answer == isinstance(expected, torch.Tensor) or made is _calls, (made.__name__, k, expected)


def test_current_stream_and_threads(setup):
    """Launches go to the calling thread's current stream; several threads call at once."""
    import threading

    import torch

    import paper_2510_10467_amd as bcq
    gpu, dl, x = setup
    want = bcq.bcq_gemv(dl.planes, dl.scales[4], 4, x)
    got = [None] * 4

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(50):
                y = bcq.bcq_gemv(dl.planes, dl.scales[4], 4, x)
            torch.cuda.current_stream().synchronize()
            got[k] = y
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(torch.equal(y, want) for y in got)
    # recorded on the capturing stream
    y = torch.zeros_like(want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bcq.bcq_gemv(dl.planes, dl.scales[4], 4, x, y=y)
    assert not y.any()
    for _ in range(2):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
