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
    """switch(True): the Python code alone, the host code declines every call.  switch(False): the host code as it is; returns the list to which
    every call to it that ends without an error adds whether it made the call."""
    from paper_2510_10467_amd import binding
    binding.lib()
    original = binding._host
    assert original.__name__.endswith("_bcq_host"), "the host code is not loaded"

    class Declines:
        gemv = gemv_multi = gemm_mixed = staticmethod(lambda *a: None)

    def recording(name, made):
        def call(*args):
            done = getattr(original, name)(*args)
            made.append(done is not None)
            return done
        return staticmethod(call)

    def switch(on):
        made = []
        watched = type("Recording", (), {name: recording(name, made) for name in ("gemv", "gemv_multi", "gemm_mixed")})
        monkeypatch.setattr(binding, "_host", Declines if on else watched)
        return made
    yield switch
    monkeypatch.setattr(binding, "_host", original)


def _calls(torch, bcq, dl, x):
    """(the host code makes it, call)"""
    z = {q: torch.randn(96, 8, device="cuda").half() for q in (2, 3)}
    p_req = torch.tensor([1, 2, 3, 4, 2], dtype=torch.int32, device="cuda")
    y = torch.empty((5, 96), dtype=torch.float16, device="cuda")
    return [(True, lambda: bcq.bcq_gemv(dl.planes, dl.scales[3], 3, x)),
            (True, lambda: bcq.bcq_gemv(dl.planes, dl.scales[3], 3, x, y=y)),
            (True, lambda: bcq.bcq_gemv(dl.planes, dl.scales[2], 2, x, offsets=z[2])),
            (False, lambda: bcq.bcq_gemv(dl.planes, dl.scales[2], np.int64(2), x)),         # not a plain int: the Python way
            (True, lambda: bcq.bcq_gemv(torch.nn.Parameter(dl.planes, requires_grad=False), dl.scales[2], 2, x)),
            (True, lambda: torch.cat(bcq.bcq_gemv_multi([dl.planes, dl.planes], [dl.scales[4], dl.scales[4]], 4, x))),
            (False, lambda: torch.cat(bcq.bcq_gemv_multi((dl.planes,), (dl.scales[1],), 1, x))),        # tuples
            (None, lambda: torch.cat(bcq.bcq_gemv_multi([dl.planes], [dl.scales[1]], 1, x, ys=[y]))),   # results of the caller's: not asked
            (True, lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req, x)),
            (True, lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req, x, y=y, offsets_by_p={})),
            (True, lambda: bcq.bcq_gemm_mixed(dl.planes, dl.scales, p_req, x, offsets_by_p=z))]


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
            lambda: bcq.bcq_gemv(dl.planes, s, 2, x[:0]),                                   # no requests: no pointer to their activations
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
    for k, (natively, call) in enumerate(_calls(torch, bcq, dl, x)):
        python_only(True)
        expected = call().clone()
        made = python_only(False)
        got = call().clone()
        assert torch.equal(got, expected) and got.dtype == expected.dtype, k
        assert made == ([] if natively is None else [natively]), f"call {k}: the host code made it: {made}"
    for k, call in enumerate(_refused(torch, bcq, dl, x)):
        python_only(True)
        expected = outcome(call)
        made = python_only(False)
        got = outcome(call)
        assert not isinstance(expected, torch.Tensor) and got == expected, (k, got, expected)
        assert True not in made, k              # (the host code answers with a result, the library's own refusal, or not at all)


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
