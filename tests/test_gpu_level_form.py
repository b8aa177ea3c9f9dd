"""The two forms of the large-batch kernel against each other and bit for bit against the definition: the level form (weights by
look-up, codes 100 .. 105 of the forced shapes) and the summing form, on shapes that the automatic choice would give to either."""
import numpy as np
import pytest

import synthetic_inputs as syn

pytestmark = pytest.mark.gpu

SHAPES = [(1, 100), (1, 101), (1, 102), (1, 103), (1, 104), (1, 105), (1, 4), (4, 8)]       # the last two: the summing form


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from tests import gpu_util
    return gpu_util


@pytest.fixture
def force():
    import paper_2510_10467_amd as bcq

    def forced(shape):
        print(f"shape {shape}", flush=True)
        bcq.select_kernel("dequant_mfma")
        bcq.select_dequant_shape(*shape)
    yield forced
    bcq.select_dequant_shape(0, 0)
    bcq.select_kernel("auto")


def weights16(layer, p, group, offsets):
    """W_p: z + (+-alpha_1) + ... in float32, plane by plane, rounded once to binary16."""
    bits = np.unpackbits(layer.planes.view(np.uint8), axis=-1, bitorder="little").astype(bool)
    w = np.zeros((layer.m, layer.n), dtype=np.float32)
    if offsets is not None:
        w += np.repeat(offsets.astype(np.float32), group, axis=1)
    for i in range(p):
        a = np.repeat(layer.scales[p][i].astype(np.float32), group, axis=1)
        w = w + np.where(bits[i], a, -a)
    return w.astype(np.float16)


@pytest.mark.parametrize("n,group", [(512, 64), (512, 128), (768, 256)])
@pytest.mark.parametrize("with_offsets", [False, True])
def test_every_weight_bit_for_bit(gpu, force, n, group, with_offsets):
    """One-hot activations read every weight of two and three pairs of column groups: a wrong byte of a look-up, a swapped column or a
    second rounding shows, where the tolerance of a whole product would hide it.  300 rows: a ragged last tile in every shape."""
    import paper_2510_10467_amd as bcq
    m = 300
    layer = syn.make_layer(m, n, group=group, seed=(950, n, group), signed=True)
    dl = gpu.DeviceLayer(layer)
    x = gpu.to_dev(np.eye(n, dtype=np.float16))
    for p in (1, 2, 3, 4):
        z = syn.make_offsets(p, m, n, group, seed=(951, n, p)) if with_offsets else None
        expected = weights16(layer, p, group, z).T.view(np.uint16)
        for shape in SHAPES:
            force(shape)
            y = bcq.bcq_gemv(dl.planes, dl.scales[p], p, x, group=group, offsets=None if z is None else gpu.to_dev(z))
            got = (y + 0.0).cpu().numpy().view(np.uint16)           # (-0 and +0 are the same weight)
            wrong = np.argwhere(got != (expected.view(np.float16) + np.float16(0)).view(np.uint16))
            assert wrong.size == 0, f"shape {shape} p={p}: {len(wrong)} weights differ, first [column, row] {wrong[0]}"


@pytest.mark.parametrize("n,group", [(256, 256), (2304, 256), (1280, 128), (4352, 64), (4352, 128)])
@pytest.mark.parametrize("with_offsets", [False, True])
def test_every_weight_over_several_windows_of_scales(gpu, force, n, group, with_offsets):
    """Widths of 1, 5, 9 and 17 pairs of column groups: a last block of one pair, teams without one, windows of scales that end in the
    middle of a row; 67 rows, so that in groups of 256 rows and planes of scales start at odd multiples of two bytes."""
    import paper_2510_10467_amd as bcq
    m = 67
    layer = syn.make_layer(m, n, group=group, seed=(956, n, group), signed=True)
    dl = gpu.DeviceLayer(layer)
    x = gpu.to_dev(np.eye(n, dtype=np.float16))
    for p in (1, 2, 3, 4):
        z = syn.make_offsets(p, m, n, group, seed=(957, n, p)) if with_offsets else None
        z_dev = None if z is None else gpu.to_dev(z)
        expected = (weights16(layer, p, group, z).T + np.float16(0)).view(np.uint16)
        for shape in SHAPES[:6]:
            force(shape)
            y = bcq.bcq_gemv(dl.planes, dl.scales[p], p, x, group=group, offsets=z_dev)
            wrong = np.argwhere((y + 0.0).cpu().numpy().view(np.uint16) != expected)
            assert wrong.size == 0, f"shape {shape} p={p}: {len(wrong)} weights differ, first [column, row] {wrong[0]}"


@pytest.mark.parametrize("n,group", [(256, 64), (256, 128), (512, 256), (768, 64), (1792, 256)])
@pytest.mark.parametrize("with_offsets", [False, True])
def test_every_weight_on_narrow_matrices(gpu, force, n, group, with_offsets):
    """Rows whose scales take less than a window: 4, 8, 16 (an odd start, 14 bytes) and 32 bytes of LDS per row and plane; 131 rows, so that a
    plane of scales starts at an odd multiple of two bytes in groups of 256, and a workgroup's last rows are not there."""
    import paper_2510_10467_amd as bcq
    m = 131
    layer = syn.make_layer(m, n, group=group, seed=(958, n, group), signed=True)
    dl = gpu.DeviceLayer(layer)
    x = gpu.to_dev(np.eye(n, dtype=np.float16))
    for p in (1, 2, 3, 4):
        z = syn.make_offsets(p, m, n, group, seed=(959, n, p)) if with_offsets else None
        z_dev = None if z is None else gpu.to_dev(z)
        expected = (weights16(layer, p, group, z).T + np.float16(0)).view(np.uint16)
        for shape in SHAPES[:6]:
            force(shape)
            y = bcq.bcq_gemv(dl.planes, dl.scales[p], p, x, group=group, offsets=z_dev)
            wrong = np.argwhere((y + 0.0).cpu().numpy().view(np.uint16) != expected)
            assert wrong.size == 0, f"shape {shape} p={p}: {len(wrong)} weights differ, first [column, row] {wrong[0]}"


@pytest.mark.parametrize("n,group", [(5376, 128), (6400, 64)])
@pytest.mark.parametrize("with_offsets", [False, True])
def test_every_weight_where_tiles_of_64_rows_take_words_for_two_pairs(gpu, force, n, group, with_offsets):
    """Beyond 5120 columns: 21 and 25 pairs, whole blocks for every team and then one pair, five or one."""
    import paper_2510_10467_amd as bcq
    m = 67
    layer = syn.make_layer(m, n, group=group, seed=(976, n, group), signed=True)
    dl = gpu.DeviceLayer(layer)
    x = gpu.to_dev(np.eye(n, dtype=np.float16))
    for p in (1, 2, 3, 4):
        z = syn.make_offsets(p, m, n, group, seed=(977, n, p)) if with_offsets else None
        z_dev = None if z is None else gpu.to_dev(z)
        expected = (weights16(layer, p, group, z).T + np.float16(0)).view(np.uint16)
        for shape in ((1, 103), (1, 105)):
            force(shape)
            y = bcq.bcq_gemv(dl.planes, dl.scales[p], p, x, group=group, offsets=z_dev)
            wrong = np.argwhere((y + 0.0).cpu().numpy().view(np.uint16) != expected)
            assert wrong.size == 0, f"shape {shape} p={p}: {len(wrong)} weights differ, first [column, row] {wrong[0]}"


@pytest.mark.parametrize("shape", SHAPES)
def test_products_that_are_exact(gpu, force, shape):
    """Scales of 1, 1/4, 1/16, 1/64 and whole activations up to 8: every partial sum is a multiple of 1/64 below 2^14 and therefore
    exact in float32, so each result is the exact one rounded once to binary16, whatever the order.  Planes from p on are
    not read, and the same call gives the same bits on ordinary inputs too."""
    import torch

    import paper_2510_10467_amd as bcq
    m, n, batch = 290, 1280, 70
    layer = syn.make_layer(m, n, seed=(952, 0), signed=True)
    dl = gpu.DeviceLayer(layer)
    whole = np.random.default_rng([syn.BASE_SEED, 952]).integers(-8, 9, size=(batch, n)).astype(np.float16)
    x = gpu.to_dev(syn.make_x(batch, n, seed=(952, 1)))
    force(shape)
    for p in (1, 2, 3, 4):
        powers = np.repeat(np.array([1, 0.25, 0.0625, 0.015625], dtype=np.float16)[:p], m * n // 128).reshape(p, m, n // 128)
        exact = whole.astype(np.float64) @ weights16(syn.BcqLayer(m, n, 128, layer.planes, {p: powers}), p, 128, None).astype(np.float64).T
        y = bcq.bcq_gemv(dl.planes, gpu.to_dev(powers), p, gpu.to_dev(whole)).cpu().numpy()
        assert np.array_equal(y, exact.astype(np.float16)), f"shape {shape} p={p}"
        other = dl.planes.clone()
        other[p:] = ~other[p:]
        y = bcq.bcq_gemv(dl.planes, dl.scales[p], p, x)
        assert torch.equal(y, bcq.bcq_gemv(dl.planes, dl.scales[p], p, x)), f"shape {shape} p={p}: not deterministic"
        assert torch.equal(y, bcq.bcq_gemv(other, dl.scales[p], p, x)), f"shape {shape} p={p}: planes >= p influenced the result"


PER_REQUEST = [(1, 96), (1, 101), (1, 102), (1, 103), (1, 104), (1, 105)]         # the first: 128 x 96, of these calls only


@pytest.mark.parametrize("shape", PER_REQUEST + [(0, 0)])
@pytest.mark.parametrize("m,n,batch,group", [(150, 1280, 33, 128), (70, 768, 129, 64), (259, 1536, 300, 256)])
def test_per_request_precision(gpu, force, shape, m, n, batch, group):
    """The form per precision, its requests wherever they sit in the batch: with offsets for some precisions and without, a precision without
    a scale set (zeros), precisions out of range (clamped), all requests at one precision, a ragged last tile of rows and of requests."""
    layer = syn.make_layer(m, n, group=group, seed=(960, m, n), signed=True)
    dl = gpu.DeviceLayer(layer)
    x = syn.make_x(batch, n, seed=(961, batch))
    p_req = syn.make_p_req(batch, 1, 4, seed=(962, batch))
    some = {q: syn.make_offsets(q, m, n, group, seed=(963, q)) for q in (2, 4)}
    import paper_2510_10467_amd as bcq
    force(shape)
    assert shape == (0, 0) or bcq.mixed_shape_for((1, 2, 3, 4), m, n, batch, group) == shape
    for req in (p_req, np.full(batch, 3, dtype=np.int32)):
        for z in (None, some):
            force(shape)
            used, _ = gpu.check_mixed(dl, req, x, "dequant_mfma", group, offsets_by_p=z)
            assert used == "dequant_mfma"
    force(shape)
    x_dev = gpu.to_dev(x)
    y = bcq.bcq_gemm_mixed(dl.planes, dl.scales, gpu.to_dev(p_req), x_dev, group=group).cpu().numpy()
    outside = np.where(p_req == 1, -3, np.where(p_req == 4, 9, p_req)).astype(np.int32)
    assert np.array_equal(y, bcq.bcq_gemm_mixed(dl.planes, dl.scales, gpu.to_dev(outside), x_dev, group=group).cpu().numpy())
    del dl.scales[2]
    z = bcq.bcq_gemm_mixed(dl.planes, dl.scales, gpu.to_dev(p_req), x_dev, group=group).cpu().numpy()
    assert not z[p_req == 2].any() and np.array_equal(z[p_req != 2], y[p_req != 2])


@pytest.mark.parametrize("shape", PER_REQUEST)
@pytest.mark.parametrize("group", [64, 128, 256])
def test_every_weight_with_per_request_precision(gpu, force, group, shape):
    """One-hot activations of 4352 requests, each at a precision of its own, over 17 pairs of column groups: blocks of two pairs and a single one after
    them, windows of scales that are loaded again, tiles of ranks that precisions leave ragged; offsets for two of the four precisions."""
    import paper_2510_10467_amd as bcq
    m, n = 67, 4352
    layer = syn.make_layer(m, n, group=group, seed=(971, n, group), signed=True)
    dl = gpu.DeviceLayer(layer)
    x = gpu.to_dev(np.eye(n, dtype=np.float16))
    p_req = syn.make_p_req(n, 1, 4, seed=(972, n))
    some = {q: syn.make_offsets(q, m, n, group, seed=(973, q)) for q in (2, 4)}
    force(shape)
    assert bcq.mixed_shape_for((1, 2, 3, 4), m, n, n, group) == shape
    for z in ({}, some):
        w = {q: weights16(layer, q, group, z.get(q)) for q in (1, 2, 3, 4)}
        expected = np.stack([w[q][:, b] for b, q in enumerate(p_req)]) + np.float16(0)
        y = bcq.bcq_gemm_mixed(dl.planes, dl.scales, gpu.to_dev(p_req), x, group=group, offsets_by_p={q: gpu.to_dev(o) for q, o in z.items()})
        assert bcq.last_kernel() == "dequant_mfma"
        wrong = np.argwhere((y + 0.0).cpu().numpy().view(np.uint16) != expected.view(np.uint16))
        assert wrong.size == 0, f"{len(wrong)} weights differ, first [column, row] {wrong[0]} at precision {p_req[wrong[0][0]]}"


def test_per_request_precision_on_tiles_of_96(gpu, oracle):
    """Sizes that the automatic choice gives 128 rows x 96 requests; capture in a graph and replays give what the call gives."""
    import torch

    import paper_2510_10467_amd as bcq
    m, n, batch = 6000, 4352, 255
    assert bcq.mixed_shape_for((2, 3, 4), m, n, batch) == (1, 96)
    layer = syn.make_layer(m, n, seed=(964, m), precisions=[2, 3, 4], signed=True)
    dl = gpu.DeviceLayer(layer)
    x = syn.make_x(batch, n, seed=(964, batch))
    p_req = syn.make_p_req(batch, 2, 4, seed=(964, 0))
    x_dev, r_dev = gpu.to_dev(x), gpu.to_dev(p_req)
    out = gpu.Guarded((batch, m))
    eager = bcq.bcq_gemm_mixed(dl.planes, dl.scales, r_dev, x_dev, y=out.t)
    assert bcq.last_kernel() == "dequant_mfma"
    out.check("tiles of 96")
    rows = np.unique(np.concatenate([[0, 127, 128, m - 1], np.random.default_rng([syn.BASE_SEED, 974]).integers(0, m, size=60)]))
    y_ref, a_ref = oracle.gemm_mixed(np.ascontiguousarray(layer.planes[:, rows, :]), {q: np.ascontiguousarray(t[:, rows, :]) for q, t in layer.scales.items()},
                                     p_req, x)
    gpu.assert_within_tolerance(eager[:, rows], y_ref, a_ref, "tiles of 96")
    y = torch.empty_like(eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bcq.bcq_gemm_mixed(dl.planes, dl.scales, r_dev, x_dev, y=y)
    for other in (p_req, np.roll(p_req, 7), np.full(batch, 4, dtype=np.int32)):
        r_dev.copy_(gpu.to_dev(other))
        y.fill_(0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, bcq.bcq_gemm_mixed(dl.planes, dl.scales, r_dev, x_dev))


@pytest.mark.parametrize("group", [64, 256])
@pytest.mark.parametrize("shape", [(1, 2), (2, 4), (4, 40), (2, 8)])
def test_summing_form_where_the_level_form_is_the_default(gpu, force, group, shape):
    """Groups of 64 and 256 with and without offsets, of which the automatic choice leaves the summing form little above 32 requests."""
    m, n, batch = 150, 1536, 70
    layer = syn.make_layer(m, n, group=group, seed=(953, group), signed=True)
    dl = gpu.DeviceLayer(layer)
    x = syn.make_x(batch, n, seed=(953, 1))
    force(shape)
    for p in (1, 2, 3, 4):
        for z in (None, syn.make_offsets(p, m, n, group, seed=(954, p))):
            gpu.check_gemv(dl, p, x, "dequant_mfma", group, offsets=z)


def test_both_forms_at_the_limit_of_32_bit_offsets(gpu, oracle, force):
    """Two planes of just under 2 GiB, past 2^31 bytes in 32-bit offsets: sampled rows of either form against the oracle."""
    import paper_2510_10467_amd as bcq
    m, n, p, batch = 262144 - 11, 65536, 2, 80
    layer = syn.make_layer(m, n, p_max=p, seed=(280, m, p), precisions=[p], signed=True)
    dl = gpu.DeviceLayer(layer)
    x = syn.make_x(batch, n, seed=(280, batch))
    rows = np.unique(np.concatenate([[0, 31, 32, 131071, 131072, m - 65, m - 33, m - 32, m - 1],
                                     np.random.default_rng([syn.BASE_SEED, 955]).integers(0, m, size=40)]))
    y_ref, a_ref = oracle.gemv(np.ascontiguousarray(layer.planes[:, rows, :]), np.ascontiguousarray(layer.scales[p][:, rows, :]), x)
    for shape in ((1, 105), (1, 101), (1, 4)):
        force(shape)
        out = gpu.Guarded((batch, m))
        bcq.bcq_gemv(dl.planes, dl.scales[p], p, gpu.to_dev(x), y=out.t)
        y = out.check(f"shape {shape}")
        gpu.assert_within_tolerance(y[:, rows], y_ref, a_ref, f"shape {shape}")
