"""The work that is timed: what a serving process and an offline quantiser ask of this library.

A case is one call of the Python binding, or the calls that the linear layers of decoder blocks take:

  product   one ``bcq_gemv`` (with ``offsets``: the asymmetric scheme), or one ``bcq_gemm_mixed`` where ``p`` is 0
            (every request at a precision of its own, drawn from ``p_low`` .. 4)
  blocks    the linear layers of ``layers`` decoder blocks at one precision: q, k and v in one ``bcq_gemv_multi``, o,
            gate and up in one ``bcq_gemv_multi``, down; in the asymmetric scheme, which the several-matrices call does
            not have, seven ``bcq_gemv`` calls.  With ``graph`` the calls are recorded once in a HIP graph, as a
            decoding loop does that repeats the same launches for every token, and a pass is one replay
  quantize  one ``bcq_quantize`` (Algorithm 1) of a full-precision matrix

Layer sizes are those of the Llama-3-8B, Phi-4-14B and Llama-3-70B linear layers that the benchmark and the tests use.
The distributions are those of ``synthetic_inputs.py``, drawn on the GPU: fair bits, a scale set per precision whose
scales halve from plane to plane, normal activations, weights with a spread per row and a few large entries.
"""
import math

import torch

import paper_2510_10467_amd as bcq

P_MAX = 4
# hidden size, rows of the k and v projections, rows of the gate and up projections
DIMS = {"llama3_8b": (4096, 1024, 14336), "phi4_14b": (5120, 1280, 17920), "llama3_70b": (8192, 1024, 28672)}
MOST_FLOPS = 2.0 * 28672 * 8192 * 2048          # the largest listed case
MOST_QUANTIZED = 4096 * 4096 * 20 * 3           # weights x cycles x stages of the largest quantiser case


def _product(m, n, batch, p, group=128, offsets=False, p_low=2):
    return {"kind": "product", "m": m, "n": n, "batch": batch, "p": p, "p_low": p_low, "group": group, "offsets": offsets}


def _blocks(dims, layers, batch, p, graph=False, offsets=False):
    return {"kind": "blocks", "dims": dims, "layers": layers, "batch": batch, "p": p, "graph": graph, "offsets": offsets}


def _quantize(m, n, p_low, p_high, cycles, group=128, offsets=False):
    return {"kind": "quantize", "m": m, "n": n, "p_low": p_low, "p_high": p_high, "cycles": cycles, "group": group, "offsets": offsets}


def listed():
    return [
        # one token, the smallest projection on its own, called from Python: launch and host latency
        dict(_product(1024, 4096, 1, 2), name="gemv_kv_1"),
        # one token through four decoder blocks, the decoding loop of a single user
        dict(_blocks("llama3_8b", 4, 1, 4, graph=True), name="decode_8b_1_graph"),
        # the same for a program that calls layer by layer, under the asymmetric scheme the models are quantised with
        dict(_blocks("phi4_14b", 1, 1, 3, offsets=True), name="decode_phi4_1_asym"),
        # a handful of users at low precision, called from Python
        dict(_blocks("llama3_8b", 1, 4, 2), name="decode_8b_4"),
        # a server's decoding batch
        dict(_blocks("llama3_8b", 2, 16, 4, graph=True), name="decode_8b_16_graph"),
        # a decoding batch whose users each chose a precision
        dict(_product(14336, 4096, 13, 0), name="mixed_13"),
        # a width and a row count that no tile divides
        dict(_product(3000, 4224, 24, 3), name="ragged_24"),
        # the finer group size, a large decoding batch
        dict(_product(8192, 8192, 96, 4, group=64), name="group64_96"),
        # a large batch with a precision per user
        dict(_product(8192, 8192, 200, 0), name="mixed_200"),
        # a prompt through one decoder block
        dict(_blocks("llama3_8b", 1, 500, 4), name="prefill_8b_500"),
        # a long prompt on the largest layer
        dict(_product(28672, 8192, 2048, 3), name="prefill_70b_2048"),
        # offline: full-precision weights to planes and the scale sets of 2, 3 and 4 bits
        dict(_quantize(4096, 4096, 2, 4, 20), name="quantize_4096"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("product", "product", "product", "blocks", "blocks", "mixed", "mixed", "quantize"))
    if kind == "quantize":
        group = rng.choice((32, 64, 128, 128, 256))
        n = 256 * _log_uniform(rng, 4, 32)
        p_low = rng.choice((1, 2, 2))
        p_high = rng.choice((3, 4, 4))
        cycles = rng.randint(5, 20)
        m = min(_log_uniform(rng, 256, 8192), MOST_QUANTIZED // (n * cycles * 4))
        return _quantize(m, n, p_low, p_high, cycles, group, rng.random() < 0.3)
    if kind == "blocks":
        dims = rng.choice(sorted(DIMS))
        batch = _log_uniform(rng, 1, 512)
        asym = rng.random() < 0.2
        return _blocks(dims, 1 if batch > 16 else rng.randint(1, 3), batch, rng.choice((2, 3, 4)), graph=batch <= 64 and rng.random() < 0.6,
                       offsets=asym)
    m = _log_uniform(rng, 1024, 28672)
    if rng.random() < 0.6:
        m = -(-m // 256) * 256
    n = 128 * _log_uniform(rng, 8, 224)
    if rng.random() < 0.7:
        n = -(-n // 1024) * 1024
    group = rng.choice((64, 128, 128, 128, 256)) if n % 256 == 0 else rng.choice((64, 128, 128))
    batch = _log_uniform(rng, 1, 2048 if kind == "product" else 512)
    batch = max(1, min(batch, int(MOST_FLOPS // (2.0 * m * n))))
    if kind == "mixed":
        return _product(m, n, max(2, batch), 0, group, rng.random() < 0.2, rng.choice((1, 2, 2)))
    return _product(m, n, batch, rng.choice((2, 3, 4)), group, rng.random() < 0.2)


def _planes(m, n, gen):
    return torch.randint(-2 ** 31, 2 ** 31, (P_MAX, m, n // 32), dtype=torch.int32, device="cuda", generator=gen)


def _scales(p, m, n, group, gen):
    rows = [(torch.randn((m, n // group), device="cuda", generator=gen) * 0.02).abs()]
    for _ in range(1, p):
        rows.append(rows[-1] * (0.4 + 0.2 * torch.rand((m, n // group), device="cuda", generator=gen)))
    return torch.stack(rows).half().contiguous()


def _offsets(m, n, group, gen):
    return (torch.randn((m, n // group), device="cuda", generator=gen) * 0.01).half()


def _x(batch, n, gen):
    return torch.randn((batch, n), device="cuda", generator=gen).half()


def _block_rows(case):
    """The linear layers of one block: (rows of the matrices that share an input, width of the input)."""
    hidden, kv, ffn = DIMS[case["dims"]]
    return [([hidden, kv, kv], hidden), ([hidden], hidden), ([ffn, ffn], hidden), ([hidden], ffn)]


def _run_blocks(s):
    case, out = s["case"], []
    for stage in s["stages"]:
        if case["offsets"]:
            out += [bcq.bcq_gemv(w, a, case["p"], stage["x"], offsets=z) for w, a, z in zip(stage["planes"], stage["scales"], stage["offsets"])]
        elif len(stage["planes"]) > 1:
            out += bcq.bcq_gemv_multi(stage["planes"], stage["scales"], case["p"], stage["x"])
        else:
            out.append(bcq.bcq_gemv(stage["planes"][0], stage["scales"][0], case["p"], stage["x"]))
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = {"case": case}
    if case["kind"] == "quantize":
        m, n = case["m"], case["n"]
        sigma = 0.02 * torch.exp(0.25 * torch.randn((m, 1), device="cuda", generator=gen))
        w = torch.randn((m, n), device="cuda", generator=gen) * sigma
        s["w"] = torch.where(torch.rand((m, n), device="cuda", generator=gen) < 1.0 / 256.0, 6.0 * w, w).half()
        return s
    if case["kind"] == "blocks":
        p = case["p"]
        s["stages"] = []
        for _ in range(case["layers"]):
            for rows, n in _block_rows(case):
                s["stages"].append({"x": _x(case["batch"], n, gen), "planes": [_planes(m, n, gen) for m in rows],
                                    "scales": [_scales(p, m, n, 128, gen) for m in rows],
                                    "offsets": [_offsets(m, n, 128, gen) for m in rows] if case["offsets"] else None})
        if case["graph"]:
            _run_blocks(s)          # first use of a kernel is not recorded
            torch.cuda.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                s["out"] = _run_blocks(s)
        return s
    m, n, group = case["m"], case["n"], case["group"]
    s["planes"], s["x"] = _planes(m, n, gen), _x(case["batch"], n, gen)
    sets = [case["p"]] if case["p"] else list(range(case["p_low"], P_MAX + 1))
    s["scales"] = {p: _scales(p, m, n, group, gen) for p in sets}
    s["offsets"] = {p: _offsets(m, n, group, gen) for p in sets} if case["offsets"] else None
    if not case["p"]:
        s["p_req"] = torch.randint(case["p_low"], P_MAX + 1, (case["batch"],), dtype=torch.int32, device="cuda", generator=gen)
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "quantize":
        planes, scales, offsets = bcq.bcq_quantize(state["w"], case["p_low"], case["p_high"], case["cycles"], case["group"], case["offsets"])
        return {"planes": planes, "scales": scales, "offsets": offsets}
    if case["kind"] == "blocks":
        if not case["graph"]:
            return _run_blocks(state)
        state["graph"].replay()
        return state["out"]
    if case["p"]:
        p = case["p"]
        return bcq.bcq_gemv(state["planes"], state["scales"][p], p, state["x"], group=case["group"],
                            offsets=state["offsets"][p] if state["offsets"] else None)
    return bcq.bcq_gemm_mixed(state["planes"], state["scales"], state["p_req"], state["x"], group=case["group"], offsets_by_p=state["offsets"])


def _weights64(planes, scales, offsets, group):
    """W_p in 64 bits from the storage format: bit j of word k is column 32 k + j, set for +1."""
    p, m, ngroups = scales.shape
    w = torch.zeros((m, ngroups * group), dtype=torch.float64, device=planes.device)
    shifts = torch.arange(32, dtype=torch.int32, device=planes.device)
    for i in range(p):
        bits = ((planes[i].unsqueeze(-1) >> shifts) & 1).reshape(m, ngroups, group)
        w += ((2 * bits - 1) * scales[i].double().unsqueeze(-1)).reshape(m, -1)
    if offsets is not None:
        w += offsets.double().repeat_interleave(group, dim=1)
    return w


def _product64(planes, scales, offsets, group, x):
    y = torch.empty((x.shape[0], planes.shape[1]), dtype=torch.float64, device=x.device)
    for r in range(0, planes.shape[1], 4096):
        rows = slice(r, r + 4096)
        y[:, rows] = x.double() @ _weights64(planes[:, rows], scales[:, rows], None if offsets is None else offsets[rows], group).t()
    return y


def exact(case, seed):
    """The results in 64 bits, without the library.  The quantiser has no such value: its scales are what its codes make them, and
    both are compared bit for bit."""
    if case["kind"] == "quantize":
        return None
    s = prepare(dict(case, graph=False), seed)
    if case["kind"] == "blocks":
        return [_product64(w, a, z, 128, t["x"]) for t in s["stages"]
                for w, a, z in zip(t["planes"], t["scales"], t["offsets"] or [None] * len(t["planes"]))]
    if case["p"]:
        return _product64(s["planes"], s["scales"][case["p"]], s["offsets"][case["p"]] if s["offsets"] else None, case["group"], s["x"])
    y = torch.empty((case["batch"], case["m"]), dtype=torch.float64, device="cuda")
    for p, scales in s["scales"].items():
        picked = (s["p_req"] == p).nonzero().flatten()
        y[picked] = _product64(s["planes"], scales, s["offsets"][p] if s["offsets"] else None, case["group"], s["x"][picked])
    return y


def _product_bytes(m, n, p, scale_rows, group, offset_rows):
    return m * n // 8 * p + m * (n // group) * 2 * (scale_rows + offset_rows)


def work(case):
    if case["kind"] == "quantize":
        m, n, lo, hi = case["m"], case["n"], case["p_low"], case["p_high"]
        scale_rows = sum(range(lo, hi + 1)) + ((hi - lo + 1) if case["offsets"] else 0)
        # per weight, in double precision: a cycle of the base stage compares with the 2^p levels and gathers p signed
        # sums, a cycle of the expansion to p bits takes a residual and gathers a signed sum
        ops = case["cycles"] * (2 * 2 ** lo + lo + 2 * (hi - lo) * 2)
        return {"bytes": 2 * m * n + m * n // 8 * hi + m * (n // case["group"]) * 2 * scale_rows, "flops": ops * m * n}
    if case["kind"] == "blocks":
        nbytes = flops = 0
        for rows, n in _block_rows(case):
            nbytes += case["batch"] * (n + sum(rows)) * 2
            nbytes += sum(_product_bytes(m, n, case["p"], case["p"], 128, 1 if case["offsets"] else 0) for m in rows)
            flops += 2 * case["batch"] * n * sum(rows)
        return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * flops}
    m, n, batch, p = case["m"], case["n"], case["batch"], case["p"]
    sets = [p] if p else list(range(case["p_low"], P_MAX + 1))
    nbytes = _product_bytes(m, n, max(sets), sum(sets), case["group"], len(sets) if case["offsets"] else 0)
    return {"bytes": nbytes + batch * (n + m) * 2 + (0 if p else 4 * batch), "flops": 2 * batch * m * n}


def tolerance(case):
    # the quantiser's codes and scales are fixed sequences of double-precision operations: bit for bit
    if case["kind"] == "quantize":
        return "exact"
    # results are rounded once to binary16 (2^-11), and the large-batch kernels round the rebuilt weights to it as well
    return {"rel": 1.2e-3, "max": 6e-3}
