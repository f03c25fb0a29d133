"""The calls whose speed is measured, with their inputs, work and 64-bit values.

Each case is one pass of work that a user of the library has it do, through the
functions of ``paper_2606_12487_amd``: a quantized linear from fp16 activations
(rotate + quantize, then the GEMM on the weight layout of that path), the whole
linear set of one transformer layer in decode, the 4-bit KV-cache codec, and the
residual-dynamics calibration of a layer.

Kinds (``case["kind"]``):

* ``fused``   ``qlinear_decode_fused``: a decode linear from fp16 x;
* ``native``  ``rotate_quant`` + ``qlinear_decode_native`` (decode weight layout);
* ``packed``  ``rotate_quant`` + ``qlinear`` (canonical weights);
* ``a8``      ``rotate_quant`` + ``qlinear_a8`` (8-bit-order weights);
* ``fp6``     ``rotate_quant_fp6`` + ``qlinear_fp6`` (FP6 block layout);
* ``range``   ``rotate_quant_range`` + ``qlinear_range`` (zero points);
* ``layer``   the four linears of one layer at decode, on the ``native`` path;
* ``kv``      ``kv_quant`` of new rows and ``kv_dequant`` of a cache;
* ``stats``   ``residual_dynamics``.
"""

import math

import torch

import paper_2606_12487_amd as dptq


def listed():
    return [
        # One token of one sequence through a fused QKV projection: latency.
        dict(name="decode_qkv_m1_a4", kind="fused", M=1, K=4096, h=4096, N=12288, bits=4),
        # A few sequences through an 8-bit (sensitive) layer's down projection.
        dict(name="decode_down_m4_a8", kind="native", M=4, K=14336, h=14336, N=4096, bits=8, signs=False),
        # A decode step of one layer of a large model: all four linears, weight bound.
        dict(name="decode_layer_m8_a4", kind="layer", M=8, d=8192, qkv=10240, ffn=28672, hf=28672, bits=4),
        # Continuous batching: tens of sequences in one decode step, ragged count.
        dict(name="batch_o_m48_a4", kind="packed", M=48, K=8192, h=8192, N=8192, bits=4, signs=False),
        # A larger decode batch through an 8-bit layer with randomized signs.
        dict(name="batch_qkv_m128_a8", kind="a8", M=128, K=4096, h=4096, N=6144, bits=8, signs=True),
        # A ragged chunk of a prompt (chunked prefill), 8-bit layer, long rows.
        dict(name="chunk_down_m333_a8", kind="a8", M=333, K=14336, h=14336, N=4096, bits=8, signs=False),
        # The same for a 4-bit layer: a chunk of a prompt through an output projection.
        dict(name="chunk_o_m500_fp6", kind="fp6", M=500, K=4096, h=4096, N=4096, bits=4, signs=False),
        # The range quantizer with zero points at a medium batch.
        dict(name="range_gate_m256_a4", kind="range", M=256, K=4096, h=4096, N=11008, bits=4),
        # Prefill of one prompt through an 8-bit layer, block-diagonal rotation.
        dict(name="prefill_down_m2048_a8", kind="a8", M=2048, K=11008, h=256, N=4096, bits=8, signs=False),
        # Prefill of a long prompt through the largest linear: the throughput case.
        dict(name="prefill_down_m4096_fp6", kind="fp6", M=4096, K=28672, h=28672, N=8192, bits=4, signs=False),
        # A prompt's keys written to the 4-bit cache, and a cache read back.
        dict(name="kv_chunk_and_cache", kind="kv", new=2048, cached=16384, D=1024, group=128),
        # Calibration of one layer over a calibration sequence.
        dict(name="stats_t2048", kind="stats", M=2048, K=4096, h=4096, bits=4),
    ]


# (K, had_size) of linears in use: power-of-two widths, 28 * 2^j widths, and
# widths rotated in blocks.
_ROWS = [(2048, 2048), (2560, 512), (3584, 3584), (4096, 4096), (5120, 1024), (8192, 8192),
         (11008, 256), (13824, 512), (14336, 14336), (28672, 28672)]
_MOST = 4096 * 28672 * 8192 // 4   # M * K * N of a drawn case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fused", "native", "packed", "packed", "a8", "a8", "fp6", "fp6", "range", "layer",
                       "kv", "stats"])
    if kind == "kv":
        return dict(kind=kind, new=_log_int(rng, 1, 8192), cached=_log_int(rng, 256, 32768),
                    D=rng.choice([512, 1024, 4096]), group=rng.choice([64, 128, 128]))
    if kind == "layer":
        d = rng.choice([2048, 4096, 5120])
        ffn, hf = rng.choice([(11008, 256), (14336, 14336), (13824, 512)])
        return dict(kind=kind, M=rng.randint(1, 16), d=d, qkv=d + 256 * rng.randint(1, 2 * d // 256), ffn=ffn,
                    hf=hf, bits=rng.choice([4, 4, 8]))
    K, h = rng.choice(_ROWS)
    bits = rng.choice([4, 8])
    if kind == "stats":
        return dict(kind=kind, M=_log_int(rng, 64, 8192), K=K, h=h, bits=bits)
    M = {"fused": lambda: rng.randint(1, 16), "native": lambda: rng.randint(1, 16),
         "packed": lambda: _log_int(rng, 17, 2048), "a8": lambda: _log_int(rng, 17, 4096),
         "fp6": lambda: _log_int(rng, 64, 4096), "range": lambda: _log_int(rng, 1, 2048)}[kind]()
    N = 16 * _log_int(rng, 64, min(1792, max(65, _MOST // (16 * M * K))))
    case = dict(kind=kind, M=M, K=K, h=h, N=N, bits={"a8": 8, "fp6": 4}.get(kind, bits))
    if kind in ("native", "packed", "a8", "fp6"):
        case["signs"] = rng.random() < 0.25
    return case


# ---------------------------------------------------------------------------
# Inputs: fp16 activations with a few large channels (or heavy tails where a
# row is a 28 * 2^j-wide product of an activation function) and N(0, 0.02^2)
# weights, all from the seed.
# ---------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + stream)
    return g


def _activations(g, M, K, heavy):
    x = torch.randn((M, K), generator=g, device="cuda")
    if heavy:   # Student-t with 3 degrees of freedom
        c = torch.zeros((M, K), device="cuda")
        for _ in range(3):
            c += torch.randn((M, K), generator=g, device="cuda").square_()
        x /= (c / 3).sqrt_()
    else:
        cols = torch.randperm(K, generator=g, device="cuda")[:4]
        x[:, cols] *= torch.rand((4,), generator=g, device="cuda") * 150 + 50
    return x.clamp_(-65504, 65504).half()


def _weights(g, N, K):
    return torch.randn((N, K), generator=g, device="cuda").mul_(0.02)


def _sign_bits(g, K):
    return torch.randint(0, 256, ((K + 7) // 8,), generator=g, device="cuda", dtype=torch.uint8)


def _linears(case):
    """(K, N, h) of the linears of a case, in call order."""
    if case["kind"] == "layer":
        d = case["d"]
        hd = d & -d
        return [(d, case["qkv"], hd), (d, d, hd), (d, 2 * case["ffn"], hd), (case["ffn"], d, case["hf"])]
    return [(case["K"], case["N"], case["h"])]


def _linear_inputs(case, seed, i):
    K, N, h = _linears(case)[i]
    g = _gen(seed, 16 * i)
    x = _activations(g, case["M"], K, heavy=h % 28 == 0)
    signs = _sign_bits(g, K) if case.get("signs") else None
    return x, signs, _weights(g, N, K)


def _kv_inputs(case, seed):
    g = _gen(seed, 1)
    new = _activations(g, case["new"], case["D"], heavy=False)
    return new, _activations(g, case["cached"], case["D"], heavy=False)


def _stats_inputs(case, seed):
    g = _gen(seed, 2)
    x = _activations(g, case["M"], case["K"], heavy=False)
    dx = (0.1 * torch.randn(x.shape, generator=g, device="cuda")).half()
    return x, dx


def prepare(case, seed):
    kind = case["kind"]
    if kind == "kv":
        new, old = _kv_inputs(case, seed)
        return dict(case=case, new=new, cache=dptq.kv_quant(old, case["group"]))
    if kind == "stats":
        x, dx = _stats_inputs(case, seed)
        return dict(case=case, x=x, dx=dx)
    calls = []
    for i, (K, N, h) in enumerate(_linears(case)):
        x, signs, w = _linear_inputs(case, seed, i)
        wp, ws = dptq.prepare_weights(w, h, signs=signs)
        del w
        c = dict(x=x, signs=signs, h=h, ws=ws, N=N, w=wp)
        if kind in ("native", "layer"):
            c["w"] = dptq.prepack_weights(wp, dptq.WEIGHTS_DECODE)
        elif kind == "a8":
            c["w"] = dptq.pack_w4_a8(wp)
        elif kind == "fp6":
            c["w"] = dptq.pack_fp6(wp)
        elif kind == "range":
            c["wsum"] = dptq.weight_sums(wp)
        if kind in ("fused", "native", "layer"):
            # A decode loop keeps its buffers.
            M, bits = case["M"], case["bits"]
            c["codes"] = torch.empty((M, K // 2) if bits == 4 else (M, K), device="cuda",
                                     dtype=torch.uint8 if bits == 4 else torch.int8)
            c["scales"] = torch.empty((M,), device="cuda")
            c["y"] = torch.empty((M, N), device="cuda", dtype=torch.float16)
        calls.append(c)
    return dict(case=case, calls=calls)


def _run_linear(kind, bits, M, c):
    x, h = c["x"], c["h"]
    if kind == "fused":
        return dptq.qlinear_decode_fused(x, h, bits, c["w"], c["ws"], c["y"], c["codes"], c["scales"])
    if kind in ("native", "layer"):
        codes, s = dptq.rotate_quant(x, h, bits, c["codes"], c["scales"], c["signs"])
        return dptq.qlinear_decode_native(codes, s, bits, c["w"], c["ws"], c["y"]), codes, s
    if kind == "packed":
        codes, s = dptq.rotate_quant(x, h, bits, signs=c["signs"])
        return dptq.qlinear(codes, s, bits, c["w"], c["ws"]), codes, s
    if kind == "a8":
        codes, s = dptq.rotate_quant(x, h, 8, signs=c["signs"])
        return dptq.qlinear_a8(codes, s, c["w"], c["ws"]), codes, s
    if kind == "fp6":
        a6, s = dptq.rotate_quant_fp6(x, h, signs=c["signs"])
        return dptq.qlinear_fp6(a6, s, c["w"], c["ws"], M, x.shape[1], c["N"]), a6, s
    codes, s, z = dptq.rotate_quant_range(x, h, bits)
    return dptq.qlinear_range(codes, s, z, bits, c["w"], c["ws"], c["wsum"]), codes, s, z


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "kv":
        codes, s, m = dptq.kv_quant(state["new"], case["group"])
        return codes, s, m, dptq.kv_dequant(*state["cache"], case["group"])
    if kind == "stats":
        return dptq.residual_dynamics(state["x"], state["dx"], case["h"], case["bits"])
    return [_run_linear(kind, case["bits"], case["M"], c) for c in state["calls"]]


def work(case):
    kind = case["kind"]
    if kind == "kv":
        n = (case["new"] + case["cached"]) * case["D"]
        return {"bytes": n * 2.5 + n / case["group"] * 8, "flops": 0}
    if kind == "stats":
        return {"bytes": case["M"] * (4 * case["K"] + 8) + 16,
                "flops": case["M"] * case["K"] * (math.log2(case["h"]) + 8)}
    M, b, f = case["M"], 0, 0
    for K, N, h in _linears(case):
        wbytes = N * K * (0.75 if kind == "fp6" else 0.5) + 4 * N
        cbytes = M * K * (0.75 if kind == "fp6" else case["bits"] / 8) + 4 * M   # returned codes and scales
        b += 2 * M * K + wbytes + cbytes + 2 * M * N
        if kind == "range":
            b += 4 * M + 4 * N
        f += 2 * M * N * K
    return {"bytes": b, "flops": f}


def tolerance(case):
    # The codes, scales and outputs have a pinned order of fp32 operations and
    # exact integer sums; only the calibration's norms may be summed in any order.
    # Its statistics are 5e-8 (2-norm) and 2e-7 (largest) from the 64-bit values
    # at 4096 elements a row; rows are up to 28672.
    return {"rel": 1e-6, "max": 1e-5} if case["kind"] == "stats" else "exact"


# ---------------------------------------------------------------------------
# The same values in 64 bits, in plain torch.
# ---------------------------------------------------------------------------
def _h28():
    """Hadamard matrix of order 28: Paley's second construction over GF(13)."""
    sq = {(a * a) % 13 for a in range(1, 13)}
    c = torch.zeros((14, 14), dtype=torch.float64)
    c[0, 1:] = 1
    c[1:, 0] = 1
    for i in range(13):
        for j in range(13):
            d = (j - i) % 13
            c[1 + i, 1 + j] = 0 if d == 0 else (1 if d in sq else -1)
    a = torch.tensor([[1., 1.], [1., -1.]], dtype=torch.float64)
    b = torch.tensor([[1., -1.], [-1., -1.]], dtype=torch.float64)
    return torch.kron(c, a) + torch.kron(torch.eye(14, dtype=torch.float64), b)


def _rotate(x, h):
    """x (I (x) H_h) in 64 bits."""
    R, K = x.shape
    f = 28 if h % 28 == 0 else 1
    p = h // f
    v = x.double().reshape(R * (K // p), p)
    s = 1
    while s < p:
        u = v.reshape(-1, p // (2 * s), 2, s)
        v = torch.stack((u[:, :, 0] + u[:, :, 1], u[:, :, 0] - u[:, :, 1]), dim=2).reshape(-1, p)
        s *= 2
    if f == 28:
        t = v.reshape(-1, 28, p).transpose(1, 2).reshape(-1, 28)
        v = (t @ _h28().to(t.device)).reshape(-1, p, 28).transpose(1, 2)
    return v.reshape(R, K)


def _with_signs(x, signs):
    if signs is None:
        return x.double()
    bits = (signs[:, None] >> torch.arange(8, device=signs.device, dtype=torch.uint8)) & 1
    return x.double() * (1 - 2 * bits.reshape(-1)[:x.shape[1]].double())


def _codes(y, qmax):
    s = y.abs().amax(1, keepdim=True) / qmax
    q = torch.where(s > 0, torch.round(y / torch.where(s > 0, s, 1.0)), torch.zeros_like(y))
    return q.clamp(-qmax - 1, qmax), s


def _exact_weights(w, signs, h):
    """Codes and scales of the weights, a block of rows at a time."""
    q, s = [], []
    for b in torch.split(w, 4096):
        cb, sb = _codes(_rotate(_with_signs(b, signs), h), 7)
        q.append(cb)
        s.append(sb)
    return torch.cat(q), torch.cat(s) / h


def exact(case, seed):
    kind = case["kind"]
    if kind == "kv":
        new, old = _kv_inputs(case, seed)
        g = case["group"]

        def groups(x):
            v = x.double().reshape(x.shape[0], -1, g)
            m = v.amin(2, keepdim=True)
            s = (v.amax(2, keepdim=True) - m) / 15
            q = torch.round((v - m) / torch.where(s > 0, s, 1.0)).clamp(0, 15)
            return s, m, (q * s + m).reshape(x.shape)

        s, m, _ = groups(new)
        return None, s[:, :, 0], m[:, :, 0], groups(old)[2]
    if kind == "stats":
        x, dx = _stats_inputs(case, seed)
        qmax = 7 if case["bits"] == 4 else 127
        y = _rotate(x.double() + dx.double(), case["h"])
        q, s = _codes(y, qmax)
        err = (q * s - y).square().sum(1) / case["h"]
        xx, eps = x.double().square().sum(1), 1e-8
        jr = dx.double().square().sum(1).sqrt() / (xx.sqrt() + eps)
        snr = 10 * torch.log10(xx / (err + eps))
        return jr, snr, torch.stack((jr.mean(), snr.mean()))
    outs = []
    for i, (K, N, h) in enumerate(_linears(case)):
        x, signs, w = _linear_inputs(case, seed, i)
        wq, ws = _exact_weights(w, signs, h)
        del w
        y = _rotate(_with_signs(x, signs), h)
        if kind == "range":
            n = 2 ** case["bits"] - 1
            mx, mn = y.amax(1, keepdim=True).clamp(min=0), y.amin(1, keepdim=True).clamp(max=0)
            s = (mx - mn) / n
            z = torch.round(-mn / s).clamp(0, n)
            q = (torch.round(y / s) + z).clamp(0, n) - z
        else:
            q, s = _codes(y, 7 if case["bits"] == 4 else 127)
        out = (q @ wq.t()) * s * ws.t()
        outs.append((out, None, s[:, 0]) + ((None,) if kind == "range" else ()))
    return outs
