"""The work that users of this library have it do, as cases that can be timed and checked.

Quantized inference is one linear after another: at decode with one activation row or a few, in
batched decode with tens of rows, at prefill with hundreds or thousands. A serving program keeps
the codes and codebooks on the GPU and calls the linears directly, or captures a decode pass in a
HIP graph and replays it. Before that, every tensor is quantized at load (fit and encode),
calibrated (GPTQ) or decoded again (dequantize). Shapes are the Llama-style ones this repository
benchmarks, and general ones with in-feature counts that are not powers of two and odd
out-feature and batch counts.

Codes and codebooks of the products are made here with plain torch (a logarithmic codebook over
the tensor's effective range), so the products' inputs do not depend on the library.
"""
import math

import numpy as np
import torch

from paper_2607_01127_amd import inputs
from paper_2607_01127_amd import logbq as L

DEV = "cuda:0"


def listed():
    return [
        # The smallest call: one row through a 2048 x 2048 projection, called eagerly.
        _linear("linear_2048x2048_m1", 2048, 2048, 1),
        # One token through the linears of two 4096-wide decoder layers, replayed as a graph:
        # the steady state of single-stream decode.
        _decode("decode_4096_m1", 4096, 14336, 1024, 1),
        # The same with four sequences decoded together.
        _decode("decode_4096_m4", 4096, 14336, 1024, 4),
        # The largest single linear at one row: bound by streaming its codes.
        _linear("linear_8192x28672_m1", 28672, 8192, 1),
        # A down projection whose in-feature count is no power of two, eight sequences.
        _linear("linear_11008x4096_m8", 4096, 11008, 8),
        # Batched decode: 64 sequences through a gate projection.
        _linear("linear_4096x14336_m64", 14336, 4096, 64),
        # Prefill of a 2048-token prompt through the same projection.
        _linear("linear_4096x14336_m2048", 14336, 4096, 2048),
        # 8-bit codes, four sequences.
        _linear("linear8_4096x14336_m4", 14336, 4096, 4, bits=8),
        # 8-bit codes, a ragged 777-token prompt through a projection with odd sizes.
        _linear("linear8_3072x8199_m777", 8199, 3072, 777, bits=8),
        # Quantize at load: fit one gate projection on the device and encode it.
        dict(name="quantize_14336x4096", kind="quantize", n=14336, k=4096, bits=4),
        # Decode codes back to float32 weights, e.g. to merge an adapter or to export.
        dict(name="dequantize_14336x4096", kind="dequantize", n=14336, k=4096, bits=4),
        # GPTQ calibration of an up projection.
        dict(name="gptq_8192x2048", kind="gptq", n=8192, k=2048, book="log"),
    ]


def _linear(name, n, k, m, bits=4, book="log"):
    return dict(name=name, kind="linear", n=n, k=k, m=m, bits=bits, book=book)


def _decode(name, hidden, inter, kv, m):
    return dict(name=name, kind="decode", hidden=hidden, inter=inter, kv=kv, m=m, layers=2)


def _log_int(rng, lo, hi, step=1):
    """An integer spread over the logarithm of [lo, hi], a multiple of step."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(round(v / step)) * step, -(-lo // step) * step), hi // step * step)


def draw(rng):
    kind = rng.choice(["decode_rows"] * 3 + ["batch"] * 3 + ["prefill"] * 3
                      + ["layer", "quantize", "dequantize", "gptq"])
    if kind in ("decode_rows", "batch", "prefill"):
        # Half of the in-feature counts are those of common models, half any multiple of 32.
        k = (rng.choice([2048, 4096, 8192, 14336]) if rng.random() < 0.5
             else _log_int(rng, 512, 16384, 32))
        n = (rng.choice([1024, 2048, 4096, 8192, 14336, 28672]) if rng.random() < 0.5
             else _log_int(rng, 512, 28672))
        m = _log_int(rng, *{"decode_rows": (1, 16), "batch": (17, 256),
                            "prefill": (257, 2048)}[kind])
        while m * n * k > 2048 * 4096 * 14336:
            n = max(512, n // 2)
            k = k if n > 512 else 4096
        bits = rng.choice([4, 4, 4, 8])
        # One 4-bit linear in six carries the asymmetric linear baseline's codebook.
        book = "uniform" if bits == 4 and rng.random() < 1 / 6 else "log"
        return dict(kind="linear", n=n, k=k, m=m, bits=bits, book=book)
    if kind == "layer":
        hidden = _log_int(rng, 1024, 4096, 256)
        return dict(kind="decode", hidden=hidden, inter=_log_int(rng, 2 * hidden, 14336, 128),
                    kv=max(256, hidden // rng.choice([1, 2, 4, 8]) // 32 * 32),
                    m=rng.choice([1, 1, 2, 3, 4, 6, 8]), layers=2)
    if kind in ("quantize", "dequantize"):
        return dict(kind=kind, n=_log_int(rng, 256, 14336), k=_log_int(rng, 512, 4096, 32),
                    bits=rng.choice([4, 4, 8]))
    return dict(kind="gptq", n=_log_int(rng, 256, 8192), k=_log_int(rng, 512, 2048, 32),
                book=rng.choice(["log", "log", "uniform"]))


# ------------------------------------------------------------------ inputs

def _weights(n, k, seed):
    """Heavy-tailed float32 weights, the spread of Llama-style projections."""
    return inputs.student_t_weights(n, k, 4, 0.02, seed, device=DEV)


def _log_book(w, bits):
    """Base, shift and float32 codebook of a logarithmic quantizer over the effective range of
    w: the largest magnitude, and the magnitude below which a fraction eps of the energy lies
    (taken from a sample)."""
    eps = 4e-3 if bits == 4 else 1e-6
    a = np.sort(np.abs(w.reshape(-1)[:1 << 18].cpu().numpy().astype(np.float64)))
    c = np.cumsum(a * a)
    wmax, wmin = float(w.abs().max()), float(a[np.searchsorted(c, eps * c[-1])])
    qmax = (1 << (bits - 1)) - 1
    base = (wmax / wmin) ** (1.0 / qmax)
    shift = qmax - math.floor(math.log(wmax) / math.log(base))
    book = np.zeros(2 << (bits - 1))
    mag = base ** (np.arange(1, qmax + 1) - float(shift))
    book[1:qmax + 1], book[qmax + 2:] = mag, -mag
    return base, shift, book.astype(np.float32)


def _quantize(w, bits, book):
    """Packed codes of w on the GPU and the host codebook."""
    if book == "uniform":
        lo, hi = float(w.min()), float(w.max())
        s = (hi - lo) / 15
        z = round(lo / s)
        q = (torch.floor(w / s + 0.5) - z).clamp_(0, 15).to(torch.uint8)
        values = (s * (np.arange(16) + z)).astype(np.float32)
    else:
        base, shift, values = _log_book(w, bits)
        qmax = (1 << (bits - 1)) - 1
        mag = torch.floor(torch.log(w.abs()) / math.log(base) + (shift + 0.5)).clamp_(0, qmax)
        q = mag.to(torch.uint8)
        q += ((w < 0) & (q > 0)).to(torch.uint8) << (bits - 1)
    if bits == 4:
        q = q[:, 0::2] | (q[:, 1::2] << 4)
    return q.contiguous(), values


def _decoder(case):
    """(name, in features, out features) of one decoder layer's linears."""
    lins = inputs.decoder_linears(case["hidden"], case["inter"], case["kv"])
    return [(lin.name, lin.k, lin.n) for lin in lins]


GROUPS = (("q", "k", "v"), ("o",), ("gate", "up"), ("down",))


def _decode_inputs(case, seed):
    layers = []
    for layer in range(case["layers"]):
        lins = {}
        for i, (name, k, n) in enumerate(_decoder(case)):
            w = _weights(n, k, [seed, layer, i, 0])
            lins[name] = _quantize(w, 4, "log")
        layers.append(lins)
    xs = {k: inputs.activations(case["m"], k, [seed, 0, k, 1], device=DEV)
          for k in {k for _, k, _ in _decoder(case)}}
    return layers, xs


def _hessian_factor(k, seed):
    """Upper factor of the damped inverse Hessian of correlated synthetic activations."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7919 + 17)
    scale = torch.exp(0.5 * torch.randn(k, generator=g, device=DEV))
    x = torch.randn(4096, k, generator=g, device=DEV) * scale
    x += torch.randn(4096, 8, generator=g, device=DEV) @ torch.randn(8, k, generator=g, device=DEV)
    x = x.double()
    h = 2.0 / x.shape[0] * (x.T @ x)
    h += 0.01 * h.diagonal().mean() * torch.eye(k, dtype=h.dtype, device=DEV)
    inv = torch.cholesky_inverse(torch.linalg.cholesky(h))
    return torch.linalg.cholesky(inv, upper=True).float().contiguous()


def _linear_inputs(case, seed):
    w = _weights(case["n"], case["k"], [seed, 0, 0, 0])
    codes, book = _quantize(w, case["bits"], case["book"])
    x = inputs.activations(case["m"], case["k"], [seed, 0, 0, 1], device=DEV)
    return x, codes, book


def prepare(case, seed):
    kind = case["kind"]
    if kind == "linear":
        x, codes, book = _linear_inputs(case, seed)
        return dict(kind=kind, x=x, codes=codes, book=book,
                    call=L.linear if case["bits"] == 4 else L.linear8)
    if kind == "decode":
        layers, xs = _decode_inputs(case, seed)
        ks = {name: k for name, k, _ in _decoder(case)}

        def one_pass():
            out = []
            for lins in layers:
                for names in GROUPS:
                    x = xs[ks[names[0]]]
                    if len(names) == 1:
                        out.append(L.linear(x, *lins[names[0]]))
                    else:
                        out += L.linear_multi(x, [lins[a][0] for a in names],
                                              [lins[a][1] for a in names])
            return out

        one_pass()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outs = one_pass()
        return dict(kind=kind, graph=graph, outs=outs, layers=layers, xs=xs)
    w = _weights(case["n"], case["k"], [seed, 0, 0, 0])
    if kind == "quantize":
        work = torch.empty(L.FIT_WORKSPACE_BYTES, dtype=torch.uint8, device=DEV)
        return dict(kind=kind, w=w, bits=case["bits"], eps=4e-3 if case["bits"] == 4 else 1e-6,
                    work=work)
    if kind == "dequantize":
        codes, book = _quantize(w, case["bits"], "log")
        return dict(kind=kind, codes=codes, book=book,
                    call=L.dequantize if case["bits"] == 4 else L.dequantize8)
    params = L.fit_uniform(w) if case["book"] == "uniform" else L.fit_device(w)
    return dict(kind=kind, w=w, u=_hessian_factor(case["k"], seed), params=params,
                work=torch.empty((case["n"], L.GPTQ_BLOCK), dtype=torch.float32, device=DEV))


def run(state):
    kind = state["kind"]
    if kind == "linear":
        return state["call"](state["x"], state["codes"], state["book"])
    if kind == "decode":
        state["graph"].replay()
        return state["outs"]
    if kind == "quantize":
        p = L.fit_device(state["w"], state["bits"], state["eps"], workspace=state["work"])
        codes, book = L.encode(state["w"], p)
        return dict(codes=codes, book=book, base=p.base, shift=p.shift, wmin=p.wmin, wmax=p.wmax,
                    index=p.wmin_index, thresholds=p.thresholds_array()[:p.qmax])
    if kind == "dequantize":
        return state["call"](state["codes"], state["book"])
    w = state["w"].clone()          # the calibration updates its weights in place
    codes = L.gptq(w, state["u"], state["params"], workspace=state["work"])
    return dict(codes=codes, w=w)


# ------------------------------------------------------------------ what a pass needs

def _linear_work(m, n, k, bits):
    return n * k * bits // 8 + 2 * m * k + 4 * m * n, 2 * m * n * k


def work(case):
    kind = case["kind"]
    if kind == "linear":
        b, f = _linear_work(case["m"], case["n"], case["k"], case["bits"])
    elif kind == "decode":
        b = f = 0
        for _, k, n in _decoder(case):
            wb, wf = _linear_work(case["m"], n, k, 4)
            b, f = b + case["layers"] * wb, f + case["layers"] * wf
    else:
        n, k = case["n"], case["k"]
        code_bytes = n * k * case.get("bits", 4) // 8
        b, f = 4 * n * k + code_bytes, 0
        if kind == "gptq":
            # Weights in and out, the factor's upper triangle, the codes; a multiplication and a
            # subtraction for every pair of columns of every row.
            b, f = 8 * n * k + 2 * k * k + code_bytes, n * k * k
    return {"bytes": b, "flops": f}


def tolerance(case):
    # Codes, parameters, looked-up weights and the calibration's fixed order of float32
    # operations are exact. Products round each codebook entry to float16 and sum in float32.
    return {"rel": 1e-3} if case["kind"] in ("linear", "decode") else "exact"


# ------------------------------------------------------------------ 64-bit results

def _values(codes, book, bits):
    """float64 weights of packed codes."""
    table = torch.tensor(book.astype(np.float64), device=codes.device)
    if bits == 8:
        return table[codes.int()]
    n, h = codes.shape
    out = torch.empty((n, 2 * h), dtype=torch.float64, device=codes.device)
    out[:, 0::2] = table[(codes & 15).int()]
    out[:, 1::2] = table[(codes >> 4).int()]
    return out


def _product(x, codes, book, bits):
    out = [x.double() @ _values(c, book, bits).T.contiguous() for c in codes.split(4096)]
    return torch.cat(out, dim=1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        x, codes, book = _linear_inputs(case, seed)
        return _product(x, codes, book, case["bits"])
    if kind == "decode":
        layers, xs = _decode_inputs(case, seed)
        ks = {name: k for name, k, _ in _decoder(case)}
        return [_product(xs[ks[a]], *lins[a], 4) for lins in layers for g in GROUPS for a in g]
    if kind == "dequantize":
        w = _weights(case["n"], case["k"], [seed, 0, 0, 0])
        return _values(*_quantize(w, case["bits"], "log"), case["bits"])
    # Whole-number codes, and float32 results that the calibration's own decisions lead to, have
    # no 64-bit value that differs from what they are.
    return None
