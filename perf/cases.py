"""The calls whose speed is watched: what a program that links this GEMM asks of it, over the range it asks it.

A case is one call of the C ABI (through the ctypes binding) on operands that lie in device memory, as a linear
layer, its gradients, an attention product or a scientific fp32 product makes it.  `layout` names the storage of A
and B: the first letter is N for A stored M x K and T for K x M, the second N for B stored K x N and T for N x K (a
weight kept as [out, in])."""
import math

import torch

import paper_2512_16465_amd as lg

_TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
_CODE = {"bf16": lg.GEMM_BF16, "fp16": lg.GEMM_F16, "fp32": lg.GEMM_F32}
_BYTES = {"bf16": 2, "fp16": 2, "fp32": 4}
_ACT = {"none": lg.GEMM_ACT_NONE, "gelu": lg.GEMM_ACT_GELU_ERF, "relu": lg.GEMM_ACT_RELU, "silu": lg.GEMM_ACT_SILU,
        "gelu_tanh": lg.GEMM_ACT_GELU_TANH}


def _case(M, N, K, layout, dtype, out="", beta=0.0, bias="", act="none", batch=1, name=""):
    c = {"M": M, "N": N, "K": K, "layout": layout, "dtype": dtype, "out": out or dtype, "beta": beta, "bias": bias,
         "act": act, "batch": batch}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one token through a square projection kept as [out, in]: the smallest call of a decoding step
        _case(1, 4096, 4096, "NT", "bf16", name="decode_1x4096x4096_nt"),
        # eight tokens on a 128 MiB weight stored row by row
        _case(8, 8192, 8192, "NN", "bf16", name="decode_8x8192x8192_nn"),
        # a batch of decoding sequences, accumulated into the residual stream
        _case(32, 16384, 16384, "NN", "bf16", beta=1.0, name="decode_32x16384x16384_nn"),
        # a short prompt (or a large decoding batch) on a weight of 512 MiB
        _case(128, 16384, 16384, "NT", "bf16", name="prefill_128x16384x16384_nt"),
        # a projection of a few thousand tokens: the ordinary prefill or training forward
        _case(4096, 4096, 4096, "NT", "bf16", name="forward_4096_nt"),
        # the headline of the benchmark; as the gradient of a layer's input it has the same layout
        _case(8192, 8192, 8192, "NN", "bf16", out="fp32", name="square_8192_nn"),
        # the up-projection of an MLP with its bias and GELU: the largest call
        _case(8192, 28672, 8192, "NT", "bf16", bias="bf16", act="gelu", name="mlp_8192x28672x8192_nt"),
        # the gradient of a weight, summed over the tokens and added to an fp32 master gradient
        _case(4096, 4096, 8192, "TN", "fp16", out="fp32", beta=1.0, name="wgrad_4096x4096x8192_tn"),
        # sizes that are no multiple of anything, in every dimension
        _case(2049, 2051, 2045, "NN", "bf16", bias="fp32", name="odd_2049x2051x2045_nn"),
        # the scores of 32 heads
        _case(2048, 2048, 128, "NT", "bf16", batch=32, name="scores_32x2048x2048x128_nt"),
        # fp32 from end to end: the smallest of the benchmark and a large one
        _case(256, 256, 256, "NN", "fp32", name="fp32_256_nn"),
        _case(4096, 4096, 4096, "NN", "fp32", name="fp32_4096_nn"),
    ]


def _log(rng, lo, hi, step):
    """A size between lo and hi, spread over its logarithm; step 1 gives odd sizes."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    v = max(1, round(v / step)) * step
    return int(v | 1) if step == 1 else int(v)


def draw(rng):
    kind = rng.choice(("decode", "forward", "forward", "grad", "odd", "odd_decode", "batch", "fp32", "fp32"))
    half = rng.choice(("bf16", "bf16", "fp16"))
    step = rng.choice((8, 64, 256))
    if kind == "decode":
        return _case(_log(rng, 1, 64, 1) - rng.randint(0, 1) or 1, _log(rng, 1024, 16384, step), _log(rng, 1024, 16384, step),
                     rng.choice(("NT", "NN")), half, beta=rng.choice((0.0, 1.0)))
    if kind == "forward":
        return _case(_log(rng, 64, 8192, rng.choice((1, 8, 256))), _log(rng, 512, 16384, step), _log(rng, 512, 8192, step), "NT", half,
                     bias=rng.choice(("", half, "fp32")), act=rng.choice(("none", "gelu", "relu", "silu", "gelu_tanh")))
    if kind == "grad":
        layout = rng.choice(("NN", "TN"))
        return _case(_log(rng, 256, 8192, step), _log(rng, 256, 8192, step), _log(rng, 256, 8192, step), layout, half,
                     out="fp32" if layout == "TN" else half, beta=1.0 if layout == "TN" else 0.0)
    if kind == "odd":
        return _case(_log(rng, 64, 3072, 1), _log(rng, 64, 3072, 1), _log(rng, 64, 4096, 1), rng.choice(("NT", "NN", "TN")),
                     rng.choice((half, half, "fp32")), bias=rng.choice(("", "fp32")), act=rng.choice(("none", "gelu")))
    if kind == "odd_decode":
        return _case(rng.randint(1, 32), _log(rng, 1024, 16384, 1), _log(rng, 512, 8192, rng.choice((1, 64))),
                     rng.choice(("NT", "NN")), half)
    if kind == "batch":
        s, d = _log(rng, 128, 2048, rng.choice((1, 8, 64))), rng.choice((64, 80, 128))
        heads = rng.randint(4, 32)
        # the scores, or the weighted sum of the values
        return _case(s, s, d, "NT", half, batch=heads) if rng.random() < 0.5 else _case(s, d, s, "NN", half, batch=heads)
    return _case(_log(rng, 1, 4096, rng.choice((1, 4, 64))), _log(rng, 64, 4096, rng.choice((4, 64))), _log(rng, 64, 4096, rng.choice((4, 64))),
                 rng.choice(("NN", "NT", "TN")), "fp32", beta=rng.choice((0.0, 0.0, 1.0)), act=rng.choice(("none", "none", "silu")))


def _inputs(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    ta, tb = c["layout"][0] == "T", c["layout"][1] == "T"
    dt, nb = _TORCH[c["dtype"]], c["batch"]

    def normal(std, *shape, dtype=dt):
        return (torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dtype)

    # activations are of order one; a weight has the 0.02 of an initialised layer, the keys of a batch 1 / sqrt(K)
    A = normal(1.0, nb, *((c["K"], c["M"]) if ta else (c["M"], c["K"])))
    B = normal(c["K"] ** -0.5 if nb > 1 else 0.02, nb, *((c["N"], c["K"]) if tb else (c["K"], c["N"])))
    C = normal(1.0, nb, c["M"], c["N"], dtype=_TORCH[c["out"]]) if c["beta"] else None
    bias = normal(0.02, c["N"], dtype=_TORCH[c["bias"]]) if c["bias"] else None
    return A, B, C, bias


_handles = {}


def _handle():
    """The one handle that a program keeps for its device."""
    dev = torch.cuda.current_device()
    if dev not in _handles:
        _handles[dev] = lg.gemm_create()
    return _handles[dev]


def prepare(case, seed):
    A, B, C, bias = _inputs(case, seed)
    if C is None:
        C = torch.empty(case["batch"], case["M"], case["N"], device="cuda", dtype=_TORCH[case["out"]])
    epi = lg.make_epilogue(_CODE[case["out"]], bias.data_ptr() if bias is not None else 0,
                           _CODE[case["bias"] or "fp32"], _ACT[case["act"]])
    return {"case": case, "A": A, "B": B, "C": C, "bias": bias, "epi": epi, "handle": _handle(),
            "ta": int(case["layout"][0] == "T"), "tb": int(case["layout"][1] == "T"), "dt": _CODE[case["dtype"]]}


def run(s):
    c, A, B, C = s["case"], s["A"], s["B"], s["C"]
    stream = torch.cuda.current_stream().cuda_stream
    M, N, K = c["M"], c["N"], c["K"]
    if c["batch"] == 1:
        lg.gemm_run(s["handle"], M, N, K, s["ta"], s["tb"], s["dt"], 1.0, A.data_ptr(), A.shape[2], B.data_ptr(), B.shape[2],
                    c["beta"], C.data_ptr(), N, s["epi"], stream)
    else:
        lg.gemm_run_batched(s["handle"], c["batch"], M, N, K, s["ta"], s["tb"], s["dt"], 1.0, A.data_ptr(), A.shape[2], M * K,
                            B.data_ptr(), B.shape[2], N * K, c["beta"], C.data_ptr(), N, M * N, s["epi"], stream)
    return C


def work(case):
    M, N, K, nb = case["M"], case["N"], case["K"], case["batch"]
    b = (M * K + K * N) * _BYTES[case["dtype"]] + M * N * _BYTES[case["out"]] * (2 if case["beta"] else 1)
    b = b * nb + (N * _BYTES[case["bias"]] if case["bias"] else 0)
    return {"bytes": b, "flops": 2 * M * N * K * nb}


def tolerance(case):
    # about four times what the path shows against 64 bits: one rounding of a 16-bit result (bf16 1.7e-3, fp16 2.1e-4
    # in the 2-norm), and the rounding of fp32 sums of up to 16384 terms
    return {"rel": {"bf16": 7e-3, "fp16": 9e-4, "fp32": 1e-5}[case["out"]]}


def exact(case, seed):
    A, B, C, bias = _inputs(case, seed)
    a = (A.transpose(1, 2) if case["layout"][0] == "T" else A)
    b = (B.transpose(1, 2) if case["layout"][1] == "T" else B)
    out = torch.stack([a[i].double() @ b[i].double() for i in range(case["batch"])])
    if C is not None:
        out += case["beta"] * C.double()
    if bias is not None:
        out += bias.double()
    f = torch.nn.functional
    return {"none": lambda x: x, "gelu": f.gelu, "relu": f.relu, "silu": f.silu,
            "gelu_tanh": lambda x: f.gelu(x, approximate="tanh")}[case["act"]](out)
