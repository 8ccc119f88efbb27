"""Measured cases: the calls that users of the library make, over the ranges they make them in.

Four kinds of work, each through the public binding:

* ``spmm``   one ``us_spmm`` on a weight matrix encoded beforehand: decode
  widths (1 to 32 activation columns), prefill widths (up to 1024), 4-bit rows
  in stored order, row-reordered, and 2-bit weights, with and without the
  dequant epilogue;
* ``layer``  the projections of one decoder layer, captured once in a HIP
  graph and replayed per token, as a serving loop does;
* ``gemm``   ``us_gemm_i8``, the dense INT8 product of the same shapes, for
  layers that are not pruned;
* ``encode`` the conversion of a pruned matrix on the host and its upload, as
  when a model is loaded.

Weights, masks, activations and scales follow ``paper_2608_09291_amd.synth``
(nonzeros uniform over the value range, i.i.d. or row-skewed masks, uniform
INT4 activations), drawn here on the GPU because the inputs are made often.
"""
import math

import numpy as np
import torch

from paper_2608_09291_amd import binding

#: Largest weight matrix (elements) and largest M K N of one call here.
MK_MAX = 28672 * 8192
MKN_MAX = 12288 * 4096 * 1024


def _spmm(name, M, K, N, s, bits=4, reorder=False, dequant=False, skew=False):
    c = {"kind": "spmm", "M": M, "K": K, "N": N, "sparsity": s, "bits": bits, "reorder": reorder,
         "dequant": dequant, "skew": skew}
    return {"name": name, **c} if name else c


def listed():
    return [
        # Grouped-query key/value projection of an 8B model: the smallest
        # call, bound by launch latency.
        _spmm("kv_1024x4096_n8", 1024, 4096, 8, 0.5),
        # Decode of a batch of 8 through one layer of LLaMA-2-7B's shapes:
        # fused QKV, the two FFN up projections and the FFN down projection
        # (the benchmark's shape), replayed from a HIP graph.
        {"name": "layer_7b_n8", "kind": "layer", "hidden": 4096, "ffn": 11008, "N": 8, "sparsity": 0.5},
        # One-column decode of a 70B-class FFN matrix held whole on one GPU.
        _spmm("ffn_28672x8192_s70_n1", 28672, 8192, 1, 0.7, dequant=True),
        # Row-skewed density at 16 columns (LLaMA-2-13B FFN).
        _spmm("ffn_13824x5120_skew60_n16", 13824, 5120, 16, 0.6, skew=True),
        # The widest single pass on the large matrix.
        _spmm("ffn_28672x8192_s70_n32", 28672, 8192, 32, 0.7, dequant=True),
        # 2-bit weights (W2A4), an odd width above one MFMA column block.
        _spmm("w2_ffn_up_11008x4096_n27", 11008, 4096, 27, 0.5, bits=2),
        # Row-reordered weights at a decode width.
        _spmm("reordered_28672x8192_s70_n5", 28672, 8192, 5, 0.7, reorder=True, dequant=True),
        # A short prompt: ragged prefill width.
        _spmm("prefill_4096x11008_n100", 4096, 11008, 100, 0.5, dequant=True),
        # A full prefill chunk, the widest accepted.
        _spmm("prefill_12288x4096_n1024", 12288, 4096, 1024, 0.5),
        # The dense INT8 product of the benchmark's shape, decode and prefill.
        {"name": "gemm_4096x11008_n8", "kind": "gemm", "M": 4096, "K": 11008, "N": 8},
        {"name": "gemm_4096x11008_n256", "kind": "gemm", "M": 4096, "K": 11008, "N": 256},
        # Conversion and upload of one pruned matrix (host work).
        {"name": "encode_4096x11008", "kind": "encode", "M": 4096, "K": 11008, "sparsity": 0.5, "bits": 4,
         "reorder": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, m_lo, m_hi, k_lo, k_hi, most):
    """M a multiple of 16, K a multiple of 64 (what the format takes), M K at most `most`."""
    while True:
        M, K = 16 * _log_int(rng, m_lo // 16, m_hi // 16), 64 * _log_int(rng, k_lo // 64, k_hi // 64)
        if M * K <= most:
            return M, K


def draw(rng):
    kind = rng.choices(["spmm", "layer", "gemm", "encode"], [10, 1, 2, 1])[0]
    s = round(rng.uniform(0.3, 0.7), 2)
    if kind == "layer":
        return {"kind": "layer", "hidden": 64 * rng.randint(16, 80), "ffn": 64 * rng.randint(32, 172),
                "N": _log_int(rng, 1, 32), "sparsity": s}
    if kind == "encode":
        M, K = _shape(rng, 256, 12288, 256, 12288, 4096 * 11008)
        form = rng.choice([(4, False), (4, False), (4, True), (2, False)])
        return {"kind": "encode", "M": M, "K": K, "sparsity": s, "bits": form[0], "reorder": form[1]}
    N = _log_int(rng, 1, 32) if rng.random() < 0.5 else _log_int(rng, 33, 1024)
    if kind == "gemm":
        M, K = _shape(rng, 256, 16384, 256, 16384, min(12288 * 8192, MKN_MAX // (2 * N)))
        return {"kind": "gemm", "M": M, "K": K, "N": N}
    M, K = _shape(rng, 256, 28672, 256, 28672, min(MK_MAX, MKN_MAX // N))
    bits, reorder = rng.choice([(4, False), (4, False), (4, False), (4, True), (2, False)])
    return _spmm(None, M, K, N, s, bits=bits, reorder=reorder, dequant=rng.random() < 0.5,
                 skew=rng.random() < 0.2)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(1_000_003 * int(seed) + salt)


def _weights(M, K, s, bits, skew, seed, salt=0):
    """Masked INT4 (or 2-bit) weights, int8 (M, K) on the GPU; zero means pruned."""
    g = _gen(seed, 10 + salt)
    keep = 1.0 - s
    if skew:   # keep rate per row ~ Beta(2, 3) rescaled to the mean
        p = np.random.default_rng([int(seed), salt]).beta(2.0, 3.0, size=M)
        keep = torch.from_numpy(np.clip(p * (keep / p.mean()), 0.0, 1.0).astype(np.float32)).cuda()[:, None]
    if bits == 4:      # uniform over {-8..-1, 1..7}
        v = torch.randint(-8, 7, (M, K), dtype=torch.int8, device="cuda", generator=g)
        v += (v >= 0).to(torch.int8)
    else:              # uniform over {-2, -1, 1}
        v = torch.randint(-2, 1, (M, K), dtype=torch.int8, device="cuda", generator=g)
        v += (v >= 0).to(torch.int8)
    return v.mul_(torch.rand((M, K), device="cuda", generator=g) < keep)


def _activations(N, K, seed, salt=0):
    return torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda", generator=_gen(seed, 20 + salt))


def _pack(xt):
    """binding.pack_int4's layout: even k in the low nibble."""
    u = xt.view(torch.uint8) & 0xF
    return (u[:, 0::2] | (u[:, 1::2] << 4)).contiguous()


def _scales(M, seed, salt=0):
    return 0.01 + 0.09 * torch.rand(M, device="cuda", generator=_gen(seed, 30 + salt))


def _projection(M, K, N, s, seed, bits=4, reorder=False, dequant=False, skew=False, salt=0):
    enc = binding.encode(_weights(M, K, s, bits, skew, seed, salt).cpu().numpy(), reorder=reorder, bits=bits)
    p = {"w": binding.to_device(enc), "x": _pack(_activations(N, K, seed, salt)), "N": N,
         "y": torch.empty((N, M), dtype=torch.int32, device="cuda"), "scale": None, "yf": None}
    enc.free()
    if dequant:
        p["scale"] = _scales(M, seed, salt)
        p["yf"] = torch.empty((N, M), dtype=torch.float32, device="cuda")
    return p


def _layer_shapes(c):
    h, f = c["hidden"], c["ffn"]
    return [(3 * h, h), (f, h), (f, h), (h, f)]


def _call(p):
    binding.spmm(p["w"], p["x"], p["N"], p["y"], p["scale"], p["yf"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "spmm":
        return {"kind": kind, "p": _projection(case["M"], case["K"], case["N"], case["sparsity"], seed, case["bits"],
                                               case["reorder"], case["dequant"], case["skew"])}
    if kind == "layer":
        ps = [_projection(M, K, case["N"], case["sparsity"], seed, dequant=True, salt=100 * i)
              for i, (M, K) in enumerate(_layer_shapes(case))]
        for p in ps:                       # each shape runs once before the capture
            _call(p)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for p in ps:
                _call(p)
        return {"kind": kind, "ps": ps, "graph": graph}
    if kind == "gemm":
        M, K, N = case["M"], case["K"], case["N"]
        g = _gen(seed)
        return {"kind": kind, "M": M, "K": K, "N": N,
                "w": torch.randint(-128, 128, (M, K), dtype=torch.int8, device="cuda", generator=g),
                "x": torch.randint(-128, 128, (N, K), dtype=torch.int8, device="cuda", generator=g),
                "y": torch.empty((N, M), dtype=torch.int32, device="cuda")}
    # The payload's length follows from the mask: the tiles of one mask in
    # another order for each seed, so that every seed's arrays have one shape.
    M, K = case["M"], case["K"]
    mask = _weights(M, K, case["sparsity"], case["bits"], False, 0) != 0
    g = _gen(seed, 40)
    rb = torch.randperm(M // 16, device="cuda", generator=g)
    kb = torch.randperm(K // 64, device="cuda", generator=g)
    mask = mask.view(M // 16, 16, K // 64, 64)[rb][:, :, kb].reshape(M, K)
    w = _weights(M, K, 0.0, case["bits"], False, seed).mul_(mask)
    return {"kind": kind, "w": w.cpu().numpy(), "bits": case["bits"], "reorder": case["reorder"]}


def run(state):
    kind = state["kind"]
    if kind == "spmm":
        p = state["p"]
        _call(p)
        return p["y"] if p["yf"] is None else (p["y"], p["yf"])
    if kind == "layer":
        state["graph"].replay()
        return [(p["y"], p["yf"]) for p in state["ps"]]
    if kind == "gemm":
        binding.gemm_i8(state["w"], state["x"], state["M"], state["K"], state["N"], state["y"])
        return state["y"]
    dev = binding.to_device(binding.encode(state["w"], reorder=state["reorder"], bits=state["bits"]))
    out = [dev.bitmaps, dev.offsets, dev.payload]
    return out if dev.perm is None else out + [dev.perm]


# ---------------------------------------------------------------------------
# Bytes, operations, accuracy
# ---------------------------------------------------------------------------

def _encoded_bytes(M, K, s, bits, reorder=False, skew=False):
    """Expected IE-BME bytes: four values per union-mask entry that any of the four areas activates
    (two rows, two columns each), 36 bytes of bitmaps and offsets per tile, 8 of permutation."""
    empty = s ** 4
    if skew:   # E[(1 - p)^2]^2 over two independent rows; exact for Beta(2, 3) at keep 0.4, close elsewhere
        q = (1.0 - s) / 0.4
        empty = (1.0 - 2 * q * 0.4 + q * q * 0.2) ** 2
    tiles = (M // 16) * (K // 64)
    return tiles * (36 + (8 if reorder else 0) + 1024 * (1.0 - empty) * bits / 8)


def _spmm_bytes(M, K, N, s, bits=4, reorder=False, dequant=False, skew=False):
    b = _encoded_bytes(M, K, s, bits, reorder, skew) + K * N / 2 + 4 * M * N
    return b + (4 * M + 4 * M * N if dequant else 0)


def work(case):
    kind = case["kind"]
    if kind == "layer":
        N, s = case["N"], case["sparsity"]
        shapes = _layer_shapes(case)
        return {"bytes": sum(_spmm_bytes(M, K, N, s, dequant=True) for M, K in shapes),
                "flops": sum(2.0 * M * K * (1 - s) * N for M, K in shapes)}
    M, K = case["M"], case["K"]
    if kind == "spmm":
        return {"bytes": _spmm_bytes(M, K, case["N"], case["sparsity"], case["bits"], case["reorder"],
                                     case["dequant"], case["skew"]),
                "flops": 2.0 * M * K * (1 - case["sparsity"]) * case["N"]}
    if kind == "gemm":
        N = case["N"]
        return {"bytes": float(M * K + K * N + 4 * M * N), "flops": 2.0 * M * K * N}
    return {"bytes": M * K + _encoded_bytes(M, K, case["sparsity"], case["bits"], case["reorder"]), "flops": 0.0}


def tolerance(case):
    # INT32 sums are exact in any order, the dequantised outputs are one
    # rounding of each sum and one of its product with the scale, and the
    # encoding is a fixed format: any correct implementation gives these bits.
    return "exact"


def _exact_product(W, xt, scale):
    y = (xt.double() @ W.double().t())
    yi = y.round().to(torch.int64)
    return yi if scale is None else (yi, y * scale.double())


def exact(case, seed):
    kind = case["kind"]
    if kind == "encode":
        return None                        # bytes of a format, not computed numbers
    if kind == "gemm":
        st = prepare(case, seed)
        return _exact_product(st["w"], st["x"], None)
    if kind == "layer":
        out = []
        for i, (M, K) in enumerate(_layer_shapes(case)):
            W = _weights(M, K, case["sparsity"], 4, False, seed, 100 * i)
            out.append(_exact_product(W, _activations(case["N"], K, seed, 100 * i), _scales(M, seed, 100 * i)))
        return out
    M, K = case["M"], case["K"]
    W = _weights(M, K, case["sparsity"], case["bits"], case["skew"], seed)
    scale = _scales(M, seed) if case["dequant"] else None
    return _exact_product(W, _activations(case["N"], K, seed), scale)
