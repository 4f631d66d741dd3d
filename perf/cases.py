"""The work a user of the library has it do, as cases that can be timed and compared: the product, the
linear layer, building a compressed layer from dense weights, and reading a stored one back.  Each case
is a dict of plain values; shapes come from the benchmark's configurations, the tests, or their ranges.
"""
import math

import torch

from paper_2310_02065_amd import binding
from paper_2310_02065_amd.inputs import CONFIGS

DEV = "cuda"

# ranges of draw(): what the configurations, the sparsity sweep, the column-loc ablation and the tests span
BLOCK_HEIGHTS = (32, 64, 64, 96, 128, 128, 128)
GROUPS = (4, 7, 8, 10, 16, 20, 32, 40, 64, 100, 128)
MAX_RK = CONFIGS["gpt3"][0] * CONFIGS["gpt3"][1]                       # dense elements of the largest weight
MAX_FLOPS = 4.0 * MAX_RK * CONFIGS["gpt3"][2] / CONFIGS["gpt3"][4]     # useful FLOP of the largest product
MAX_OUT = CONFIGS["bert_large"][0] * CONFIGS["bert_large"][2]          # elements of the largest output but one


def _product(name, kind, R, K, C, V, M, out="fp16", bias=False, act="none"):
    return {"name": name, "kind": kind, "R": R, "K": K, "C": C, "V": V, "M": M, "out": out, "bias": bias, "act": act}


def _config(name, kind, config, **more):
    R, K, C, V, M, _ = CONFIGS[config]
    return _product(name, kind, R, K, more.pop("C", C), V, M, **more)


def listed():
    return [
        # the smallest call: one layer-sized toy problem, where the launch and the host path are what counts
        _config("spmm_tiny", "spmm", "tiny"),
        # FFN-up of BERT-base over 4096 tokens: a short reduction (12 k-steps), medium output
        _config("spmm_bert_base", "spmm", "bert_base"),
        # FFN-up of BERT-large over 16384 tokens: the output is four fifths of the traffic
        _config("spmm_bert_large", "spmm", "bert_large"),
        # FFN-up of GPT-3 over 2048 tokens: the benchmark's headline, the largest product
        _config("spmm_gpt3", "spmm", "gpt3"),
        # the sparsity sweep's narrow end: few columns, as in small-batch inference
        _product("spmm_sweep_c256", "spmm", 8192, 8192, 256, 128, 16),
        # the sparsity sweep at V = 64, the less regular block height
        _product("spmm_sweep_v64", "spmm", 8192, 8192, 2048, 64, 8),
        # the column-loc ablation: eight block rows, a long reduction at high sparsity
        _product("spmm_ablation", "spmm", 1024, 16000, 4096, 128, 40),
        # nothing divides: V = 96, 35 block rows, 331 groups, ragged columns, bias, fp32 output
        _product("spmm_odd_fp32", "spmm", 3360, 3310, 1096, 96, 10, out="fp32", bias=True),
        # the linear layer in a prefill or training-sized batch, bias and GELU fused
        _config("linear_bert_large", "linear", "bert_large", bias=True, act="gelu"),
        # the linear layer while decoding: sixteen sequences, one token each
        _config("linear_decode", "linear", "gpt3", C=16, bias=True, act="gelu"),
        # building a sparse layer from dense weights for storage: prune, compress, export the arrays
        {"name": "encode_gpt3", "kind": "encode", "R": 49152, "K": 12288, "V": 128, "M": 32},
        # reading a stored layer back: import the arrays, expand to dense
        {"name": "decode_sweep", "kind": "decode", "R": 8192, "K": 8192, "V": 64, "M": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(("spmm", "spmm", "spmm", "linear", "linear", "encode", "decode"))
        V, M = rng.choice(BLOCK_HEIGHTS), rng.choice(GROUPS)
        R = max(V, _log_int(rng, 64, 49152) // V * V)
        K = max(M, _log_int(rng, 256, 16000) // M * M)
        if R * K > MAX_RK:
            continue
        case = {"kind": kind, "R": R, "K": K, "V": V, "M": M}
        if kind in ("encode", "decode"):
            return case
        C = max(8, _log_int(rng, 8, 16384) // 8 * 8)                  # the library takes multiples of 8
        if R * C > MAX_OUT or 4.0 * R * K * C / M > MAX_FLOPS:
            continue
        case.update(C=C, out=rng.choice(("fp16", "fp16", "fp16", "fp32")), bias=rng.random() < 0.5,
                    act=rng.choice(("none", "none", "gelu", "gelu_tanh")))
        if kind == "linear":
            case["bias"] = True
        return case


def prepare(case, seed):
    """Weights N(0, 0.02^2) pruned by magnitude, activations N(0, 1), a small bias: what a layer meets."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(*shape, scale=1.0):
        return torch.randn(*shape, dtype=torch.float16, device=DEV, generator=gen).mul_(scale)

    kind, R, K, V, M = (case[k] for k in ("kind", "R", "K", "V", "M"))
    W = normal(R, K, scale=0.02)
    state = {"case": dict(case)}
    if kind == "encode":
        state["W"] = W
        return state
    if kind == "decode":
        mask, _, _ = binding.venom_prune(W, V, 2, M)
        state["arrays"] = binding.venom_export(binding.venom_compress(W, mask, V, 2, M))
        return state
    bias = normal(R, scale=0.1) if case["bias"] else None
    if kind == "linear":
        state["layer"] = binding.Spmm.from_dense(W, bias, V, 2, M, case["act"])
        state["x"] = normal(case["C"], K)
        return state
    mask, _, _ = binding.venom_prune(W, V, 2, M)
    state["handle"] = binding.venom_compress(W, mask, V, 2, M)
    state["bias"] = bias
    state["B"] = normal(K, case["C"])
    state["out"] = torch.empty((R, case["C"]), dtype=_dtype(case), device=DEV)
    return state


def _dtype(case):
    return torch.float32 if case["out"] == "fp32" else torch.float16


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "spmm":
        return binding.venom_spmm(state["handle"], state["B"], out=state["out"], bias=state["bias"], activation=case["act"])
    if kind == "linear":
        return state["layer"](state["x"], out_dtype=_dtype(case))
    R, K, V, M = (case[k] for k in ("R", "K", "V", "M"))
    if kind == "encode":
        mask, kept, total = binding.venom_prune(state["W"], V, 2, M)
        return (mask, kept, total, *binding.venom_export(binding.venom_compress(state["W"], mask, V, 2, M)))
    return binding.venom_decompress(binding.venom_import(*state["arrays"], R, K, V, 2, M))


def work(case):
    R, K, V, M = (case[k] for k in ("R", "K", "V", "M"))
    G, blocks = K // M, R // V
    arrays = 4 * R * G + 4 * R * ((G + 7) // 8) + 8 * blocks * G      # values, index words, column ids
    if case["kind"] == "encode":
        return {"bytes": 2 * R * K + R * K + 16 * blocks + arrays, "flops": 0}
    if case["kind"] == "decode":
        return {"bytes": arrays + 2 * R * K, "flops": 0}
    rows = K * (1.0 - (1.0 - 4.0 / M) ** blocks)                      # rows of B that some block selects (expected)
    size = 4 if case["out"] == "fp32" else 2
    nbytes = arrays + 2 * rows * case["C"] + size * R * case["C"] + (2 * R if case["bias"] else 0)
    return {"bytes": nbytes, "flops": 4.0 * R * case["C"] * K / M}


def tolerance(case):
    """The format's arrays are whole numbers and bits.  The products were compared with the same product in 64 bits
    (26 shapes of the ranges above): fp16 outputs are 2.1e-4 off in norm and at most 4.9e-4 elementwise (half a unit
    in the last place), fp32 outputs 2.1e-7 and 1.0e-6, more where a reduction is longer."""
    if case["kind"] in ("encode", "decode"):
        return "exact"
    if case["out"] == "fp32":
        return {"rel": 2e-6, "max": 1e-5}
    return {"rel": 8e-4, "max": 2e-3}
