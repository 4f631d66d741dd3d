"""The token-major output stage (16-byte and 8-byte stores of fp16, fp32) and the fused epilogue in every tile variant, also
those that the choice by expected time seldom or never takes for a layer: one and several tiles per workgroup, ragged
tokens, a ragged last k-step, column tiles side by side.  venom_linear takes no variant, so the variant is given to
the function behind it.  The reference is the masked dense product in fp64; accepted is what fp32
accumulation and one fp16 rounding allow (1e-2 of |A|.|B| + |bias| elementwise, stretched by GELU's largest slope 1.13, 1e-3
in norm)."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

from paper_2310_02065_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LAUNCH = "_ZN5venom11launch_spmmERK12venom_handlePKvllS4_iPvliiiP12ihipStream_t"     # venom::launch_spmm
ACTIVATE = {"none": lambda x: x, "gelu": torch.nn.functional.gelu,
            "gelu_tanh": lambda x: torch.nn.functional.gelu(x, approximate="tanh")}


def launch(h, B, bias, act, Y, variant):
    f = getattr(binding.lib(), LAUNCH)
    p, n, i = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
    f.argtypes, f.restype = [p, p, n, n, p, i, p, n, i, i, i, p], i
    return f(h.ptr, B.data_ptr(), B.stride(0), B.shape[1], bias.data_ptr(), binding.ACTIVATIONS[act], Y.data_ptr(), Y.stride(0),
             int(Y.dtype == torch.float32), 1, variant, torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("R,T,steps,M", [
    (2, 584, 1, 7), (2, 584, 4, 7), (2, 1096, 9, 7),  # one tile per workgroup: 512 + 72 tokens, twice 512 + 72
    (1100, 40, 3, 5),                                 # 1100 tiles of any width: three to five per workgroup
    (300, 200, 6, 5),                                 # 300 x 4 tiles of 64 tokens, ragged in all widths
    (96, 264, 40, 5),                                 # many k-steps: 64-token tiles side by side
])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
def test_token_major_output(V, R, T, steps, M):
    R, K = R * V, (8 * steps - 3) * M
    gen = torch.Generator(device=DEV)
    gen.manual_seed(R + steps)
    A = torch.randn(R, K, dtype=torch.float16, device=DEV, generator=gen)
    B = torch.randn(K, T, dtype=torch.float16, device=DEV, generator=gen)
    bias = torch.randn(R, dtype=torch.float16, device=DEV, generator=gen)
    mask, _, _ = binding.venom_prune(A, V, 2, M)
    h = binding.venom_compress(A, mask, V, 2, M)
    kept = A.double() * mask
    raw = B.double().t().contiguous() @ kept.t().contiguous() + bias.double()
    bound = 1.13 * (B.double().abs().t().contiguous() @ kept.abs().t().contiguous() + bias.double().abs())
    variants = [(i, n) for i, n in enumerate(binding.venom_spmm_variants()) if n.startswith(f"v{V}_")]
    for act in ACTIVATE:
        want = ACTIVATE[act](raw)
        for dtype, shift in ((torch.float16, 8), (torch.float16, 4), (torch.float32, 4)):
            for i, name in variants:
                big = torch.full((T, R + 16), -7.0, dtype=dtype, device=DEV)
                Y = big[:, shift:shift + R]
                assert launch(h, B, bias, act, Y, i) == binding.VENOM_OK
                off = (Y.double() - want).abs()
                assert bool((off <= 1e-2 * bound).all()) and float(off.norm()) <= 1e-3 * float(want.norm()), (name, act, dtype, shift)
                assert bool((big[:, :shift] == -7.0).all()) and bool((big[:, shift + R:] == -7.0).all()), (name, act, dtype, shift)
    X = B.t().contiguous()
    got = binding.venom_linear(h, X, bias=bias, activation="gelu")          # the chosen one, transposition included
    assert float((got.double() - ACTIVATE["gelu"](raw)).norm()) <= 1e-3 * float(ACTIVATE["gelu"](raw).norm())
