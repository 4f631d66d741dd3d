"""The kernel for at most 32 columns, each form by itself whatever the choice would be: products by whole block rows and by single tiles,
layers that read X in place by single tiles and by pairs of block rows, 8 and 16 pieces of X a lane, one to four tiles per block row, an
odd number of block rows.  The reductions are long enough for the waves' loops: single tiles deal their k-steps to 8 waves, the others to
4, and a wave goes through 1 to 10 of them, as many as others or one fewer, with and without a ragged last k-step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ctypes import c_bool, c_int, c_int64, c_void_p

from library_internals import PAIR, SPLIT, WHOLE, inner
from oracle import vnm_oracle as o
from paper_2310_02065_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GROUPS = [8 * 9, 8 * 14 + 3, 8 * 17 + 7, 8 * 24, 8 * 27 + 1, 8 * 31, 8 * 40 + 5]   # 9, 14, ... whole k-steps


def launch(h, form, src, bias, act, out, in_place, token_major):
    f = inner("_ZN5venom13launch_skinnyERK12venom_handleiPKvllS4_iPvlibbP12ihipStream_t", c_int, c_void_p, c_int, c_void_p, c_int64, c_int64,
              c_void_p, c_int, c_void_p, c_int64, c_int, c_bool, c_bool, c_void_p)
    cols = src.shape[0] if in_place else src.shape[1]
    return f(h.ptr, form, src.data_ptr(), src.stride(0), cols, bias.data_ptr(), binding.ACTIVATIONS[act], out.data_ptr(), out.stride(0),
             int(out.dtype == torch.float32), in_place, token_major, torch.cuda.current_stream().cuda_stream)


def problem(V, M, C, groups):
    R, K = 3 * V, groups * M
    A, mask, B = inputs.gen_problem(R, K, C, V, M, 1.0, seed=groups + V + C)
    bias = np.random.default_rng(C).standard_normal(R).astype(np.float16)
    h = binding.venom_compress(torch.from_numpy(A.view(np.float16)).to(DEV), torch.from_numpy(mask).to(DEV), V, 2, M)
    want = o.linear_fp64(*o.compress(A, mask, V, M), R, K, V, M, np.ascontiguousarray(B.T), bias.view(np.uint16), "gelu")
    return h, torch.from_numpy(B.view(np.float16)).to(DEV), torch.from_numpy(bias).to(DEV), want


@pytest.mark.parametrize("groups", GROUPS)
@pytest.mark.parametrize("M,C", [(7, 24), (20, 32)])             # 8 pieces (168 of 512), 16 (640 of 1024)
@pytest.mark.parametrize("form", [SPLIT, PAIR])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
def test_layer_from_x_in_place(V, form, M, C, groups):
    h, B, bias, (Ys, Ey) = problem(V, M, C, groups)
    X = torch.zeros((C, h.K + 3), dtype=torch.float16, device=DEV)[:, 3:]          # rows at any 2-byte address
    X.copy_(B.t())
    for dtype in (torch.float16, torch.float32):
        Y = torch.full((C, h.R + 8), -7.0, dtype=dtype, device=DEV)
        assert launch(h, form, X, bias, "gelu", Y[:, 4:4 + h.R], True, True) == binding.VENOM_OK
        ok, info = o.accept(Y[:, 4:4 + h.R].double().cpu().numpy(), Ys, Ey)
        assert ok, (dtype, info)
        assert bool((Y[:, :4] == -7.0).all()) and bool((Y[:, 4 + h.R:] == -7.0).all())


@pytest.mark.parametrize("groups", GROUPS)
@pytest.mark.parametrize("form", [WHOLE, SPLIT])
@pytest.mark.parametrize("V,C", [(32, 32), (64, 8), (96, 24), (128, 16)])
def test_product(V, C, form, groups):
    h, B, bias, (Ys, Ey) = problem(V, 5, C, groups)
    for dtype in (torch.float16, torch.float32):
        for token_major in (False, True):                       # a product, and a layer whose X was transposed first
            shape = (C, h.R + 8) if token_major else (h.R, C + 8)
            big = torch.full(shape, -7.0, dtype=dtype, device=DEV)
            out = big[:, :shape[1] - 8]
            assert launch(h, form, B, bias, "gelu", out, False, token_major) == binding.VENOM_OK
            ok, info = o.accept((out if token_major else out.t()).double().cpu().numpy(), Ys, Ey)
            assert ok, (dtype, token_major, info)
            assert bool((big[:, shape[1] - 8:] == -7.0).all())


def test_a_form_that_does_not_serve_is_refused():
    h, B, bias, _ = problem(32, 40, 32, 8)                        # 1280 pieces of X
    X, Y = B.t().contiguous(), torch.empty((32, h.R), dtype=torch.float16, device=DEV)
    for form, src, in_place in ((SPLIT, X, True), (WHOLE, X[:8], True), (PAIR, B, False), (-1, B, False)):
        assert launch(h, form, src, bias, "gelu", Y, in_place, True) == binding.VENOM_ERR_UNSUPPORTED
