"""Layers whose output lies over their input, wholly or in part, against the oracle: of few tokens (which would be read in place
otherwise, by single tiles or by pairs of block rows) and of more."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vnm_oracle as o
from paper_2310_02065_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(R, K, V, M, T):
    A, mask, _ = inputs.gen_problem(R, K, 8, V, M, 1.0, seed=R + K + T)
    X = np.random.default_rng(T).standard_normal((T, K)).astype(np.float16)
    bias = np.random.default_rng(R).standard_normal(R).astype(np.float16)
    args = (torch.from_numpy(A.view(np.float16)).to(DEV), torch.from_numpy(mask).to(DEV))
    want = o.linear_fp64(*o.compress(A, mask, V, M), R, K, V, M, X.view(np.uint16), bias.view(np.uint16), "gelu")
    return args, torch.from_numpy(X).to(DEV), torch.from_numpy(bias).to(DEV), want


@pytest.mark.parametrize("T", [8, 16, 32, 40])
@pytest.mark.parametrize("R,V,M", [(1024, 64, 16), (192, 96, 8), (2048, 128, 32)])
def test_the_output_takes_the_input_s_place(R, V, M, T):
    (A, mask), X, bias, (Ys, Ey) = problem(R, R, V, M, T)
    layer = binding.Spmm(A, mask, bias, V, 2, M, "gelu")
    for call in (lambda x: layer(x, out=x), lambda x: binding.venom_linear(layer.handle, x, bias=bias, activation="gelu", out=x),
                 lambda x: binding.venom_linear_static(layer.handle, x, x, bias=bias, activation="gelu")):
        x = X.clone()
        assert call(x).data_ptr() == x.data_ptr()
        ok, info = o.accept(x.double().cpu().numpy(), Ys, Ey)
        assert ok, info


@pytest.mark.parametrize("T", [8, 32, 40])
def test_input_and_output_share_the_rows_of_one_buffer(T):
    R, K, V, M = 1024, 512, 64, 16
    (A, mask), X, bias, (Ys, Ey) = problem(R, K, V, M, T)
    h = binding.venom_compress(A, mask, V, 2, M)
    for x_at, y_at in ((0, K), (R, 0)):
        both = torch.full((T, K + R + 4), -7.0, dtype=torch.float16, device=DEV)
        x, y = both[:, x_at:x_at + K], both[:, y_at:y_at + R]
        x.copy_(X)
        binding.venom_linear(h, x, bias=bias, activation="gelu", out=y)
        ok, info = o.accept(y.double().cpu().numpy(), Ys, Ey)
        assert ok and torch.equal(x, X) and bool((both[:, K + R:] == -7.0).all()), info


@pytest.mark.parametrize("T", [8, 32, 40])
@pytest.mark.parametrize("R,K,V,M", [(1024, 512, 64, 16), (9664, 800, 64, 16)])
def test_the_input_is_a_part_of_the_output(R, K, V, M, T):
    (A, mask), X, bias, (Ys, Ey) = problem(R, K, V, M, T)
    h = binding.venom_compress(A, mask, V, 2, M)
    for dtype, at in ((torch.float16, 0), (torch.float16, R - K), (torch.float32, R)):
        Y = torch.zeros((T, R), dtype=dtype, device=DEV)
        x = Y.view(torch.float16)[:, at:at + K]
        x.copy_(X)
        binding.venom_linear(h, x, bias=bias, activation="gelu", out=Y)
        ok, info = o.accept(Y.double().cpu().numpy(), Ys, Ey)
        assert ok, (dtype, at, info)
