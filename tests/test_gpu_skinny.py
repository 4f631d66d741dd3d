"""Products with at most 32 columns and layers with at most 32 tokens against the oracle, in the form that is chosen for them (each form
by itself, with longer reductions: tests/test_gpu_few_columns_forms.py): single tiles, whole block rows, pairs of them (an odd number,
too), X read in place or transposed first, fewer k-steps than waves, a last k-step with some of its groups, rows of X that end
inside a 16-byte piece or start at any address."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vnm_oracle as o
from paper_2310_02065_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(R, K, C, V, M):
    A, mask, B = inputs.gen_problem(R, K, C, V, M, 1.0, seed=R + K + C)
    h = binding.venom_compress(torch.from_numpy(A.view(np.float16)).to(DEV), torch.from_numpy(mask).to(DEV), V, 2, M)
    return h, o.compress(A, mask, V, M), B, np.random.default_rng(C).standard_normal(R).astype(np.float16)


@pytest.mark.parametrize("R,K,C,V,M", [
    (128, 16, 8, 128, 16),            # one group in all
    (96, 7 * 33, 24, 96, 7),          # odd rows, five k-steps, one group in the last; a wave has none
    (64, 8 * 64, 32, 64, 8),          # eight k-steps, all whole: one for each wave
    (32, 10 * 77, 16, 32, 10),        # ten k-steps: two waves have a second one
    (256, 32 * 100, 32, 128, 32),     # 1024 pieces of X, the most that can be staged; transposed first
    (256, 32 * 24, 16, 128, 32),      # 512: the most of the smaller staging, 8 a lane
    (192, 100 * 12, 8, 64, 100), (192, 100 * 12, 16, 64, 100),   # 800; 1600: transposed first
    (10240 + 128, 4 * 50, 32, 128, 4),                # 81 block rows of 128, 324 tiles: by pairs, a half one at the end
    (9600 + 96, 10 * 30, 16, 96, 10),                 # 101 of 96, ragged
    (9600 + 64, 20 * 40, 32, 64, 20),                 # 151 of 64, 640 pieces: transposed first, then whole block rows
    (9600 + 32, 16 * 9, 24, 32, 16),                  # 301 of 32
    (26 * 1024, 7 * 20, 8, 128, 7),                   # 208 of 128: the product stays with the 64-column tile, the layer goes by pairs
])
def test_few_columns_match_oracle(R, K, C, V, M):
    h, (ov, oc, om), B, bias = problem(R, K, C, V, M)
    B_d, bias_d = torch.from_numpy(B.view(np.float16)).to(DEV), torch.from_numpy(bias).to(DEV)
    Xt = np.ascontiguousarray(B.T)
    Cs, E = o.spmm_fp64(ov, oc, om, R, K, V, M, B)
    Ys, Ey = o.linear_fp64(ov, oc, om, R, K, V, M, Xt, bias.view(np.uint16), "gelu")
    for dt in (torch.float16, torch.float32):
        big = torch.full((R, C + 16), -7.0, dtype=dt, device=DEV)
        binding.venom_spmm(h, B_d, out=big[:, 8:8 + C])
        ok, info = o.accept(big[:, 8:8 + C].double().cpu().numpy(), Cs, E)
        assert ok, (dt, info)
        assert bool((big[:, :8] == -7.0).all()) and bool((big[:, 8 + C:] == -7.0).all())
        for shift, gap in ((0, 0), (4, 1)):           # X at any 2-byte address, with an odd row pitch; Y on 8-byte runs
            Xb = torch.zeros((C, K + gap), dtype=torch.float16, device=DEV)
            X = Xb[:, gap:]
            X.copy_(torch.from_numpy(Xt.view(np.float16)))
            Y = torch.full((C, R + 12), -7.0, dtype=dt, device=DEV)
            binding.venom_linear(h, X, bias=bias_d, activation="gelu", out=Y[:, shift:shift + R])
            ok, info = o.accept(Y[:, shift:shift + R].double().cpu().numpy(), Ys, Ey)
            assert ok, (dt, shift, info)
            assert bool((Y[:, R + shift:] == -7.0).all()) and bool((Y[:, :shift] == -7.0).all())


@pytest.mark.parametrize("R,K,C,V,M", [(128, 16 * 11, 16, 128, 16), (10240 + 128, 16 * 11, 16, 128, 16), (64, 100 * 9, 16, 64, 100)])
def test_infinities_stay_with_the_rows_that_are_selected(R, K, C, V, M):
    # B has Inf in row 0, to which the groups past the end of the last k-step point, and NaN in another row; blocks that select
    # neither have finite results, and the same ones as without them
    h, (ov, oc, om), B, _ = problem(R, K, C, V, M)
    Bf = torch.from_numpy(B.view(np.float16)).to(DEV)
    bad = Bf.clone()
    bad[0] = float("inf")
    bad[K - 1] = float("nan")
    oc = oc.reshape(R // V, K // M, 4)
    clean = ~((oc[:, 0] == 0).any(1) | (oc[:, -1] == M - 1).any(1))
    rows = torch.from_numpy(np.repeat(clean, V)).to(DEV)
    want, got = binding.venom_spmm(h, Bf), binding.venom_spmm(h, bad)
    assert torch.equal(got[rows], want[rows])
    assert torch.equal(binding.venom_linear(h, bad.t().contiguous()).t()[rows], binding.venom_linear(h, Bf.t().contiguous()).t()[rows])


def test_repeatable_and_under_capture():
    h, _, B, _ = problem(512, 1024, 16, 128, 16)
    X = torch.from_numpy(np.ascontiguousarray(B.T).view(np.float16)).to(DEV)
    scratch = torch.empty(1024 * 16 * 2, dtype=torch.uint8, device=DEV)
    want = binding.venom_linear(h, X, scratch=scratch)
    Y = torch.empty_like(want)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        binding.venom_linear(h, X, scratch=scratch, out=Y)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            binding.venom_linear(h, X, scratch=scratch, out=Y)
    for _ in range(3):
        Y.fill_(-7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
