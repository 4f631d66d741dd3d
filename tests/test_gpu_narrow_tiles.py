"""The 64-column tile against the oracle, chosen explicitly and by default: its edges in the columns (64 / 72), sizes on
both sides of one tile per unit (256 tiles / 260), one to three waves per strip, ragged last k-steps, several tiles per
workgroup (every second one runs its k-steps backwards), every output form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vnm_oracle as o
from paper_2310_02065_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("R,K,C,V,M", [
    (256, 1040, 8, 128, 16),          # 65 groups: nine k-steps, one group in the last; one piece of the tile's columns
    (256, 640, 64, 128, 16),          # exactly one tile
    (256, 640, 72, 128, 16),          # ... and a second one with 8 columns
    (576, 330, 200, 96, 10),          # three waves per strip, 33 groups
    (512, 56, 4096, 128, 7),          # one k-step, 4 x 64 = 256 tiles
    (512, 56, 4104, 128, 7),          # 260
    (64, 136, 56, 64, 8), (32, 4000, 16, 32, 100),
    (1100 * 64, 17 * 8, 16, 64, 8),   # 1100 tiles: two or three per workgroup; three k-steps, one group in the last
    (700 * 96, 9 * 10, 40, 96, 10),   # 700 tiles; two k-steps
])
def test_narrow_tile_matches_oracle(R, K, C, V, M):
    A, mask, B = inputs.gen_problem(R, K, C, V, M, 1.0, seed=R + K + C)
    bias = np.random.default_rng(C).standard_normal(R).astype(np.float16)
    h = binding.venom_compress(torch.from_numpy(A.view(np.float16)).to(DEV), torch.from_numpy(mask).to(DEV), V, 2, M)
    ov, oc, om = o.compress(A, mask, V, M)
    B_d, bias_d = torch.from_numpy(B.view(np.float16)).to(DEV), torch.from_numpy(bias).to(DEV)
    narrow = binding.venom_spmm_variants().index(f"v{V}_c64")
    Cs, E = o.spmm_fp64(ov, oc, om, R, K, V, M, B)
    Xt = np.ascontiguousarray(B.T)
    Ys, Ey = o.linear_fp64(ov, oc, om, R, K, V, M, Xt, bias.view(np.uint16), "gelu")
    for dt in (torch.float16, torch.float32):
        for var in (-1, narrow):
            big = torch.full((R, C + 16), -7.0, dtype=dt, device=DEV)
            binding.venom_spmm(h, B_d, out=big[:, 8:8 + C], variant=var)
            ok, info = o.accept(big[:, 8:8 + C].double().cpu().numpy(), Cs, E)
            assert ok, (dt, var, info)
            assert bool((big[:, :8] == -7.0).all()) and bool((big[:, 8 + C:] == -7.0).all())
            Z = binding.venom_spmm(h, B_d, out_dtype=dt, variant=var, bias=bias_d, activation="gelu")
            ok, info = o.accept(Z.t().double().cpu().numpy(), Ys, Ey)
            assert ok, (dt, var, info)
        X = torch.from_numpy(Xt.view(np.float16)).to(DEV)
        for shift in (0, 4):              # 16-byte stores through LDS, and 8-byte runs straight from the accumulators
            Y = torch.full((C, R + 12), -7.0, dtype=dt, device=DEV)
            binding.venom_linear(h, X, bias=bias_d, activation="gelu", out=Y[:, shift:shift + R])
            ok, info = o.accept(Y[:, shift:shift + R].double().cpu().numpy(), Ys, Ey)
            assert ok, (dt, shift, info)
            assert bool((Y[:, R + shift:] == -7.0).all()) and bool((Y[:, :shift] == -7.0).all())
