"""Tiles whose barrier hands over two k-steps, against the oracle: one k-step in all, even and odd numbers of them, a last k-step with
some of its groups in the first and in the second half of its stage, and workgroups that walk two tiles, the second one backwards (so that
with an odd number its first stage holds the single k-step)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vnm_oracle as o
from paper_2310_02065_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("V", [32, 64, 96, 128])
@pytest.mark.parametrize("groups", [8, 16, 24, 13, 21, 72, 80, 76, 133])
def test_odd_and_even_stages_match_oracle(V, groups):
    M = 6
    R, K, C = 9 * V, groups * M, 64 * 64 - 8        # 9 x 64 narrow tiles: two for some of the workgroups of a full chip
    A, mask, B = inputs.gen_problem(R, K, C, V, M, 1.0, seed=groups + V)
    bias = np.random.default_rng(V).standard_normal(R).astype(np.float16)
    h = binding.venom_compress(torch.from_numpy(A.view(np.float16)).to(DEV), torch.from_numpy(mask).to(DEV), V, 2, M)
    ov, oc, om = o.compress(A, mask, V, M)
    B_d, bias_d = torch.from_numpy(B.view(np.float16)).to(DEV), torch.from_numpy(bias).to(DEV)
    Cs, E = o.spmm_fp64(ov, oc, om, R, K, V, M, B)
    names = binding.venom_spmm_variants()
    for name in (n for n in names if n.startswith(f"v{V}_c") and "512" not in n):
        out = binding.venom_spmm(h, B_d, variant=names.index(name), out_dtype=torch.float32, bias=bias_d)
        ok, info = o.accept((out - bias_d.float()[:, None]).double().cpu().numpy(), Cs, E + np.abs(bias.astype(np.float64))[:, None])
        assert ok, (name, info)
        plain = binding.venom_spmm(h, B_d, variant=names.index(name))
        ok, info = o.accept(plain.double().cpu().numpy(), Cs, E)
        assert ok, (name, info)
