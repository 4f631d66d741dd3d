"""The load streams of the product kernel, in every tile variant: sequences shorter than the lead of any stream, tiles
that end in each of its phases, one and several tiles per workgroup (every second one backwards), a ragged last
k-step, and column tiles walked side by side (also with a narrower last group).  The reference is the masked dense
product in fp64; accepted is what fp32 accumulation and one fp16 rounding allow (1e-2 of |A|.|B| elementwise, 1e-3 in norm)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2310_02065_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(R, K, C, V, M, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    A = torch.randn(R, K, dtype=torch.float16, device=DEV, generator=gen)
    B = torch.randn(K, C, dtype=torch.float16, device=DEV, generator=gen)
    mask, _, _ = binding.venom_prune(A, V, 2, M)
    kept = A.double() * mask
    return binding.venom_compress(A, mask, V, 2, M), B, kept @ B.double(), kept.abs() @ B.double().abs()


def check(out, want, bound, what):
    off = (out.double() - want).abs()
    assert bool((off <= 1e-2 * bound).all()), what
    assert float(off.norm()) <= 1e-3 * float(want.norm()), what


def variants(V, R=None, M=None):
    V = 128 if M == 4 and R % 128 == 0 else V
    return [(i, n) for i, n in enumerate(binding.venom_spmm_variants()) if n.startswith(f"v{V}_")]


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 13, 17, 33])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
def test_one_tile_per_workgroup(V, steps):
    M, C = 7, 584                                     # 512 + 72 columns
    R, K = 2 * V, (8 * steps - 3) * M
    h, B, want, bound = problem(R, K, C, V, M, seed=steps)
    for i, name in [(-1, "chosen")] + variants(V):
        check(binding.venom_spmm(h, B, variant=i), want, bound, (name, steps))


@pytest.mark.parametrize("steps", [1, 2, 3, 5, 6, 8, 12, 21])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
def test_several_tiles_per_workgroup(V, steps):
    M, C = 5, 40
    R, K = 1100 * V, (8 * steps - 5) * M              # 1100 tiles of any width: three to five per workgroup
    h, B, want, bound = problem(R, K, C, V, M, seed=100 + steps)
    for i, name in [(-1, "chosen")] + variants(V):
        check(binding.venom_spmm(h, B, variant=i), want, bound, (name, steps))


@pytest.mark.parametrize("R,K,C,V,M", [
    (8192, 1280, 192, 128, 4),                        # 64 x 3 tiles of 64 columns, 40 k-steps: groups of two, then one
    (16384, 1400, 248, 64, 5),                        # 256 x 4 tiles, two per workgroup
    (24576, 648, 520, 96, 4),                         # 192 row blocks of 128 x 9 tiles
])
def test_column_tiles_side_by_side(R, K, C, V, M):
    h, B, want, bound = problem(R, K, C, V, M, seed=R + C)
    for i, name in variants(V, R, M):
        check(binding.venom_spmm(h, B, variant=i), want, bound, name)
    again = binding.venom_spmm(h, B)
    check(again, want, bound, "chosen")
    assert torch.equal(again, binding.venom_spmm(h, B))   # bitwise repeatable
