"""venom_import where a workgroup takes all tiles of a packed block row (768 workgroups or more, fewer than 2^24 groups from three
tiles on, packed blocks the same as the canonical ones) and where it takes one: the canonical
arrays come back, the packed copies expand to the masked matrix, and a fault in the last row and group is refused."""
import pytest

torch = pytest.importorskip("torch")

from paper_2310_02065_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("R,K,V,M", [
    (64 * 128, 1890, 64, 10),        # two tiles, 24 words of which the last has five groups: 768 workgroups
    (64 * 127, 1890, 64, 10),        # 762: split
    (96 * 110, 7 * 220, 96, 7),      # three tiles, 770; the last words of a row are half a workgroup's
    (128 * 100, 16 * 250, 128, 16),  # four
    (128 * 3, 16 * 9, 128, 16),      # ... split
    (128 * 8192, 128, 128, 8), (128 * 8191, 128, 128, 8),   # 2^24 groups: split, and one block row less: whole
    (128 * 100, 1000, 128, 4),       # M = 4: whole
    (256 * 50, 1000, 256, 4), (32 * 400, 1000, 32, 4),   # ... split: packed blocks of 128 rows under blocks of 256 and of 32
    (256 * 3, 1000, 256, 4), (32 * 12, 1000, 32, 4),
])
def test_import_packs_whole_block_rows_and_tiles(R, K, V, M):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(R + K)
    A = torch.randn(R, K, dtype=torch.float16, device=DEV, generator=gen)
    mask, _, _ = binding.venom_prune(A, V, 2, M)
    arrays = binding.venom_export(binding.venom_compress(A, mask, V, 2, M))
    h = binding.venom_import(*arrays, R, K, V, 2, M)
    for got, want in zip(binding.venom_export(h), arrays):
        assert torch.equal(got, want)
    assert torch.equal(binding.venom_decompress(h), A * mask)
    values, columns, meta = (a.clone() for a in arrays)
    meta[-1, -1] |= 0xf << (4 * ((K // M - 1) % 8)) if (K // M) % 8 else -(1 << 28)   # both m-indices 3
    with pytest.raises(binding.VenomError) as e:
        binding.venom_import(values, columns, meta, R, K, V, 2, M)
    assert e.value.status == binding.VENOM_ERR_INVALID_ARG
