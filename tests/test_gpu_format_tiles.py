"""Edges of the format kernels' tilings against the oracle, bit for bit: several metadata words per workgroup with a
ragged last one, mask loads of every width, blocks too tall for on-chip mask bits or for the pruning
tile, odd M, groups per row that are no multiple of 4, block heights that differ from the packed ones."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vnm_oracle as o
from paper_2310_02065_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("R,K,V,M,shift", [
    (16384, 33 * 8, 64, 8, 0),       # 256 block rows x 5 words: several words per workgroup, the last with one group
    (4096, 130 * 32, 32, 32, 0),     # 128 block rows x 17 words, two groups in the last one
    (192, 23 * 7, 96, 7, 0),         # odd M: 8-byte mask loads on rows of 161 bytes are not allowed
    (128, 27 * 12, 64, 12, 8),       # mask rows on 8-byte boundaries only
    (128, 27 * 12, 64, 12, 3),       # ... on none
    (1024, 8 * 64, 1024, 64, 0),     # the mask bits of a block do not fit LDS
    (2304, 64, 2304, 8, 0),          # taller than the pruning tile serves
    (64, 2048, 32, 1024, 0),         # widest groups
    (384, 25 * 4, 192, 4, 0),        # M = 4: packed blocks of 128 rows straddle the canonical ones
    (9, 50 * 5, 1, 5, 0),            # single-row blocks
])
def test_format_path_bit_exact(R, K, V, M, shift):
    rng = np.random.default_rng(R + K + shift)
    A = (rng.standard_normal((R, K)) * 0.05).astype(np.float16)
    bits = A.view(np.uint16)
    A_d = torch.from_numpy(A).to(DEV)
    pmask, kept, total = binding.venom_prune(A_d, V, 2, M)
    omask, okept, ototal = o.prune(bits, V, M)
    assert np.array_equal(pmask.cpu().numpy(), omask)
    assert sum(int(x) for x in kept.cpu().tolist()) == okept and sum(int(x) for x in total.cpu().tolist()) == ototal

    mask = inputs.gen_mask(R, K, V, M, rng)
    mask = np.where(rng.random((R, K)) < 0.2, 0, mask).astype(np.uint8)           # under-full rows and blocks too
    wide = torch.full((R, K + 24), 7, dtype=torch.uint8, device=DEV)              # any non-zero byte means "kept"
    wide[:, shift:shift + K] = torch.from_numpy(np.where(mask, rng.integers(1, 256, (R, K)), 0).astype(np.uint8)).to(DEV)
    want = o.compress(bits, mask, V, M)
    h = binding.venom_compress(A_d, wide[:, shift:shift + K] if shift else torch.from_numpy(mask).to(DEV), V, 2, M)
    arrays = binding.venom_export(h)
    for got, w in zip(arrays, want):
        assert np.array_equal(got.cpu().numpy().view(w.dtype), w)
    h2 = binding.venom_import(*arrays, R, K, V, 2, M)
    for got, w in zip(binding.venom_export(h2), want):
        assert np.array_equal(got.cpu().numpy().view(w.dtype), w)
    if V % 32 == 0 and V <= 128 or M == 4 and R % 128 == 0:
        dense = torch.from_numpy(np.where(mask != 0, bits, 0).view(np.float16)).to(DEV)
        for x in (h, h2):
            assert torch.equal(binding.venom_decompress(x).view(torch.int16), dense.view(torch.int16))
            big = torch.full((R, K + 5), -7.0, dtype=torch.float16, device=DEV)   # rows on 2-byte boundaries
            binding.venom_decompress(x, out=big[:, 3:3 + K])
            assert torch.equal(big[:, 3:3 + K].contiguous().view(torch.int16), dense.view(torch.int16))
            assert bool((big[:, :3] == -7.0).all()) and bool((big[:, 3 + K:] == -7.0).all())


@pytest.mark.parametrize("R,K,V,M,offset", [
    (256, 72 * 8, 64, 8, 2), (256, 71 * 7, 32, 7, 6),     # arrays that begin in the middle of a word
    (256, 71 * 7, 32, 7, 0), (1024, 71 * 7, 1, 7, 4),     # groups per row that are no multiple of 4; single-row blocks
])
def test_import_of_arrays_at_any_address(R, K, V, M, offset):
    rng = np.random.default_rng(R + K)
    bits = (rng.standard_normal((R, K)) * 0.05).astype(np.float16).view(np.uint16)
    want = o.compress(bits, inputs.gen_mask(R, K, V, M, rng), V, M)
    moved = []
    for w in want:
        buf = torch.zeros(w.nbytes + 16, dtype=torch.uint8, device=DEV)
        buf[offset:offset + w.nbytes] = torch.from_numpy(np.frombuffer(w.tobytes(), np.uint8).copy()).to(DEV)
        moved.append(buf[offset:])
    for got, w in zip(binding.venom_export(binding.venom_import(*moved, R, K, V, 2, M)), want):
        assert np.array_equal(got.cpu().numpy().view(w.dtype), w)
