"""Edges of the format kernels' tilings against the oracle, bit for bit: several metadata words per workgroup with a
ragged last one, mask loads of both widths with columns left over, rows at every alignment, blocks too tall
for on-chip mask bits or for the pruning tile, odd M, groups per row that are no multiple of 4, block heights
that differ from the packed ones."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vnm_oracle as o
from paper_2310_02065_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("R,K,V,M,shift", [
    (16384, 33 * 8, 64, 8, 0),       # 256 block rows x 5 words of which the last has one group: one word per workgroup
    (65536, 17 * 8, 32, 8, 0),       # 2048 x 3: one workgroup takes all three words, the last with one group
    (16384, 45 * 8, 8, 8, 0),        # 2048 x 6: four words per workgroup, then two, the last with five groups
    (4096, 130 * 32, 32, 32, 0),     # 128 block rows x 17 words, two groups in the last one
    (192, 23 * 7, 96, 7, 0),         # odd M: 8-byte mask loads on rows of 161 bytes
    (128, 27 * 12, 64, 12, 8),       # 16-byte loads and four columns left over; mask rows on 4-byte boundaries
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


@pytest.mark.parametrize("R,K,V,M,lda,ldm", [
    (128, 9 * 4, 64, 4, 40, 48),     # the last word is narrower than a 16-byte load
    (128, 15 * 4, 64, 4, 64, 64),    # ... is one load and 12 columns
    (128, 9 * 5, 64, 5, 48, 56),     # ... narrower than the 8-byte loads of an odd chunk
    (96, 13 * 10, 32, 10, 136, 130), # two columns left over, of A too
    (96, 21 * 40, 32, 40, 840, 843), # K % 16 == 8
    (640, 9 * 6, 640, 6, 55, 55),    # a tall block: a pruning tile of 24 columns
    (1024, 9 * 64, 1024, 64, 579, 577),   # too tall for one: the general kernel, rows at any boundary
    (8192, 325 * 8, 1024, 8, 2600, 2600), # tiles of 8 columns against 328 workgroups of the general kernel: the latter
    (48, 11 * 100, 2, 100, 1104, 1100),   # blocks of few rows: tiles of ten groups, and one
])
def test_padded_rows_bit_exact(R, K, V, M, lda, ldm):
    rng = np.random.default_rng(R + K)
    bits = (rng.standard_normal((R, K)) * 0.05).astype(np.float16).view(np.uint16)
    A = torch.full((R, lda), 9.0, dtype=torch.float16, device=DEV)
    A[:, :K] = torch.from_numpy(bits.view(np.float16)).to(DEV)
    pmask, kept, total = binding.venom_prune(A[:, :K], V, 2, M)
    omask, okept, ototal = o.prune(bits, V, M)
    assert np.array_equal(pmask.cpu().numpy(), omask)
    assert sum(int(x) for x in kept.cpu().tolist()) == okept and sum(int(x) for x in total.cpu().tolist()) == ototal
    mask = np.where(rng.random((R, K)) < 0.2, 0, inputs.gen_mask(R, K, V, M, rng)).astype(np.uint8)
    wide = torch.full((R, ldm), 7, dtype=torch.uint8, device=DEV)
    wide[:, :K] = torch.from_numpy(mask * rng.integers(1, 256, (R, K)).astype(np.uint8)).to(DEV)
    h = binding.venom_compress(A[:, :K], wide[:, :K], V, 2, M)
    for got, w in zip(binding.venom_export(h), o.compress(bits, mask, V, M)):
        assert np.array_equal(got.cpu().numpy().view(w.dtype), w)


def test_two_words_per_workgroup():
    """The chunk of columns in between (2 words: mask bits of 4 would not fit) needs 107 million entries; the same block
    rows compressed by themselves take one word at a time."""
    V, M, G = 96, 64, 17
    R, K = 1024 * V, G * M
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    A = torch.randn(R, K, dtype=torch.float16, device=DEV, generator=gen)
    mask, _, _ = binding.venom_prune(A, V, 2, M)
    h = binding.venom_compress(A, mask, V, 2, M)
    whole = binding.venom_export(h)
    assert torch.equal(binding.venom_decompress(h), torch.where(mask != 0, A, 0))
    for b in (0, 511, 1023):
        rows = slice(b * V, (b + 1) * V)
        values, columns, meta = binding.venom_export(binding.venom_compress(A[rows], mask[rows], V, 2, M))
        assert torch.equal(whole[0][rows], values) and torch.equal(whole[1][b:b + 1], columns)
        assert torch.equal(whole[2][rows], meta)


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


@pytest.mark.parametrize("R,K,V,M", [(64, 5 * 8, 64, 8), (32, 1024 * 4, 32, 4), (96, 33 * 7, 96, 7), (9, 50 * 5, 1, 5)])
def test_export_at_any_address_and_in_part(R, K, V, M):
    rng = np.random.default_rng(R + K)
    mask = inputs.gen_mask(R, K, V, M, rng)
    A = rng.standard_normal((R, K)).astype(np.float16)
    h = binding.venom_compress(torch.from_numpy(A).to(DEV), torch.from_numpy(mask).to(DEV), V, 2, M)
    want = [torch.from_numpy(np.ascontiguousarray(x).view(np.uint8).reshape(-1)) for x in o.compress(A.view(np.uint16), mask, V, M)]
    for shifts in ((0, 0, 0), (2, 6, 4), (1, 3, 5)):
        for skip in (None, 0, 1, 2):
            bufs = [torch.full((w.numel() + 16,), 0xA5, dtype=torch.uint8, device=DEV) for w in want]
            ptrs = [None if k == skip else b.data_ptr() + s for k, (b, s) in enumerate(zip(bufs, shifts))]
            assert binding.lib().venom_export(h.ptr, *ptrs, None) == binding.VENOM_OK
            torch.cuda.synchronize()
            for k, (b, s, w) in enumerate(zip(bufs, shifts, want)):
                got = b.cpu()
                inside = got[s:s + w.numel()]
                assert bool((inside == 0xA5).all()) if k == skip else torch.equal(inside, w), (shifts, skip, k)
                assert bool((got[:s] == 0xA5).all()) and bool((got[s + w.numel():] == 0xA5).all())


def test_export_on_another_stream_and_in_a_graph():
    R, K, V, M = 64, 5 * 8, 64, 8
    rng = np.random.default_rng(3)
    mask = inputs.gen_mask(R, K, V, M, rng)
    A = rng.standard_normal((R, K)).astype(np.float16)
    h = binding.venom_compress(torch.from_numpy(A).to(DEV), torch.from_numpy(mask).to(DEV), V, 2, M)
    want = [torch.from_numpy(np.ascontiguousarray(x).view(np.uint8).reshape(-1)) for x in o.compress(A.view(np.uint16), mask, V, M)]
    bufs = [torch.zeros(w.numel(), dtype=torch.uint8, device=DEV) for w in want]
    ptrs = [b.data_ptr() for b in bufs]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    assert binding.lib().venom_export(h.ptr, *ptrs, side.cuda_stream) == binding.VENOM_OK
    side.synchronize()
    for b, w in zip(bufs, want):
        assert torch.equal(b.cpu(), w)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        st = binding.lib().venom_export(h.ptr, *ptrs, torch.cuda.current_stream().cuda_stream)
    assert st == binding.VENOM_OK
    for _ in range(3):
        for b in bufs:
            b.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for b, w in zip(bufs, want):
            assert torch.equal(b.cpu(), w)


@pytest.mark.parametrize("R,K,V,M", [(64, 5 * 8, 64, 8), (96, 33 * 7, 96, 7)])
def test_export_to_pinned_host_memory(R, K, V, M):
    # memory that is not on the handle's device, or only some of it: the runtime's copies
    rng = np.random.default_rng(R + K)
    mask = inputs.gen_mask(R, K, V, M, rng)
    A = rng.standard_normal((R, K)).astype(np.float16)
    h = binding.venom_compress(torch.from_numpy(A).to(DEV), torch.from_numpy(mask).to(DEV), V, 2, M)
    want = [torch.from_numpy(np.ascontiguousarray(x).view(np.uint8).reshape(-1)) for x in o.compress(A.view(np.uint16), mask, V, M)]
    for where in ((1, 1, 1), (0, 1, 0), (1, 0, 0), (0, 0, 1)):
        bufs = [torch.empty(w.numel() + 16, dtype=torch.uint8, pin_memory=True).fill_(0xA5) if host else
                torch.full((w.numel() + 16,), 0xA5, dtype=torch.uint8, device=DEV) for host, w in zip(where, want)]
        torch.cuda.synchronize()
        assert binding.lib().venom_export(h.ptr, *(b.data_ptr() for b in bufs), None) == binding.VENOM_OK
        torch.cuda.synchronize()
        for b, w in zip(bufs, want):
            got = b.cpu()
            assert torch.equal(got[:w.numel()], w) and bool((got[w.numel():] == 0xA5).all()), where
