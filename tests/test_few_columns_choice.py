"""Which layers of few tokens are read in place: asked of the library on the host, no GPU needed."""
import pytest

from library_internals import host_handle, layer_reads_in_place

X0 = 1 << 32


@pytest.mark.parametrize("R,K,V,M", [(1024, 1024, 64, 16), (9664, 800, 64, 20)])   # single tiles; pairs of block rows
@pytest.mark.parametrize("tokens", [8, 16, 32])
@pytest.mark.parametrize("dtype,size", [(0, 2), (1, 4)])
def test_an_output_over_the_activations_is_not_written_while_they_are_read(R, K, V, M, tokens, dtype, size):
    h = host_handle(R, K, V, M)
    ldx, ldy = K + 6, R + 12
    x_bytes, y_bytes = 2 * ((tokens - 1) * ldx + K), size * ((tokens - 1) * ldy + R)

    def in_place(y):
        return layer_reads_in_place(h, X0, ldx, tokens, y, ldy, dtype)

    assert in_place(X0 + x_bytes) and in_place(X0 - y_bytes)                       # end to end
    for y in (X0, X0 + x_bytes - 2, X0 - y_bytes + 2, X0 + x_bytes // 2, X0 - y_bytes // 2):
        assert not in_place(y), y - X0


def test_more_rows_than_a_launch_has_threads_for_are_transposed_first():
    # 2^31 rows, 2^24 packed block rows: pairs of them, 512 threads each, are 2^32
    assert not layer_reads_in_place(host_handle(1 << 31, 36, 1 << 16, 4), X0, 36, 8, X0 << 8, 1 << 31)
