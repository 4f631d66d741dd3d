"""How layers of few tokens are served: asked of the library on the host, no GPU needed."""
import pytest

from library_internals import NONE, PAIR, SPLIT, host_handle, layer_form

X0 = 1 << 32


@pytest.mark.parametrize("R,K,V,M,form", [(1024, 1024, 64, 16, SPLIT), (9664, 800, 64, 16, PAIR)])
@pytest.mark.parametrize("tokens", [8, 16, 32])
@pytest.mark.parametrize("dtype,size", [(0, 2), (1, 4)])
def test_an_output_over_the_activations_is_not_written_while_they_are_read(R, K, V, M, form, tokens, dtype, size):
    h = host_handle(R, K, V, M)
    ldx, ldy = K + 6, R + 12
    x_bytes, y_bytes = 2 * ((tokens - 1) * ldx + K), size * ((tokens - 1) * ldy + R)

    def served(y):
        return layer_form(h, X0, ldx, tokens, y, ldy, dtype)

    assert served(X0 + x_bytes) == form and served(X0 - y_bytes) == form           # end to end: X is read in place
    for y in (X0, X0 + x_bytes - 2, X0 - y_bytes + 2, X0 + x_bytes // 2, X0 - y_bytes // 2):
        assert served(y) == NONE, y - X0


@pytest.mark.parametrize("dtype,size", [(0, 2), (1, 4)])
def test_side_by_side_in_the_rows_of_one_buffer_they_do_not_meet(dtype, size):
    R, K, tokens = 1024, 512, 16
    h, pitch = host_handle(R, K, 64, 16), 2 * K + size * R + 64

    def served(x, y):
        return layer_form(h, x, pitch // 2, tokens, y, pitch // size, dtype)

    for x, y in ((X0, X0 + 2 * K), (X0, X0 + 2 * K + 64), (X0 + size * R, X0), (X0 + size * R + 64, X0)):
        for rows_apart in (-tokens, -3, 0, 1, tokens + 1):
            assert served(x, y + rows_apart * pitch) == SPLIT
    for x, y in ((X0, X0 + 2 * K - 2), (X0, X0 + 2 * K + 66), (X0 + size * R - 2, X0), (X0 + size * R + 66, X0)):
        for rows_apart in (-3, 0, 1):
            assert served(x, y + rows_apart * pitch) == NONE


def test_more_rows_than_a_launch_has_threads_for_are_transposed_first():
    # 2^31 rows, 2^24 packed block rows: pairs of them, 512 threads each, are 2^32
    assert layer_form(host_handle(1 << 31, 36, 1 << 16, 4), X0, 36, 8, X0 << 8, 1 << 31) == NONE


@pytest.mark.parametrize("R,K,V,M,tokens,form", [
    (35712, 896, 32, 64, 16, NONE),      # 558 pairs, one at a time on a unit as their windows fill its LDS: 18 us, transposed first 7
    (39488, 256, 32, 128, 8, NONE), (36160, 480, 64, 32, 24, NONE),
    (49152, 12288, 128, 32, 16, PAIR),   # few tokens of a large layer: 21 us, transposed first 25
    (1024, 1024, 128, 8, 8, SPLIT),
])
def test_many_block_rows_of_few_steps_are_transposed_first(R, K, V, M, tokens, form):
    assert layer_form(host_handle(R, K, V, M), X0, K, tokens, X0 << 8, R) == form
