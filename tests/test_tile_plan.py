"""Which tiles the shapes of the lm_head tests take, from the plan itself (no GPU needed)."""
import pytest

import paper_2507_19766_amd as ulorl
import test_gpu_lmhead as lmhead
import test_gpu_random_shapes as random_shapes
from tile_plan import backward_chunks, backward_is_large, column_tiles, forward_is_large, workspace_bytes


@pytest.mark.parametrize("shape", [(777, 2048, 151936, 8, 8192), (1300, 320, 5000, 2, 64), (20000, 512, 1000, 31, 8192), (33, 64, 520, 2, 8192)])
def test_the_plan_is_the_library_s(shape):
    assert workspace_bytes(*shape) == ulorl.lmhead_workspace_bytes(*shape)


def test_large_tiles_are_reached_where_a_test_says_so():
    for n, V, hidden in lmhead.LARGE_IN_FORWARD + lmhead.LARGE_IN_BOTH:
        assert forward_is_large(n, hidden, V), (n, V, hidden)
    for n, V, hidden in lmhead.LARGE_IN_BOTH:
        assert backward_is_large(n, hidden, V), (n, V, hidden)
    for n, V, hidden, chunk in lmhead.LARGE_BACKWARD:
        assert backward_is_large(n, hidden, V), (n, V, hidden)
    for n, V, hidden in lmhead.LARGE_IN_CHUNKS:
        assert backward_is_large(n, hidden, V) and backward_chunks(n, hidden, V, 64) >= 3, (n, V, hidden)
    assert backward_chunks(1281, 448, 9480, 1024) == 3
    for hidden, V in ((320, 9536), (392, 9480)):                  # with few live rows
        assert backward_is_large(1300, hidden, V)
    assert forward_is_large(300, 2048, 65544) and not forward_is_large(300, 320, 65544)           # large logits
    for n in (257, 288):
        assert column_tiles(n) == [160, 128]
    widths = {w for n, V, hidden in lmhead.LARGE_IN_FORWARD + lmhead.LARGE_IN_BOTH for w in column_tiles(n)}
    assert widths == {128, 160, 192, 224, 256}
    widths = {w for n, V, hidden in lmhead.LARGE_IN_BOTH for w in column_tiles(n)}
    assert widths == {128, 160, 192}


def test_the_random_cases_of_large_tiles_take_them():
    cases = [(sum(c["lengths"]), c["hidden"], c["V"], c) for c in random_shapes._lmhead_large_cases()]
    assert all(backward_is_large(n, hidden, V) and backward_chunks(n, hidden, V, c["chunk"]) >= 2 for n, hidden, V, c in cases)
    assert sum(forward_is_large(n, hidden, V) for n, hidden, V, c in cases) >= 4
    assert {c["dense_rows"] for *_, c in cases} == {False, True} and {hidden % 64 == 0 for _, hidden, _, _ in cases} == {False, True}
    assert not any(backward_is_large(sum(c["lengths"]), c["hidden"], c["V"]) for c in random_shapes._lmhead_many_rows_cases())
