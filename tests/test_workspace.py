"""The workspace holds each line-solve table once, in the precision of the hierarchy's cycles."""
import pytest

from paper_2010_00626_amd import kcycle as K


@pytest.mark.parametrize("coarsening", ["full", "semi"])
@pytest.mark.parametrize("precision,item", [("f64", 8), ("f32", 4)])
def test_line_tables_once(precision, item, coarsening):
    """What a size adds beyond its arrays is a pair of tables per direction, as it is (n entries) and in the
    order of the lanes (n + 1 entries, lines of at least 63 points), and blocks' alignment."""
    n = 1023
    levels = [((n + 1) >> d) - 1 for d in range(10)]
    lines = [n if coarsening == "semi" else m for m in levels]
    padded = [(m + 63) // 64 * 64 for m in lines]
    arrays = sum(m * p for m, p in zip(levels, padded)) * item             # one buffer per level
    arrays += 2 * sum(m * p for m, p in zip(levels[precision == "f64":], padded[precision == "f64":])) * item
    vectors = 4 * n * padded[0] * 8
    tables = 4 * item * (sum(lines) + sum(m + 1 for m in lines if m >= 63))
    fixed = K.workspace_bytes([(1, 0.5, 1e-4)], precision)   # history, op lists, instance and state
    partial = 4 * 8 * 128 * 128                              # partial sums of 8 x 8 tiles
    assert K.workspace_bytes([(n, 0.5, 1e-4)], precision, coarsening) <= arrays + vectors + tables + fixed + partial + 64 * 256
