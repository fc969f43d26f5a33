"""The shipped table is the autotuner's own output: every row carries a
figure that was measured for that row."""
import os

from paper_2604_22228_amd import autotune

TABLE = os.path.join(os.path.dirname(os.path.abspath(autotune.__file__)),
                     "tuned_mi355x.txt")


def test_one_row_per_tuned_key():
    rows = autotune.read_table(TABLE)
    want = sorted((autotune.DTYPE_NAMES[d], autotune.OP_NAMES[o], r,
                   "1" if g else "*")
                  for d, o, r, g, _counts, _parts in autotune.default_keys())
    assert sorted(r[:4] for r in rows) == want


def test_no_figure_is_carried_to_another_row():
    rows = autotune.read_table(TABLE)
    for i, a in enumerate(rows):
        for b in rows[i + 1:]:
            assert a[6] != b[6], (a, b)


def test_shapes_come_from_the_search_grid():
    for d, o, ranks, _g, _lg, choice, _ms in autotune.read_table(TABLE):
        dtype = {v: k for k, v in autotune.DTYPE_NAMES.items()}[d]
        grid = autotune.grid_for(dtype, ranks)
        assert all(c in g for c, g in zip(choice, grid)), (d, o, choice)
