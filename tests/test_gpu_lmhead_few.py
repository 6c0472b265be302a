"""The LM head's weight-streaming form (at most 128 rows): both token widths
and the first row count past it, vocabularies with a partial last 32-id group,
fewer groups than CUs and ranges of one group up, one and several K stages,
against the oracle as the general form's tests are."""
import pytest

from test_gpu_lmhead import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,D,kw", [
    (33, 64, dict(bl=1, page_size=8, W_max=1, window=("fixed", 1))),    # 1 row, 2 groups, 1 stage
    (5003, 128, dict(bl=32, W_max=1, window=("fixed", 1))),             # 32 rows
    (8193, 192, dict(bl=32, W_max=2, window=("fixed", 2))),             # 64: the narrow form's last
    (70001, 192, dict(bl=13, W_max=5, window=("fixed", 5))),            # 65: the wide form's first
    (157184, 1024, dict(bl=32, W_max=4, window=("fixed", 4))),          # 128: the form's last
    (40000, 256, dict(bl=43, W_max=3, window=("fixed", 3))),            # 129: past it
    (65537, 2048, dict(B=4, bl=32, W_max=4, window=("fixed", 1))),      # 128 live of 512
    (65537, 2048, dict(B=5, bl=32, W_max=4, window=("fixed", 1))),      # 160: past the form
    (9001, 256, dict(B=4, bl=8, W_max=4, window=("uniform", 1, 4), layout="padded")),
])
def test_lmhead_few_rows(V, D, kw):
    run_case("single", V, D, seed=7, prefix=("fixed", 64), **kw)


@pytest.mark.parametrize("tied", [[5, 9, 37, 300, 5000], [4999, 5000, 157000]])
def test_lmhead_few_rows_ties_take_the_lowest_id(tied):
    """Exact ties across lane halves, groups, waves and ranges."""
    def edit(hid, weight):
        hid[:, 0] = 1.0
        weight[tied] = 0
        weight[tied, 0] = 256.0
    wl, host, packed, g, rows, o, tie, tok0 = run_case("single", 157184, 256, seed=6, edit=edit)
    assert (g["argmax"][rows] == min(tied)).all()
