"""Generated constants of the fixed-point kernel with its sums on the matrix
cores: its tables against the cyclic shifts of the matrix, its division, and
the bound of its correction words."""
import re

import numpy as np
import pytest

from paper_2412_20828_amd import gen_spec
from tests.helpers import HO_ROWS, oracle_hopt


def table(src, name):
    m = re.search(r"uint8_t %s((?:\[\d+\])+) = \{(.*?)\};" % name, src, re.S)
    shape = [int(x) for x in re.findall(r"\d+", m.group(1))]
    return np.array([int(x) for x in re.findall(r"\d+", m.group(2))], np.uint8).reshape(shape)


@pytest.mark.parametrize("name,dp,split", [("bch127_64", 42, False), ("bch127_99", 42, False), ("bch63_36", 21, True)])
def test_tables(name, dp, split):
    H = oracle_hopt(name, HO_ROWS[name])
    M, N = H.shape
    src = gen_spec.body_source_mm(H, dp, split)
    par, main = table(src, "PAR"), table(src, "MAIN")
    # branch s reads the input shifted by s d_p: entry c of its rows at c - s d_p
    want = np.concatenate([np.stack([np.roll(r, -s * dp) for r in H]) for s in range(3)])
    assert np.array_equal(par[:3 * M, :N], want) and not par[3 * M:].any() and not par[:, N:].any()
    size = M if split else 3 * M
    assert main.shape[0] == 3 * M // size
    for st in range(main.shape[0]):
        assert np.array_equal(main[st, :N, :size].T, want[st * size:(st + 1) * size])
        assert not main[st, N:].any() and not main[st, :, size:].any()


def test_division_by_nine():
    x = np.arange(1 << 15, dtype=np.uint64)
    assert np.array_equal((x * 58255 + 4 * 58255) >> 19, (x + 4) // 9)
    assert int((x * 58255 + 4 * 58255).max()) < 1 << 32


def test_heavy_columns_are_refused():
    H = np.zeros((40, 127), np.uint8)
    H[:, 5] = 1
    H[:, :3] = 1
    with pytest.raises(ValueError, match="16 bits"):
        gen_spec.body_source_mm(H, 42, False)
