"""Boundaries and codes of fbdt_bin against the oracle at the edges of the
counting passes: the one-workgroup limit, several chunks per feature, chunks
long enough to sweep their 16-bit counters, crowded counters (few distinct
values), and rows that start at any element."""
import numpy as np
import pytest
import torch

import paper_1609_06119_amd as fb
from oracle import fbdt_oracle as O

pytestmark = pytest.mark.gpu


def _values(kind, n, d, rng):
    x = rng.standard_normal((d, n)).astype(np.float32)
    if kind == "mixed":
        special = np.array([0.0, -0.0, np.inf, -np.inf, 1e-45, -1e-45, 3e38, -3e38], np.float32)
        for j in range(d):
            if j % 4 == 1:
                x[j] = rng.integers(0, 1 + j, n)              # few levels
            elif j % 4 == 2:
                x[j, rng.random(n) < 0.5] = 0.25              # half the values on one
            elif j % 4 == 3:
                x[j] = 1000.0 + x[j] * 1e-3                   # one 16-bit prefix
            some = rng.integers(0, n, max(1, n // 50))
            x[j, some] = special[rng.integers(0, 8, some.size)]
    elif kind == "half":
        x[:, rng.random(n) < 0.5] = 0.25
    elif kind == "nan":
        for j in range(d):
            x[j, rng.random(n) < (0.3 * j) % 1.1] = np.nan
        x[d - 1] = np.nan
    return x


# more than 65,280 values per workgroup (test_plans.py checks that they are)
SWEPT = [(1_000_003, 40, 256, "mixed"), (2_500_000, 40, 200, "nan"), (16_711_681, 1, 256, "half")]


@pytest.mark.parametrize("n,d,n_bins,kind", [
    (1, 1, 2, "plain"), (3, 2, 256, "mixed"), (1023, 5, 256, "mixed"), (4097, 3, 17, "nan"),
    (20_480, 3, 256, "mixed"), (20_481, 3, 256, "mixed"),
    # the last size that one workgroup per feature counts alone, and the next
    (40_960, 8, 256, "mixed"), (40_960, 5, 200, "nan"), (40_961, 8, 256, "mixed"),
    (65_280, 4, 256, "mixed"), (65_281, 4, 256, "mixed"), (65_283, 3, 255, "nan"),
    (300_001, 7, 100, "nan"), (777_777, 9, 256, "mixed"),
    (4_000_001, 8, 256, "mixed"),     # 62,504 values per workgroup: close to the 16-bit limit
    # beyond it: swept counters, of crowded slots at every digit, of NaN, and
    # with a last workgroup whose own values would need no sweep
    *SWEPT,
])
def test_bin_matches_oracle(n, d, n_bins, kind):
    rng = np.random.default_rng([n, d, n_bins])
    x = _values(kind, n, d, rng)
    wide = torch.full((d, n + 7), float("nan"), device="cuda")
    view = wide[:, 3:n + 3]             # rows of an odd stride and start
    view.copy_(torch.from_numpy(x))
    bounds, codes = fb.bin(view, n_bins)
    code = codes.numpy()
    for j in range(d):
        ob = O.quantile_boundaries(x[j], n_bins)
        # -0 and +0 compare equal and may stand for one another at a rank
        assert np.array_equal(bounds[j], ob), f"boundaries of feature {j}"
        assert np.array_equal(code[j], O.encode(x[j], ob)), f"codes of feature {j}"


def test_nan_with_256_bins_writes_no_code():
    for n in (1000, 100_000):
        x = torch.randn(3, n, device="cuda")
        x[1, n // 2] = float("nan")
        codes = fb.Codes.empty(3, n)
        codes.data.fill_(0xAB)
        with pytest.raises(fb.FbdtError):
            fb.bin(x, 256, codes)
        assert bool((codes.data == 0xAB).all())
