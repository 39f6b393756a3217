"""The parity comparison itself (CPU): a NaN output or gradient entry is a
failure, not an error that no bound exceeds."""
import numpy as np

from parity import compare


def test_nan_fails():
    shapes = [("a", "W", (2, 2))]
    ref = dict(out=np.ones(3), d_params=np.ones(4), d_halo=np.zeros((0,)))
    nan = float("nan")
    bad = lambda out, dp: [b[0] for b in compare("nan", "fp32", shapes, (np.array(out), np.array(dp), None), ref)]
    assert bad([1, 1, 1], [1, 1, 1, 1]) == []
    assert bad([1, nan, 1], [1, 1, 1, 1]) == ["out"]
    assert bad([1, 1, 1], [1, 1, nan, 1]) == ["a"]
