"""The conversion on grids of so many columns that its kernels split them
differently: deposit tiles of 64 columns above 32,768, a thread a column in the
cut above 200,000; remainders in columns and heights.  Every result is the
oracle's bit for bit; the totals are compared with the exactly rounded sums of
what the oracle's arrays gain and lose (its own running sum is off by up to
1.4e-11 over so many voxels)."""
import math

import numpy as np
import pytest

from test_gpu_conversion import any_scene, ragged_state, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,dims,fluid", [(51, (128, 256, 17), 4.0), (52, (129, 255, 65), 4.0),
                                             (53, (257, 128, 150), 8.0), (54, (181, 182, 1), 1.0),
                                             (55, (400, 500, 9), 4.0), (56, (401, 499, 9), 4.0)])
def test_many_columns_bit_exact(seed, dims, fluid):
    st, wedges = ragged_state(seed, dims)
    st["mf"] = st["mf"] * fluid
    got, ref = run_gpu(any_scene(), st, wedges), run_oracle(st, wedges)
    for k in ("phi_c", "mf_c", "phi", "wc", "mf", "h"):
        assert np.array_equal(got[k].reshape(ref[k].shape), ref[k]), k
    assert got["lib"] == pytest.approx(math.fsum((ref["mf_c"] - st["mf"]).ravel()), rel=1e-12, abs=1e-12)
    assert got["dep"] == pytest.approx(math.fsum((ref["mf_c"] - ref["mf"]).ravel()), rel=1e-12, abs=1e-12)
    assert np.any(ref["phi"] != st["phi"]) or dims[2] == 1
