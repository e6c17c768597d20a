"""The deposit on tiles of 64 columns at their edges: columns and heights that
leave a remainder, one and several mask words, columns that overflow and keep
fluid, and grids too tall for the tiles.  Every result is the oracle's bit for
bit: both replay a column's fills in the same order with the same operations."""
import numpy as np
import pytest

from test_gpu_conversion import any_scene, check_exact, ragged_state, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,dims,fluid", [(31, (3, 2, 1), 1.0), (32, (64, 2, 64), 1.0), (33, (65, 3, 65), 4.0),
                                             (34, (21, 3, 128), 1.0), (35, (29, 5, 150), 8.0), (36, (7, 3, 1024), 30.0),
                                             (37, (7, 3, 1025), 30.0), (38, (130, 2, 33), 50.0)])
def test_deposit_tiles_bit_exact(seed, dims, fluid):
    st, wedges = ragged_state(seed, dims)
    st["mf"] = st["mf"] * fluid
    got, ref = run_gpu(any_scene(), st, wedges), run_oracle(st, wedges)
    check_exact(got, ref)
    if fluid >= 8.0:  # some columns are full to the top and some of their fluid stays
        assert np.any((ref["phi"][-1] >= 1.0) & (ref["mf"].max(0) > 0.0))
