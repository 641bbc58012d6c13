"""AUTO on 2D grids whose column extent is not a multiple of 4: the gather, time
blocked where the aligned grids are, from 69 columns on."""
import numpy as np
import pytest

from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st


@pytest.mark.parametrize("shape", [inputs.STAR, inputs.BOX])
@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_auto_ragged_columns(shape, dtype, r):
    c = inputs.coefficients(2, r, shape, seed=3, dtype=np.float64)
    aligned = st.describe((96, 96), r, shape, c, dtype=dtype)
    for cols in (69, 101, 1531):
        info = st.describe((96, cols), r, shape, c, dtype=dtype)
        assert info["path"] == st.PATH_GATHER and info["time_block"] == aligned["time_block"]
        assert st.describe((96, cols), r, shape, c, dtype=dtype, time_block=1)["time_block"] == 1
    for cols in (61, 66, 67):
        info = st.describe((96, cols), r, shape, c, dtype=dtype)
        assert info["path"] == st.PATH_MFMA and info["time_block"] == 1
    assert st.describe((96, 101), r, st.GENERAL, c, dtype=dtype)["path"] == st.PATH_MFMA
