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
    for cols in (69, 101, 1531):
        aligned = st.describe((96, cols // 4 * 4 + 4), r, shape, c, dtype=dtype)
        info = st.describe((96, cols), r, shape, c, dtype=dtype)
        assert info["path"] == st.PATH_GATHER and info["time_block"] == aligned["time_block"]
        assert st.describe((96, cols), r, shape, c, dtype=dtype, time_block=1)["time_block"] == 1
    for cols in (61, 66, 67):
        info = st.describe((96, cols), r, shape, c, dtype=dtype)
        assert info["path"] == st.PATH_MFMA and info["time_block"] == 1
    general = st.describe((96, 101), r, st.GENERAL, c, dtype=dtype)
    assert general["path"] == (st.PATH_GATHER if dtype == st.F64 else st.PATH_MFMA) and general["time_block"] == 1
    # the outer products' own options keep them
    assert st.describe((96, 101), r, st.BOX, c, path=st.PATH_AUTO, dtype=st.F32, reg_rows=8)["path"] == st.PATH_MFMA
    assert st.describe((96, 101), r, shape, c, dtype=dtype, block_n=16)["path"] == st.PATH_MFMA


def test_auto_f64_order3_box():
    c = inputs.coefficients(2, 3, inputs.BOX, seed=3, dtype=np.float64)
    assert st.describe((96, 100), 3, inputs.BOX, c, dtype=st.F64)["time_block"] == 2
    assert st.describe((96, 96), 3, inputs.BOX, c, dtype=st.F64)["time_block"] == 1
