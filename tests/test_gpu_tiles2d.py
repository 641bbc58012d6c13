"""The time-blocked 2D gather on LDS tiles, inside the sizes where it is chosen:
grids alone, every step count, remainders of tiles, both boundaries, bit for bit
against one step per launch, and against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import eff_coeffs, error_bound, torch_cuda
from launched import launched

pytestmark = pytest.mark.gpu

Z, P = st.BC_ZERO, st.BC_PERIODIC


def _grid(dims, seed, dtype):
    return inputs.grid(dims, seed=seed, dtype=np.float32 if dtype == st.F32 else np.float64)


def _run(torch, a0, r, shape, c, bc, dtype, tb, steps, path=st.PATH_GATHER):
    x = torch.from_numpy(a0).cuda()
    plan = st.Plan(a0.shape, r, shape, c, boundary=bc, dtype=dtype, path=path, time_block=tb)
    out = plan.run_steps(x, torch.empty_like(x), steps).clone()
    torch.cuda.synchronize()
    plan.close()
    return out


# (dims, order, shape, boundary, type, most steps)
ALONE = [((1030, 1028), 3, st.BOX, bc, st.F32, 4) for bc in (Z, P)] + \
        [((1030, 1028), 4, s, bc, st.F32, 3) for s in (st.STAR, st.BOX) for bc in (Z, P)] + \
        [((1030, 1028), 3, st.STAR, Z, st.F32, 4), ((650, 700), 4, st.BOX, P, st.F32, 3),
         ((421, 604), 4, st.BOX, Z, st.F32, 3), ((25, 8452), 4, st.BOX, Z, st.F32, 3),
         ((799, 700), 4, st.STAR, Z, st.F32, 3), ((2050, 2052), 4, st.STAR, Z, st.F32, 3),
         ((33, 8200), 2, st.STAR, Z, st.F64, 4), ((33, 8200), 2, st.BOX, Z, st.F64, 4),
         ((33, 8200), 2, st.STAR, P, st.F64, 4), ((49, 4228), 2, st.STAR, P, st.F64, 4),
         ((33, 8200), 2, st.BOX, P, st.F64, 4), ((131, 2308), 3, st.STAR, Z, st.F64, 2),
         ((510, 516), 3, st.STAR, Z, st.F64, 2), ((65, 68), 4, st.STAR, Z, st.F64, 2),
         ((1281, 1284), 4, st.STAR, Z, st.F64, 2)]


@pytest.mark.parametrize("dims,r,shape,bc,dtype,tmax", ALONE)
def test_tiles_alone(dims, r, shape, bc, dtype, tmax):
    torch = torch_cuda()
    c = inputs.coefficients(2, r, shape, seed=300 + r, dtype=np.float64)
    a0 = _grid(dims, 301, dtype)
    for tb in range(2, tmax + 1):
        steps = 2 * tb - 1  # a launch of tb steps and a remainder
        got = _run(torch, a0, r, shape, c, bc, dtype, tb, steps)
        assert torch.equal(got, _run(torch, a0, r, shape, c, bc, dtype, 1, steps)), tb
        plan = st.Plan(dims, r, shape, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=tb)
        x = torch.from_numpy(a0).cuda()
        y = torch.empty_like(x)
        assert any("tb2d_dma_kernel" in n for n in launched(torch, lambda: plan.run_steps(x, y, tb))), tb
        plan.close()
    ce = eff_coeffs(c, dtype)
    want = oracle.run(a0.astype(np.float64), ce, r, shape, bc, steps)
    bound = error_bound(ce, 2, r, shape, dtype, st.PATH_GATHER, steps, float(np.abs(a0).max()))
    assert float(np.abs(got.cpu().numpy() - want).max()) <= bound

