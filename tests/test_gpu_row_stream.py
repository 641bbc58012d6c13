"""The register-streaming time-blocked 2D gather against one step per launch,
bit for bit: strip widths of 1, 2 and 4 columns per lane with their remainders,
grids that fit one strip whole, extents below the stencil's reach, chunks of
one row, misaligned buffers, and values that are not finite."""
import numpy as np
import pytest

from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu

TMAX = {(st.F32, 1): 12, (st.F32, 2): 6, (st.F32, 3): 4, (st.F32, 4): 3,
        (st.F64, 1): 8, (st.F64, 2): 4, (st.F64, 3): 2, (st.F64, 4): 2}
DIMS = [(1, 1), (3, 2), (7, 3), (2, 61), (33, 64), (20, 65), (70, 128), (40, 256), (9, 257), (300, 131), (1100, 47),
        (5, 2051), (700, 1010)]


def _advance(torch, x0, r, shape, c, bc, dtype, tb, steps, path=st.PATH_AUTO, shift=0):
    n = x0.numel()
    flat = [torch.zeros(n + shift, dtype=x0.dtype, device="cuda") for _ in range(2)]
    x, y = (f[shift:].view(x0.shape) for f in flat)
    x.copy_(x0)
    plan = st.Plan(x0.shape, r, shape, c, boundary=bc, dtype=dtype, path=path, time_block=tb)
    out = plan.run_steps(x, y, steps).clone()
    torch.cuda.synchronize()
    plan.close()
    return out


@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("shape", [st.STAR, st.BOX])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("bc", [st.BC_ZERO, st.BC_PERIODIC])
def test_row_stream_equals_single_steps(dtype, shape, r, bc):
    torch = torch_cuda()
    c = inputs.coefficients(2, r, shape, seed=90 + r, dtype=np.float64)
    tmax = TMAX[(dtype, r)]
    for k, dims in enumerate(DIMS):
        x0 = torch.from_numpy(inputs.grid(dims, seed=91 + k, dtype=np.float32 if dtype == st.F32 else np.float64)).cuda()
        for tb, steps in {(2, 3), (tmax, tmax), (tmax, 2 * tmax - 1)}:
            want = _advance(torch, x0, r, shape, c, bc, dtype, 1, steps, path=st.PATH_GATHER)
            assert torch.equal(_advance(torch, x0, r, shape, c, bc, dtype, tb, steps), want), (dims, tb, steps)
        assert torch.equal(_advance(torch, x0, r, shape, c, bc, dtype, tmax, steps, shift=1), want), (dims, "shifted")


@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("shape", [st.STAR, st.BOX])
@pytest.mark.parametrize("bc", [st.BC_ZERO, st.BC_PERIODIC])
def test_row_stream_values_not_finite(dtype, shape, bc):
    torch = torch_cuda()
    for r in (1, 2, 3):
        c = inputs.coefficients(2, r, shape, seed=95, dtype=np.float64)
        x0 = torch.from_numpy(inputs.grid((90, 301), seed=96, dtype=np.float32 if dtype == st.F32 else np.float64)).cuda()
        x0[4, 300], x0[50, 119], x0[89, 0] = float("inf"), float("nan"), -float("inf")
        want = _advance(torch, x0, r, shape, c, bc, dtype, 1, 2, path=st.PATH_GATHER)
        got = _advance(torch, x0, r, shape, c, bc, dtype, 2, 2)
        assert torch.equal(torch.nan_to_num(got, 7.0, 8.0, 9.0), torch.nan_to_num(want, 7.0, 8.0, 9.0))
        assert torch.equal(torch.isnan(got), torch.isnan(want))


# FP64 order 2 on grids of one round of LDS tiles, against one step per launch
@pytest.mark.parametrize("shape", [st.STAR, st.BOX])
@pytest.mark.parametrize("dims,bc", [((250, 256), st.BC_ZERO), ((431, 448), st.BC_ZERO), ((17, 11264), st.BC_ZERO),
                                     ((49, 4224), st.BC_PERIODIC), ((24, 8448), st.BC_PERIODIC)])
def test_fp64_order2_tiles_equal_one_step(shape, dims, bc):
    torch = torch_cuda()
    c = inputs.coefficients(2, 2, shape, seed=61, dtype=np.float64)
    x0 = torch.from_numpy(inputs.grid(dims, seed=62, dtype=np.float64)).cuda()
    for steps in (2, 3, 4, 9):
        outs = []
        for tb in (1, 4):
            plan = st.Plan(dims, 2, shape, c, boundary=bc, dtype=st.F64, path=st.PATH_GATHER, time_block=tb)
            x = x0.clone()
            y = torch.empty_like(x)
            outs.append(plan.run_steps(x, y, steps).clone())
            torch.cuda.synchronize()
            plan.close()
        assert torch.equal(outs[0], outs[1]), steps
