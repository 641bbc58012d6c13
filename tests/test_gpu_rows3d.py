"""The 3D row gather (the library's chunk) against the plane ring (an explicit
chunk), bit for bit: strips of 64, 128 and 256 columns with their remainders,
row groups cut short, extents below the stencil's reach, misaligned buffers,
values that are not finite; and a batch of such grids against each alone."""
import numpy as np
import pytest

from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (3, 2, 1), (2, 5, 3), (5, 3, 64), (9, 7, 61), (4, 6, 127), (3, 10, 128), (6, 5, 256), (3, 9, 251),
        (2, 33, 300), (12, 40, 44)]


def _one(torch, x0, r, shape, c, bc, dtype, shift=0, steps=2, **kw):
    n = x0.numel()
    flat = [torch.zeros(n + shift, dtype=x0.dtype, device="cuda") for _ in range(2)]
    x, y = (f[shift:].view(x0.shape) for f in flat)
    x.copy_(x0)
    plan = st.Plan(x0.shape, r, shape, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1, **kw)
    out = plan.run_steps(x, y, steps).clone()
    torch.cuda.synchronize()
    plan.close()
    return out


@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("shape", [st.STAR, st.BOX])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("bc", [st.BC_ZERO, st.BC_PERIODIC])
def test_rows3d_equals_ring(dtype, shape, r, bc):
    torch = torch_cuda()
    c = inputs.coefficients(3, r, shape, seed=70 + r, dtype=np.float64)
    for k, dims in enumerate(DIMS):
        x0 = torch.from_numpy(inputs.grid(dims, seed=71 + k, dtype=np.float32 if dtype == st.F32 else np.float64)).cuda()
        want = _one(torch, x0, r, shape, c, bc, dtype, chunk=4)
        assert torch.equal(_one(torch, x0, r, shape, c, bc, dtype), want), dims
        assert torch.equal(_one(torch, x0, r, shape, c, bc, dtype, shift=1), want), (dims, "shifted")


@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("shape", [st.STAR, st.BOX])
@pytest.mark.parametrize("bc", [st.BC_ZERO, st.BC_PERIODIC])
def test_rows3d_values_not_finite(dtype, shape, bc):
    torch = torch_cuda()
    for r in (1, 3):
        c = inputs.coefficients(3, r, shape, seed=75, dtype=np.float64)
        x0 = torch.from_numpy(inputs.grid((14, 15, 70), seed=76, dtype=np.float32 if dtype == st.F32 else np.float64)).cuda()
        x0[2, 3, 69], x0[7, 7, 30], x0[13, 14, 0] = float("inf"), float("nan"), -float("inf")
        want = _one(torch, x0, r, shape, c, bc, dtype, steps=1, chunk=4)
        got = _one(torch, x0, r, shape, c, bc, dtype, steps=1)
        assert torch.equal(torch.nan_to_num(got, 7.0, 8.0, 9.0), torch.nan_to_num(want, 7.0, 8.0, 9.0))
        assert torch.equal(torch.isnan(got), torch.isnan(want))


def test_rows3d_batch_equals_alone():
    torch = torch_cuda()
    plans, b0, b1, want = [], [], [], []
    for k, (dims, r, shape, bc, dtype) in enumerate([
            ((33, 33, 33), 4, st.BOX, st.BC_ZERO, st.F64), ((20, 41, 230), 4, st.BOX, st.BC_PERIODIC, st.F64),
            ((30, 31, 62), 2, st.STAR, st.BC_PERIODIC, st.F32), ((40, 50, 301), 2, st.STAR, st.BC_ZERO, st.F32)]):
        c = inputs.coefficients(3, r, shape, seed=80 + k, dtype=np.float64)
        x0 = torch.from_numpy(inputs.grid(dims, seed=81 + k, dtype=np.float32 if dtype == st.F32 else np.float64)).cuda()
        want.append(_one(torch, x0, r, shape, c, bc, dtype, steps=3))
        plans.append(st.Plan(dims, r, shape, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1))
        b0.append(x0.clone())
        b1.append(torch.empty_like(x0))
    batch = st.Batch(plans, b0, b1)
    out = (b0, b1)[batch.run_steps(3)]
    torch.cuda.synchronize()
    for got, w in zip(out, want):
        assert torch.equal(got, w)
    batch.close()


# few and many grids of one size: the row gather of one column per lane, the plane
# ring, and (boxes from order 3) the row gather of two or four columns
@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("shape,r", [(st.STAR, 1), (st.STAR, 4), (st.BOX, 2), (st.BOX, 3), (st.BOX, 4)])
@pytest.mark.parametrize("dims,count", [((16, 32, 64), 3), ((16, 32, 64), 150), ((21, 24, 104), 40), ((18, 21, 231), 20)])
def test_rows3d_many_equals_alone(dtype, shape, r, dims, count):
    torch = torch_cuda()
    c = inputs.coefficients(3, r, shape, seed=90 + r, dtype=np.float64)
    nd = np.float32 if dtype == st.F32 else np.float64
    x0 = torch.stack([torch.from_numpy(inputs.grid(dims, seed=91 + k % 7, dtype=nd)) for k in range(count)]).cuda()
    plan = st.Plan(dims, r, shape, c, boundary=st.BC_ZERO, dtype=dtype, path=st.PATH_GATHER, time_block=1)
    b0, b1 = x0.clone(), torch.empty_like(x0)
    batch = st.Batch([plan] * count, list(b0), list(b1))
    out = (b0, b1)[batch.run_steps(2)].clone()
    torch.cuda.synchronize()
    batch.close()
    plan.close()
    for k in range(7 if count > 7 else count):
        want = _one(torch, x0[k], r, shape, c, st.BC_ZERO, dtype)
        for j in range(k, count, 7):
            assert torch.equal(out[j], want), (k, j)
