"""Kernels that only batches launch: the merged one-step gathers, every order and
shape of a type in one launch, and the whole-grid gather of many small 3D grids;
each grid against its own run, bit for bit."""
import numpy as np
import pytest

from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import torch_cuda
from launched import launched

pytestmark = pytest.mark.gpu

Z, P = st.BC_ZERO, st.BC_PERIODIC
EIGHT = [(r, shape) for r in (1, 2, 3, 4) for shape in (st.STAR, st.BOX)]


def _grid(torch, dims, seed, dtype):
    return torch.from_numpy(inputs.grid(dims, seed=seed, dtype=np.float32 if dtype == st.F32 else np.float64)).cuda()


def _plan(dims, r, shape, bc, dtype, **kw):
    c = inputs.coefficients(len(dims), r, shape, seed=800 + 10 * r + shape, dtype=np.float64)
    return st.Plan(dims, r, shape, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1, **kw)


@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("dims,kernel", [((61, 77), "rs2d_one_merged"), ((130, 259), "rs2d_one_merged"),
                                         ((9, 21, 35), "rows3d_merged"), ((17, 30, 131), "rows3d_merged")])
def test_all_stencils_of_a_type_in_one_launch(dtype, dims, kernel):
    torch = torch_cuda()
    plans, b0, b1, want = [], [], [], []
    for k, (r, shape) in enumerate(EIGHT + EIGHT[:3]):
        for bc in (Z, P):
            d = tuple(n + (k if j == 0 else 0) for j, n in enumerate(dims))  # sizes of their own
            plans.append(_plan(d, r, shape, bc, dtype))
            b0.append(_grid(torch, d, 810 + k, dtype))
            b1.append(torch.full_like(b0[-1], float("nan")))
            x = b0[-1].clone()
            want.append(plans[-1].run_steps(x, torch.empty_like(x), 3).clone())
    x0 = [b.clone() for b in b0]
    batch = st.Batch(plans, b0, b1)
    assert batch.info()["groups"] == 1
    names = launched(torch, lambda: batch.run_steps(1))
    assert len(names) == 1 and kernel in names[0], names
    for b, x in zip(b0, x0):
        b.copy_(x)
    out = (b0, b1)[batch.run_steps(3)]
    torch.cuda.synchronize()
    for k, (got, w) in enumerate(zip(out, want)):
        assert torch.equal(got, w), k
    batch.close()


# 300 grids, so that a workgroup each fills the chip: 16, 32, 64 and 128 KiB of LDS
@pytest.mark.parametrize("dtype", [st.F32, st.F64])
@pytest.mark.parametrize("r,shape", EIGHT)
@pytest.mark.parametrize("bc", [Z, P])
def test_many_small_grids_whole(dtype, r, shape, bc):
    torch = torch_cuda()
    for dims in ((8, 8, 8), (16, 16, 16), (5, 7, 3), (1, 1, 1), (2, 13, 9)):
        count = 300
        plan, ring = _plan(dims, r, shape, bc, dtype), _plan(dims, r, shape, bc, dtype, chunk=4)
        x = [_grid(torch, dims, 820 + k, dtype) for k in range(5)]
        b0 = torch.stack([x[k % 5] for k in range(count)])
        b1 = torch.full_like(b0, float("nan"))
        batch = st.Batch([plan] * count, list(b0), list(b1))
        info = batch.info()
        assert info["groups"] == 1 and info["items"] == count, (dims, info)
        out = (b0, b1)[batch.run_steps(3)]
        torch.cuda.synchronize()
        for k in range(5):
            want = ring.run_steps(x[k].clone(), torch.empty_like(x[k]), 3)
            for j in range(k, count, 5):
                assert torch.equal(out[j], want), (dims, j)
        if dims == (8, 8, 8):
            names = launched(torch, lambda: batch.run_steps(1))
            assert len(names) == 1 and "gather3d_whole_batch" in names[0], names
        batch.close()
        plan.close()
        ring.close()


# Below 228 grids the faster by the fitted times: a workgroup a grid takes one round
# however many they are, the rows' time follows their number.
@pytest.mark.parametrize("n,count,r,shape,dtype,kernel", [
    (8, 64, 1, st.BOX, st.F64, "rows3d_batch"), (8, 200, 1, st.BOX, st.F64, "gather3d_whole_batch"),
    (8, 64, 4, st.BOX, st.F64, "rows3d_batch"), (8, 200, 2, st.STAR, st.F32, "gather3d_whole_batch"),
    (12, 64, 3, st.STAR, st.F64, "rows3d_batch"), (12, 150, 3, st.STAR, st.F64, "gather3d_whole_batch"),
    (16, 64, 3, st.STAR, st.F64, "rows3d_batch"), (16, 200, 3, st.STAR, st.F64, "gather3d_whole_batch"),
    (16, 200, 4, st.BOX, st.F64, "rows3d_batch"), (16, 200, 3, st.BOX, st.F32, "rows3d_batch"),
])
def test_whole_grids_below_a_full_chip(n, count, r, shape, dtype, kernel):
    torch = torch_cuda()
    plan = _plan((n, n, n), r, shape, P, dtype)
    x = _grid(torch, (n, n, n), 830, dtype)
    want = plan.run_steps(x.clone(), torch.empty_like(x), 3)
    b0 = x.repeat(count, 1, 1, 1)
    b1 = torch.full_like(b0, float("nan"))
    batch = st.Batch([plan] * count, list(b0), list(b1))
    names = launched(torch, lambda: batch.run_steps(1))
    assert len(names) == 1 and kernel in names[0], names
    b0.copy_(x.expand_as(b0))
    out = (b0, b1)[batch.run_steps(3)]
    torch.cuda.synchronize()
    assert torch.equal(out, want.expand_as(out))
    batch.close()
