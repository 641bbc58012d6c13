"""The one-step 2D gather: LDS windows and row walk at the sizes where each is
chosen.  Buffers shifted by one element cannot take the windows, so the same grid
runs on the walk there: both must give the same bits."""
import numpy as np
import pytest

import oracle
from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import eff_coeffs, error_bound, torch_cuda
from launched import launched

pytestmark = pytest.mark.gpu

Z, P = st.BC_ZERO, st.BC_PERIODIC
S, B = st.STAR, st.BOX
F, D = st.F32, st.F64


def _grid(dims, seed, dtype):
    return inputs.grid(dims, seed=seed, dtype=np.float32 if dtype == F else np.float64)


def _two(torch, a0, shift):
    flat = [torch.zeros(a0.size + shift, dtype=torch.from_numpy(a0).dtype, device="cuda") for _ in range(2)]
    x, y = (f[shift:].view(a0.shape) for f in flat)
    x.copy_(torch.from_numpy(a0))
    return x, y


# (type, order, shape, boundary, dims): a remainder of rows and of columns in each
WINDOWS = [
    (F, 4, S, Z, (513, 516)), (F, 4, B, Z, (511, 516)), (F, 3, S, Z, (901, 1004)), (F, 3, B, Z, (901, 1004)),
    (F, 2, S, Z, (1030, 1028)), (F, 2, B, Z, (1030, 1028)), (F, 1, S, Z, (2101, 2104)), (F, 1, B, Z, (4131, 4132)),
    (F, 4, B, P, (901, 1004)), (F, 1, S, P, (4131, 4132)), (F, 1, B, P, (4131, 4132)), (F, 2, S, P, (4131, 4132)),
    (F, 2, B, P, (4131, 4132)), (F, 3, S, P, (5841, 5844)), (F, 4, S, P, (5841, 5844)), (F, 2, B, Z, (25, 8452)),
    (D, 1, S, Z, (2921, 2924)), (D, 1, B, Z, (2301, 2308)), (D, 2, S, Z, (1030, 1028)), (D, 2, B, Z, (1030, 1028)),
    (D, 3, S, Z, (901, 1004)), (D, 3, B, Z, (513, 516)), (D, 4, S, Z, (67, 68)), (D, 4, B, Z, (203, 204)),
    (D, 1, S, P, (2921, 2924)), (D, 1, B, P, (2921, 2924)), (D, 2, S, P, (2921, 2924)), (D, 2, B, P, (2921, 2924)),
    (D, 3, S, P, (4131, 4132)), (D, 4, S, P, (4131, 4132)), (D, 4, B, P, (203, 204)), (D, 2, S, Z, (25, 8452)),
]


@pytest.mark.parametrize("dtype,r,shape,bc,dims", WINDOWS)
def test_windows_equal_walk(dtype, r, shape, bc, dims):
    torch = torch_cuda()
    c = inputs.coefficients(2, r, shape, seed=400 + r, dtype=np.float64)
    a0 = _grid(dims, 401, dtype)
    plan = st.Plan(dims, r, shape, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1)
    outs = []
    for shift, kernel in ((0, "gather2d_dma_kernel"), (1, "rs2d_kernel")):
        x, y = _two(torch, a0, shift)
        outs.append(plan.run_steps(x, y, 2).clone())
        names = launched(torch, lambda: plan.apply(x, y))
        assert len(names) == 1 and kernel in names[0], (shift, names)
    plan.close()
    assert torch.equal(outs[0], outs[1])
    if a0.size <= 1200000:
        ce = eff_coeffs(c, dtype)
        want = oracle.run(a0.astype(np.float64), ce, r, shape, bc, 2)
        bound = error_bound(ce, 2, r, shape, dtype, st.PATH_GATHER, 2, float(np.abs(a0).max()))
        assert float(np.abs(outs[0].cpu().numpy() - want).max()) <= bound


# sizes on the walk's side of the same lines
WALK = [(F, 1, S, Z, (512, 512)), (F, 2, B, Z, (768, 768)), (F, 3, S, Z, (512, 512)), (F, 4, B, Z, (700, 64)),
        (F, 3, B, Z, (2048, 2048)), (F, 4, S, Z, (2560, 2560)), (F, 4, B, P, (512, 512)), (D, 1, B, Z, (2048, 2048)),
        (D, 3, B, Z, (256, 256)), (D, 4, S, Z, (1280, 1280)), (D, 4, S, P, (512, 512)), (D, 2, S, Z, (3, 100000))]


@pytest.mark.parametrize("dtype,r,shape,bc,dims", WALK)
def test_walk_is_chosen(dtype, r, shape, bc, dims):
    torch = torch_cuda()
    c = inputs.coefficients(2, r, shape, seed=410 + r, dtype=np.float64)
    plan = st.Plan(dims, r, shape, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1)
    x, y = _two(torch, _grid(dims, 411, dtype), 0)
    names = launched(torch, lambda: plan.apply(x, y))
    plan.close()
    assert len(names) == 1 and "rs2d_kernel" in names[0], names


# rows per item asked for: windows on a zero halo, the walk on periodic grids
@pytest.mark.parametrize("bc,kernel", [(Z, "gather2d_dma_kernel"), (P, "rs2d_kernel")])
@pytest.mark.parametrize("dtype", [F, D])
def test_rows_asked_for(dtype, bc, kernel):
    torch = torch_cuda()
    c = inputs.coefficients(2, 2, S, seed=420, dtype=np.float64)
    a0 = _grid((500, 516), 421, dtype)
    outs = []
    for chunk in (0, 64):
        plan = st.Plan(a0.shape, 2, S, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1, chunk=chunk)
        x, y = _two(torch, a0, 0)
        outs.append(plan.run_steps(x, y, 2).clone())
        names = launched(torch, lambda: plan.apply(x, y))
        plan.close()
    assert len(names) == 1 and kernel in names[0], names
    assert torch.equal(outs[0], outs[1])


# several grids of one stencil: windows while they are few, the walk beyond
@pytest.mark.parametrize("dtype,r,shape,bc,dims,count,kernel", [
    (F, 4, S, Z, (250, 252), 16, "gather2d_dma_batch"), (F, 1, B, Z, (250, 252), 16, "gather2d_dma_batch"),
    (F, 1, S, Z, (250, 252), 200, "rs2d_batch"), (F, 3, B, P, (250, 252), 16, "gather2d_dma_batch"),
    (F, 1, B, P, (250, 252), 16, "rs2d_batch"), (D, 3, S, Z, (61, 64), 16, "gather2d_dma_batch"),
    (D, 4, S, Z, (250, 252), 64, "rs2d_batch"), (D, 4, S, P, (250, 252), 16, "gather2d_dma_batch")])
def test_many_of_one_stencil(dtype, r, shape, bc, dims, count, kernel):
    torch = torch_cuda()
    c = inputs.coefficients(2, r, shape, seed=430 + r, dtype=np.float64)
    plan = st.Plan(dims, r, shape, c, boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1)
    one = [torch.from_numpy(_grid(dims, 431 + k, dtype)).cuda() for k in range(min(count, 7))]
    b0 = torch.stack([one[k % 7] for k in range(count)])
    b1 = torch.empty_like(b0)
    batch = st.Batch([plan] * count, list(b0), list(b1))
    out = (b0, b1)[batch.run_steps(2)].clone()
    names = launched(torch, lambda: batch.run_steps(1))
    assert len(names) == 1 and kernel in names[0], names
    batch.close()
    for k, x in enumerate(one):
        want = plan.run_steps(x, torch.empty_like(x), 2)
        for j in range(k, count, 7):
            assert torch.equal(out[j], want), j
    plan.close()


def test_one_strip_of_many_rows_takes_the_walk():
    torch = torch_cuda()
    c = inputs.coefficients(2, 3, S, seed=440, dtype=np.float64)
    plan = st.Plan((40000, 8), 3, S, c, boundary=Z, dtype=D)
    x, y = _two(torch, _grid((40000, 8), 441, D), 0)
    assert plan.info["time_block"] == 2
    names = launched(torch, lambda: plan.run_steps(x, y, 2))
    plan.close()
    assert len(names) == 1 and "rs2d_kernel" in names[0], names


# orders 3 and 4 join the merged walk only where their class is small
@pytest.mark.parametrize("n,count,r,merged", [(64, 4, 3, True), (256, 16, 3, False), (256, 16, 1, True)])
def test_two_stencils(n, count, r, merged):
    torch = torch_cuda()
    plans, b0, want = [], [], []
    for order, shape in [(r, S), (r + 1, B)]:
        c = inputs.coefficients(2, order, shape, seed=440 + order, dtype=np.float64)
        plan = st.Plan((n, n), order, shape, c, boundary=Z, dtype=F, path=st.PATH_GATHER, time_block=1)
        x = torch.from_numpy(_grid((n, n), 441 + order, F)).cuda()
        plans += [plan] * count
        b0 += [x.clone() for _ in range(count)]
        want.append(plan.run_steps(x, torch.empty_like(x), 2).clone())
    x0 = [b.clone() for b in b0]
    b1 = [torch.full_like(b, float("nan")) for b in b0]
    batch = st.Batch(plans, b0, b1)
    names = launched(torch, lambda: batch.run_steps(1))
    assert (len(names) == 1 and "rs2d_one_merged" in names[0]) == merged, names
    for b, x in zip(b0, x0):
        b.copy_(x)
    out = (b0, b1)[batch.run_steps(2)]
    torch.cuda.synchronize()
    for k, got in enumerate(out):
        assert torch.equal(got, want[k // count]), k
    batch.close()
