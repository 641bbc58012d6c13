"""Which kernel a one-step 3D gather runs on -- register rows or plane ring -- at
sizes on both sides of each line, for a grid alone, for several of one stencil and
beside others; every run against the ring (an explicit chunk), bit for bit."""
import numpy as np
import pytest

from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import torch_cuda
from launched import launched

pytestmark = pytest.mark.gpu

Z, P = st.BC_ZERO, st.BC_PERIODIC
S, B = st.STAR, st.BOX
F, D = st.F32, st.F64
RING, ROWS = "gather3d_", "rows3d_"


def _coef(r, shape):
    return inputs.coefficients(3, r, shape, seed=500 + r, dtype=np.float64)


def _field(torch, dims, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(dims, dtype=torch.float32 if dtype == F else torch.float64, device="cuda", generator=g) * 2 - 1


@pytest.mark.parametrize("dtype,r,shape,bc,dims,kernel", [
    (F, 1, S, Z, (16, 512, 512), RING), (F, 1, S, Z, (128, 128, 128), ROWS), (F, 1, S, P, (64, 256, 256), RING),
    (F, 1, S, P, (160, 160, 160), ROWS), (F, 1, B, Z, (28, 512, 512), RING), (F, 2, S, Z, (12, 600, 600), ROWS),
    (F, 4, S, Z, (12, 600, 600), RING), (F, 4, S, P, (32, 384, 384), ROWS), (F, 2, B, Z, (16, 512, 512), ROWS),
    (D, 4, S, P, (20, 300, 300), RING), (D, 4, S, Z, (8, 400, 400), ROWS), (D, 1, S, Z, (14, 256, 512), RING),
    (D, 3, S, Z, (100, 128, 100), ROWS)])
def test_alone(dtype, r, shape, bc, dims, kernel):
    torch = torch_cuda()
    x = _field(torch, dims, dtype, 501)
    outs = []
    for chunk in (4, 0):
        plan = st.Plan(dims, r, shape, _coef(r, shape), boundary=bc, dtype=dtype, path=st.PATH_GATHER, time_block=1,
                       chunk=chunk)
        y = torch.empty_like(x)
        names = launched(torch, lambda: plan.apply(x, y))
        outs.append(y)
        plan.close()
    assert len(names) == 1 and kernel in names[0], names
    assert torch.equal(outs[0], outs[1])


def _batch(torch, members, dtype, steps=2):
    """members: (dims, r, shape, bc); the batch's kernels after a check of its results."""
    plans, rings, b0, b1 = {}, {}, [], []
    for k, m in enumerate(members):
        if m not in plans:
            dims, r, shape, bc = m
            for store, chunk in ((plans, 0), (rings, 4)):
                store[m] = st.Plan(dims, r, shape, _coef(r, shape), boundary=bc, dtype=dtype, path=st.PATH_GATHER,
                                   time_block=1, chunk=chunk)
        b0.append(_field(torch, m[0], dtype, 510 + k % 5))
        b1.append(torch.empty_like(b0[-1]))
    x0 = [b.clone() for b in b0[:8]]
    batch = st.Batch([plans[m] for m in members], b0, b1)
    out = (b0, b1)[batch.run_steps(steps)]
    torch.cuda.synchronize()
    for m, x, got in zip(members, x0, out):
        assert torch.equal(got, rings[m].run_steps(x, torch.empty_like(x), steps)), m
    names = launched(torch, lambda: batch.run_steps(1))
    batch.close()
    for p in list(plans.values()) + list(rings.values()):
        p.close()
    return names


@pytest.mark.parametrize("dtype,r,shape,bc,n,count,kernel", [
    (F, 1, S, Z, 128, 2, RING), (F, 1, S, P, 32, 16, ROWS), (F, 1, S, P, 32, 64, RING), (F, 1, B, P, 32, 64, RING),
    (F, 3, S, Z, 32, 64, ROWS), (F, 3, S, Z, 32, 256, RING), (F, 2, B, Z, 32, 128, RING), (F, 2, B, Z, 32, 32, ROWS),
    (D, 1, B, Z, 128, 2, RING), (D, 2, B, Z, 128, 2, RING), (D, 2, B, Z, 24, 256, RING),
    (D, 4, S, Z, 128, 2, RING), (D, 4, S, Z, 64, 8, ROWS),
    (D, 4, B, P, 32, 64, ROWS)])
def test_many_of_one_stencil(dtype, r, shape, bc, n, count, kernel):
    torch = torch_cuda()
    names = _batch(torch, [((n, n, n), r, shape, bc)] * count, dtype)
    assert len(names) == 1 and kernel in names[0], names


# the same grids beside another stencil share the rows' launch
@pytest.mark.parametrize("dtype", [F, D])
def test_two_stencils_share_the_rows(dtype):
    torch = torch_cuda()
    one = ((64, 64, 64), 1, S, P)
    names = _batch(torch, [one] * 16, dtype)
    assert len(names) == 1 and RING in names[0], names
    names = _batch(torch, [((32, 32, 32), 1, S, P)] * 8 + [((32, 32, 32), 2, S, Z)] * 8, dtype)
    assert len(names) == 1 and "rows3d_merged" in names[0], names
    # large classes keep the ring beside each other
    names = _batch(torch, [((128, 128, 128), r, S, P) for r in (1, 1, 2, 2)], dtype)
    assert len(names) == 2 and all(RING in n for n in names), names


# a class of grids of several sizes goes by its points, not by their number
def test_sizes_of_a_class():
    torch = torch_cuda()
    names = _batch(torch, [((64, 64, 64), 2, B, Z)] + [((8, 8, 8), 2, B, Z)] * 30, D)
    assert len(names) == 1 and "rows3d" in names[0], names
