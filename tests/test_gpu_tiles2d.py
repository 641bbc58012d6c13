"""The time-blocked 2D gather on LDS tiles, inside the sizes where it is chosen:
grids alone (every step count, remainders of tiles, both boundaries) and classes
of a batch, bit for bit against one step per launch, and against the oracle."""
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


# classes of about one round of waves
BATCH = [((250, 252), 16, 2, st.STAR, st.F32), ((250, 252), 16, 3, st.STAR, st.F32), ((250, 252), 16, 4, st.STAR, st.F32),
         ((250, 252), 16, 3, st.BOX, st.F32), ((250, 252), 16, 4, st.BOX, st.F32), ((61, 64), 256, 4, st.STAR, st.F32),
         ((518, 516), 2, 2, st.STAR, st.F64), ((518, 516), 2, 2, st.BOX, st.F64), ((518, 516), 2, 3, st.STAR, st.F64),
         ((518, 516), 2, 4, st.STAR, st.F64)]


@pytest.mark.parametrize("bc", [Z, P])
@pytest.mark.parametrize("dims,count,r,shape,dtype", BATCH)
def test_tiles_in_a_batch(dims, count, r, shape, dtype, bc):
    torch = torch_cuda()
    c = inputs.coefficients(2, r, shape, seed=310 + r, dtype=np.float64)
    seeds = [311 + k % 5 for k in range(count)]
    plan = st.Plan(dims, r, shape, c, boundary=bc, dtype=dtype)
    T = plan.info["time_block"]
    assert T > 1
    b0 = torch.stack([torch.from_numpy(_grid(dims, s, dtype)) for s in seeds]).cuda()
    x0 = b0.clone()
    b1 = torch.empty_like(b0)
    batch = st.Batch([plan] * count, list(b0), list(b1))
    names = launched(torch, lambda: batch.run_steps(2 * T))
    assert any("tb2d_dma_batch" in n for n in names), names
    for steps in range(2, T + 3):
        b0.copy_(x0)
        out = (b0, b1)[batch.run_steps(steps)]
        torch.cuda.synchronize()
        for k in range(min(count, 5)):
            want = _run(torch, _grid(dims, seeds[k], dtype), r, shape, c, bc, dtype, 1, steps)
            for j in range(k, count, 5):
                assert torch.equal(out[j], want), (steps, j)
    batch.close()
    plan.close()


# staged by element: 16-row and 32-row tiles, every remainder of a segment, buffers one
# element off a 16-byte line; the cells around the buffers stay as they are
@pytest.mark.parametrize("bc,dims,shift", [
    (Z, (1, 9), 0), (Z, (17, 10), 0), (Z, (64, 63), 0), (Z, (66, 65), 1), (Z, (64, 64), 1), (Z, (300, 201), 0),
    (Z, (1021, 1531), 0), (Z, (17, 5001), 1), (P, (301, 201), 0), (P, (300, 202), 1), (P, (3001, 9), 0),
    (P, (9, 3001), 0), (P, (901, 777), 0), (P, (300, 204), 1),
])
def test_ragged_order4_boxes(bc, dims, shift):
    torch = torch_cuda()
    c = inputs.coefficients(2, 4, st.BOX, seed=320, dtype=np.float64)
    a0 = _grid(dims, 321, st.F64)
    flat = [torch.full((a0.size + 64 + shift,), 7.5, dtype=torch.float64, device="cuda") for _ in range(2)]
    x, y = (f[32 + shift:32 + shift + a0.size].view(dims) for f in flat)
    plan = st.Plan(dims, 4, st.BOX, c, boundary=bc, dtype=st.F64, time_block=2)
    names = launched(torch, lambda: plan.run_steps(x, y, 2))
    assert len(names) == 1 and "tb2d_dma_kernel" in names[0], names
    for steps in (2, 4, 5):
        x.copy_(torch.from_numpy(a0))
        y.fill_(float("nan"))
        got = plan.run_steps(x, y, steps).clone()
        torch.cuda.synchronize()
        assert torch.equal(got, _run(torch, a0, 4, st.BOX, c, bc, st.F64, 1, steps)), steps
    for f in flat:
        edge = torch.cat([f[:32 + shift], f[32 + shift + a0.size:]])
        assert bool((edge == 7.5).all())
    plan.close()


# beside more than three classes the walks fill the chip together
@pytest.mark.parametrize("classes,tiles", [(2, True), (4, False)])
def test_tiles_beside_other_classes(classes, tiles):
    torch = torch_cuda()
    plans, b0, want = [], [], []
    for r, shape in [(3, st.STAR), (4, st.BOX), (4, st.STAR), (3, st.BOX)][:classes]:
        c = inputs.coefficients(2, r, shape, seed=330 + r, dtype=np.float64)
        plans += [st.Plan((250, 252), r, shape, c, boundary=P)] * 16
        a0 = _grid((250, 252), 331 + r, st.F32)
        b0 += [torch.from_numpy(a0).cuda() for _ in range(16)]
        want.append(_run(torch, a0, r, shape, c, P, st.F32, 1, 6))
    x0 = [b.clone() for b in b0]
    b1 = [torch.full_like(b, float("nan")) for b in b0]
    batch = st.Batch(plans, b0, b1)
    names = launched(torch, lambda: batch.run_steps(6))
    assert any("tb2d_dma_batch" in n for n in names) == tiles, names
    for b, x in zip(b0, x0):
        b.copy_(x)
    out = (b0, b1)[batch.run_steps(6)]
    torch.cuda.synchronize()
    for k, got in enumerate(out):
        assert torch.equal(got, want[k // 16]), k
    batch.close()
