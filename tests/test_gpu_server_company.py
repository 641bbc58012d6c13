"""Requests of the serving loop by the company they meet: a cheap one does not go at
a costly one's pace, one alone is cut for the whole chip, many of one stencil run
on the kernel that suits many; results equal each request alone, bit for bit."""
import numpy as np
import pytest

from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import torch_cuda
from launched import launched

pytestmark = pytest.mark.gpu


def _coef(dims, r, shape):
    return inputs.coefficients(len(dims), r, shape, seed=700 + r, dtype=np.float64)


def _alone(torch, x, r, shape, steps):
    plan = st.Plan(tuple(x.shape), r, shape, _coef(x.shape, r, shape))
    out = plan.run_steps(x.clone(), torch.empty_like(x), steps).clone()
    torch.cuda.synchronize()
    plan.close()
    return out


def test_cheap_request_beside_a_costly_one():
    torch = torch_cuda()
    big, small = (4096, 4096), (64, 64)
    x, y = (torch.from_numpy(inputs.grid(d, seed=701)).cuda() for d in (big, small))
    ox, oy = torch.empty_like(x), torch.empty_like(y)
    torch.cuda.synchronize()
    srv = st.Server(3 * x.numel() * 4)
    srv.submit(x, ox, 20, 3, st.BOX, _coef(big, 3, st.BOX))
    cheap = srv.submit(y, oy, 64, 1, st.STAR, _coef(small, 1, st.STAR))
    ticks = []
    while not ticks or ticks[-1]["active"]:
        ticks.append(srv.tick())
    # 20 ticks of one costly step each, several cheap steps in each of the first
    first = next(k for k, t in enumerate(ticks) if t["retired"])
    assert first < 8 and len(ticks) <= 24, (first, len(ticks))
    torch.cuda.synchronize()
    assert cheap in srv.poll()
    srv.close()
    assert torch.equal(oy, _alone(torch, y, 1, st.STAR, 64))
    assert torch.equal(ox, _alone(torch, x, 3, st.BOX, 20))


def _serve(torch, xs, r, shape, steps):
    outs = [torch.empty_like(x) for x in xs]
    srv = st.Server(sum(2 * x.numel() * 4 + (1 << 20) for x in xs))
    torch.cuda.synchronize()

    def burst():
        left = {srv.submit(x, o, steps, r, shape, _coef(x.shape, r, shape)) for x, o in zip(xs, outs)}
        while left:
            srv.tick()
            left.difference_update(srv.poll())

    names = launched(torch, burst)
    srv.close()
    return outs, names


@pytest.mark.parametrize("count,kernel", [(4, "rows3d_batch"), (64, "gather3d_batch")])
def test_many_of_one_stencil(count, kernel):
    torch = torch_cuda()
    xs = [torch.from_numpy(inputs.grid((64, 64, 64), seed=710 + k % 3)).cuda() for k in range(count)]
    outs, names = _serve(torch, xs, 1, st.STAR, 3)
    assert len(names) == 1 and kernel in names[0], names
    for k in range(3):
        want = _alone(torch, xs[k], 1, st.STAR, 3)
        for j in range(k, count, 3):
            assert torch.equal(outs[j], want), j


def test_order4_box_alone_takes_wide_rows():
    torch = torch_cuda()
    x = torch.from_numpy(inputs.grid((128, 128, 128), seed=720)).cuda()
    outs, names = _serve(torch, [x], 4, st.BOX, 2)
    # several columns a lane, not the merged shape of one (111 us a step against 57)
    assert len(names) == 1 and "rows3d_batch<float, 4, true, 1," not in names[0] and "rows3d_batch" in names[0], names
    assert torch.equal(outs[0], _alone(torch, x, 4, st.BOX, 2))
