"""Requests of the serving loop by the company they meet: a cheap one does not go at
a costly one's pace; results equal each request alone, bit for bit."""
import numpy as np
import pytest

from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import torch_cuda

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
