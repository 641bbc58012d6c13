"""AUTO's FP32 3D boxes of order 3 and 4 in a batch: the gather of the grid alone
while they are few, the outer products among many -- then with the bits of a plan
of path MFMA, and within the error bound of the oracle.  Plans of path GATHER keep
the gather."""
import numpy as np
import pytest

import oracle
from paper_2310_16298_amd import inputs
from paper_2310_16298_amd import stencil as st

from gpu_helpers import eff_coeffs, error_bound, torch_cuda
from launched import launched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [st.BC_ZERO, st.BC_PERIODIC])
@pytest.mark.parametrize("r,dims,count,path,outer", [
    (4, (32, 32, 32), 256, st.PATH_AUTO, True), (4, (32, 32, 32), 16, st.PATH_AUTO, False),
    (4, (32, 32, 32), 256, st.PATH_GATHER, False), (3, (32, 32, 32), 256, st.PATH_AUTO, True),
    (3, (20, 44, 48), 16, st.PATH_AUTO, False), (4, (39, 41, 64), 64, st.PATH_AUTO, False),
    (4, (31, 63, 64), 64, st.PATH_AUTO, True),
    (4, (127, 128, 128), 12, st.PATH_AUTO, True),
    (4, (33, 33, 33), 256, st.PATH_AUTO, False)])
def test_boxes_among_many(r, dims, count, path, outer, bc):
    torch = torch_cuda()
    # two stencils of one order, each shared by half of the grids
    cs = [inputs.coefficients(3, r, st.BOX, seed=600 + k, dtype=np.float64) for k in range(2)]
    plans = [st.Plan(dims, r, st.BOX, c, boundary=bc, path=path) for c in cs]
    same = [st.Plan(dims, r, st.BOX, c, boundary=bc, path=st.PATH_MFMA if outer else path) for c in cs]
    assert plans[0].info["path"] == st.PATH_GATHER
    a0 = [inputs.grid(dims, seed=610 + k) for k in range(3)]
    b0 = torch.stack([torch.from_numpy(a0[k % 3]) for k in range(count)]).cuda()
    b1 = torch.empty_like(b0)
    batch = st.Batch([plans[k % 2] for k in range(count)], list(b0), list(b1))
    out = (b0, b1)[batch.run_steps(2)].clone()
    names = launched(torch, lambda: batch.run_steps(1))
    batch.close()
    assert len(names) == 1 and ("mfma3d_b4box_batch" in names[0]) == outer, names
    for k in range(6):
        x = torch.from_numpy(a0[k % 3]).cuda()
        want = same[k % 2].run_steps(x, torch.empty_like(x), 2)
        for j in range(k, count, 6):
            assert torch.equal(out[j], want), j
    ce = eff_coeffs(cs[1], st.F32)
    want = oracle.run(a0[1].astype(np.float64), ce, r, st.BOX, bc, 2)
    bound = error_bound(ce, 3, r, st.BOX, st.F32, st.PATH_MFMA, 2, float(np.abs(a0[1]).max()))
    assert float(np.abs(out[1].cpu().numpy() - want).max()) <= bound
    for p in plans + same:
        p.close()


def test_mixed_batch_with_outer_products():
    torch = torch_cuda()
    specs = [((32, 32, 32), 4, st.BOX, 200), ((32, 32, 32), 2, st.STAR, 5), ((40, 31, 30), 3, st.BOX, 3)]
    plans, b0, b1, want = [], [], [], []
    for dims, r, shape, count in specs:
        c = inputs.coefficients(3, r, shape, seed=620 + r, dtype=np.float64)
        p = st.Plan(dims, r, shape, c, time_block=1)
        alone = st.Plan(dims, r, shape, c, time_block=1, path=st.PATH_MFMA if count == 200 else st.PATH_AUTO)
        x = torch.from_numpy(inputs.grid(dims, seed=621)).cuda()
        w = alone.run_steps(x.clone(), torch.empty_like(x), 3).clone()
        for _ in range(count):
            plans.append(p)
            b0.append(x.clone())
            b1.append(torch.empty_like(x))
            want.append(w)
    batch = st.Batch(plans, b0, b1)
    for _ in range(2):  # replayed from the batch's graph the second time
        for b, k in zip(b0, range(len(b0))):
            b.copy_(torch.from_numpy(inputs.grid(tuple(b.shape), seed=621)))
        out = (b0, b1)[batch.run_steps(3)]
        torch.cuda.synchronize()
        for got, w in zip(out, want):
            assert torch.equal(got, w)
    batch.close()
