"""GPU parity at the far ends of what the calls accept: the largest grids, few members,
workspaces of the smallest accepted size, parameters that are no numbers, and kernels that
only certain sizes reach."""
import sys

import numpy as np
import pytest
import torch

import gen
from oracle import direct
from oracle import ndf_net as nn
from paper_2307_02203_amd import ndf

pytestmark = pytest.mark.gpu

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from floors import TRAIN_OPS, check_grad_floor  # noqa: E402


# two members on just over 2^27 and on 2^28 vertices: a second row of workgroups, and the grid
# whose threads no longer fit one launch axis
@pytest.mark.parametrize("dims", [(2048, 1025, 64), (2048, 2048, 64)])
def test_prepare_of_very_many_vertices(dims):
    V = dims[0] * dims[1] * dims[2]
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.randn((2, V), generator=g, device="cuda")
    e = ndf.Ensemble(x, *dims, orders=True)
    e.flags.fill_(77)
    e.order.fill_(77)
    ndf.ndf_prepare(e)
    for v0 in (0, (1 << 27) - 500, V // 2, V - 1000):
        rows = slice(v0, v0 + 1000)
        c = x[:, rows].cpu().numpy().astype(np.float64)
        assert np.all(c[0] != c[1])
        first = c[0] < c[1]
        code = e.code[0, rows].cpu().numpy()
        assert np.array_equal(code, np.stack([~first, first], 1).astype(np.int64) << 23)
        assert np.array_equal(e.order[0, rows].cpu().numpy(), np.stack([~first, first], 1))
        assert np.array_equal(e.flags[0, rows].cpu().numpy(), np.zeros(1000))
        assert np.array_equal(e.mean[0, rows].cpu().numpy(), (c[0] + c[1]) / 2)
    del e, x
    torch.cuda.empty_cache()
