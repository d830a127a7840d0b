"""GPU parity of the size-dependent branches of the launchers at the sizes where
they can go wrong (both sides of every dispatch line, ragged remainders, the
smallest and largest member counts), against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import direct
from paper_2307_02203_amd import ndf

pytestmark = pytest.mark.gpu

PEARSON_TOL = 1e-5  # the FP32 path's bar on every configured ensemble


def _ensemble(n_members, dims, seed, orders=False, transposed=False):
    rng = np.random.default_rng(seed)
    V = dims[0] * dims[1] * dims[2]
    base = rng.standard_normal((n_members, 3)).astype(np.float32)
    load = rng.standard_normal((3, V)).astype(np.float32)
    x = base @ load + rng.standard_normal((n_members, V), dtype=np.float32)
    e = ndf.Ensemble(torch.from_numpy(x).cuda(), *dims, orders=orders, transposed=transposed)
    ndf.ndf_prepare(e)
    return x, e


# one grid per branch of the member split (vertices < 2^15, < 2^17, < 2^19 and above),
# with vertex counts of every remainder mod 4, and member counts around the rows in
# flight (8), the split (16 shares) and the members of z held at a time (1024)
_GRIDS = [((2, 2, 2), 2), ((3, 3, 3), 15), ((37, 29, 11), 33), ((181, 181, 2), 17),
          ((123, 41, 7), 130), ((181, 363, 2), 9), ((257, 341, 6), 11), ((303, 347, 5), 129)]
_LONG = [((37, 29, 11), 2049), ((123, 41, 7), 1025), ((211, 125, 5), 1024)]


@pytest.mark.parametrize("dims,n_members,n_ref",
                         [(d, n, r) for d, n in _GRIDS for r in (1, 2, 3, 5, 9)]
                         + [(d, n, r) for d, n in _LONG for r in (1, 9)])
def test_pearson_fp32_member_splits(dims, n_members, n_ref):
    x, e = _ensemble(n_members, dims, seed=n_members + n_ref)
    V = x.shape[1]
    refs = np.random.default_rng(n_ref).integers(0, V, n_ref)
    refs[-1] = V - 1
    got = ndf.pearson_field(e, refs).cpu().numpy().astype(np.float64)
    # a strided subset of the vertices with both ends, against the oracle
    sub = np.unique(np.r_[0:min(V, 300), np.arange(0, V, max(1, V // 700)), max(0, V - 300):V])
    for i, r in enumerate(refs):
        want = direct.pearson_field(np.ascontiguousarray(x[:, r]), np.ascontiguousarray(x[:, sub]))
        assert np.max(np.abs(got[i, sub] - want)) <= PEARSON_TOL
