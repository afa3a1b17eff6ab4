"""GPU parity at the sizes where single kernels and dispatch branches can go
wrong: edges of tiles, remainders, the smallest and largest of a range."""
import numpy as np
import pytest
import torch

import oracle
import scenegen
from parity import assert_parity, compare

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _native():
    from paper_2604_05794_amd import native
    native.lib()
    return native


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("samples,patch,top_k", [(1, 1, 5), (5, 7, 5), (6, 5, 5), (16, 3, 8), (16, 7, 2)])
def test_paper_candidate_layers(samples, patch, top_k):
    """The five- and the sixteen-layer kernels, every patch size."""
    nat = _native()
    sc = scenegen.make_scene("tiny", 3)
    kw = dict(patch=patch, top_k=top_k)
    fp = dict(lam=3.0, n_samples=samples, delta=5e-3)
    pts = sc.points[:3997]
    d, c = nat.fuse_directions(_t(pts), _t(sc.cams), _t(sc.theta), _t(sc.conf), depth_maps=_t(sc.depth),
                               mode=nat.FD_MODE_FPMVO, fpmvo_lambda=fp["lam"], fpmvo_samples=samples,
                               fpmvo_delta=fp["delta"], **kw)
    torch.cuda.synchronize()
    orc = oracle.Oracle(sc.cams, sc.theta, sc.conf, depth=sc.depth, **kw)
    do, co = orc.fpmvo(pts, **fp)
    assert_parity(compare(orc, pts, d.cpu().numpy(), c.cpu().numpy(), do, co))
