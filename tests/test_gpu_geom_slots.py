"""The on-the-fly step's kernel variants (lanes per token 1, 2, 4 and 8; bound
on the anchor count 2, 4 and 8), each at the anchor counts on both sides of its
bound, with and without the foreground index, as a sampler step and as a UniPC
step: bit for bit the builder followed by the stored-operator call."""
import numpy as np
import pytest
import torch

from test_gpu_limits import bits, sphere_problem

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def gc():
    import paper_2608_13255_amd as gc
    return gc


@pytest.mark.parametrize("C,dtype", [(4, torch.float32), (4, torch.bfloat16), (8, torch.float32), (16, torch.bfloat16),
                                     (12, torch.float32), (32, torch.bfloat16), (32, torch.float32)])
@pytest.mark.parametrize("a", [1, 2, 3, 4, 5, 8])
def test_variants_equal_the_stored_operator(gc, C, dtype, a):
    rs, P, cams = sphere_problem(5, 10, 37, 23, pinhole=True)
    P = P.copy()
    P[rs.random(P.shape[:-1]) < 0.1] = np.nan
    N, H, W = P.shape[1:4]
    A = sorted(rs.choice(N, a, replace=False).tolist())
    g = torch.Generator(device=DEV).manual_seed(a * 100 + C)
    lat = lambda n=N: (0.5 * torch.randn((1, n, H, W, C), generator=g, device=DEV)).to(dtype)  # noqa: E731
    prev, new, xt, xp, m2 = lat(), lat(a), lat(), lat(), lat()
    Pd, cd = torch.from_numpy(P).to(DEV), gc.camera_tensor(cams, DEV)
    bb = gc.gc_posmap_bbox(Pd, 0.05)
    corr, wts = gc.gc_build_correspondence(Pd, cd, A, 4, bb)
    assert int((corr != 0).sum()) > 0
    smp = gc.Sampler(kind=gc.GC_FLOW_EULER, pred_out=gc.GC_PRED_VEL)
    st = gc.gc_unipc_coeffs(gc.Sampler(), 10, 5)
    want = gc.gc_transport_reconstruct(prev, new, corr, wts, xt, A, smp, 0.6, 0.55)
    want_u = gc.gc_transport_unipc(prev, new, corr, wts, A, st, x_cur=xt, x_prev=xp, m_km2=m2)
    x0 = gc.gc_transport_step(prev, new, corr, wts, A)
    alone = gc.gc_unipc_update(st, x0, x_cur=xt, x_prev=xp, m_km2=m2, m_km1=prev)
    for w, y in zip(want_u, (x0,) + alone):
        assert torch.equal(bits(w), bits(y))
    for index in (None, gc.gc_index_foreground(Pd)):
        got = gc.gc_transport_reconstruct_geom(prev, new, Pd, cd, bb, xt, A, 4, smp, 0.6, 0.55, fg_index=index)
        got_u = gc.gc_transport_unipc_geom(prev, new, Pd, cd, bb, A, 4, st, x_cur=xt, x_prev=xp, m_km2=m2, fg_index=index)
        for w, y in zip(want + want_u, got + got_u):
            assert torch.equal(bits(w), bits(y))
