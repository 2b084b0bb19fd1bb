"""The binding's short cuts on the way to a launch: the raw handle of torch's
current stream follows the stream context of each thread, a tensor that is not
a contiguous device tensor is refused as before, and a sampler's C form is not
shared, neither between samplers that differ nor with a caller that writes to
one."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def gc():
    import paper_2608_13255_amd as gc
    return gc


def test_raw_stream_follows_the_context(gc):
    torch.zeros(1, device=DEV)
    seen = []

    def check():
        side = torch.cuda.Stream()
        for s in (torch.cuda.default_stream(), side):
            with torch.cuda.stream(s):
                seen.append(gc._stream(None) == s.cuda_stream == torch.cuda.current_stream().cuda_stream)
        seen.append(gc._stream(side) == side.cuda_stream)

    check()
    th = threading.Thread(target=check)
    with torch.cuda.stream(torch.cuda.Stream()):   # another thread's context does not leak into this one
        th.start()
        th.join()
    assert len(seen) == 6 and all(seen)


def test_refused_tensors(gc):
    x = torch.zeros((1, 4, 8, 8, 4), device=DEV)
    smp = gc.Sampler(kind=gc.GC_FLOW_EULER)
    with pytest.raises(ValueError, match="device tensor"):
        gc.gc_sampler_reconstruct(x.cpu(), x.cpu(), smp, 0.5, 0.4)
    with pytest.raises(ValueError, match="contiguous"):
        gc.gc_sampler_reconstruct(x.transpose(2, 3)[..., 1:], x.transpose(2, 3)[..., 1:], smp, 0.5, 0.4)
    with pytest.raises(TypeError, match="torch.Tensor"):
        gc.gc_posmap_bbox(FakeMap())


class FakeMap:
    """Shaped like position maps, and no tensor."""
    dtype, shape, device = torch.float32, (1, 1, 2, 2, 3), DEV

    def dim(self):
        return 5


def test_sampler_structs_are_their_own(gc):
    x0 = torch.randn((1, 4, 8, 8, 4), device=DEV)
    xt = torch.randn_like(x0)
    outs = []
    for b in (0.02, 0.012, 0.02):
        outs.append(gc.gc_sampler_reconstruct(xt, x0, gc.Sampler(beta_end=b), 600, 500)[0])
        gc.Sampler(beta_end=b).c().beta_end = 0.5   # a struct of this caller's own
    assert torch.equal(outs[0], outs[2]) and not torch.equal(outs[0], outs[1])
    assert np.isfinite(outs[1].cpu().numpy()).all()
