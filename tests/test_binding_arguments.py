"""Arguments the binding refuses before any call, whatever it was asked before
(no GPU): a sampler field of another type, an empty gap list, an anchor count
that is no count; and a sampler's C form belongs to the caller that asked for
it and holds what the fields hold then."""
import numpy as np
import pytest
import torch


@pytest.fixture(scope="module")
def gc():
    import paper_2608_13255_amd as gc
    return gc


def test_sampler_fields_keep_their_types(gc):
    assert gc.Sampler(T=1000).c().T == 1000
    with pytest.raises(TypeError):
        gc.Sampler(T=1000.0).c()
    assert gc.gc_sampler_alpha_bar(gc.Sampler(beta_end=0.012), 500) != gc.gc_sampler_alpha_bar(gc.Sampler(), 500)


def test_sampler_struct_belongs_to_its_caller(gc):
    want = gc.gc_sampler_alpha_bar(gc.Sampler(), 9)
    mine = gc.Sampler().c()
    mine.T = 10                                    # of no other caller's concern
    assert gc.Sampler().c().T == 1000
    assert gc.gc_sampler_alpha_bar(gc.Sampler(), 9) == want


@pytest.mark.parametrize("scalar", [lambda x: torch.tensor(x, dtype=torch.float64), np.array],
                         ids=["tensor", "array"])
def test_sampler_fields_are_read_at_the_call(gc, scalar):
    beta = scalar(0.02)
    smp = gc.Sampler(beta_end=beta)
    assert gc.gc_sampler_alpha_bar(smp, 500) == gc.gc_sampler_alpha_bar(gc.Sampler(beta_end=0.02), 500)
    beta -= 0.008                                  # changed in place
    now = gc.Sampler(beta_end=float(beta))
    assert gc.gc_sampler_alpha_bar(smp, 500) == gc.gc_sampler_alpha_bar(now, 500)
    assert gc.gc_sampler_alpha_bar(smp, 500) != gc.gc_sampler_alpha_bar(gc.Sampler(), 500)
    assert gc.Sampler(T=np.array(500)).c().T == 500


def test_schedule_arguments(gc):
    with pytest.raises(gc.GeoCacheError) as e:
        gc.gc_schedule_advance_gaps([], [], False)
    assert gc.ERRORS[e.value.code] == "GC_ERR_CAPACITY"
    with pytest.raises(ValueError):
        gc.gc_schedule_anchors(6, -1, 0)
    with pytest.raises(gc.GeoCacheError):
        gc.gc_schedule_anchors(6, 100, 0)
    assert gc.gc_schedule_advance_gaps([0, 3, 1], [1], False) == [1, 0, 2]
    assert gc.gc_schedule_anchors(6, 2, 1) == [1, 4]
