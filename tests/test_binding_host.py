"""The binding's output tensors, without a GPU."""

import pytest
import torch

import paper_2608_28726_amd as pr


@pytest.mark.parametrize("alloc", [pr._alloc_features, pr._alloc_agg])
@pytest.mark.parametrize("n", [0, 1, 5, 8])
def test_outputs_are_tensors_of_their_own(alloc, n):
    """Outputs of one call share an allocation, and nothing else: each can be
    written in place, also with a tensor that requires a gradient, detached in
    place and saved for a backward pass, whatever is done to the others."""
    out = alloc(n, torch.device("cpu"))
    spans = []
    for k, t in out.items():
        assert t.shape[0] == n and t.is_contiguous() and t.data_ptr() % 16 == 0, k
        assert not t._is_view() and t._version == 0, k
        spans.append((t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()))
    spans.sort()
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))
    names = [k for k, t in out.items() if t.dtype == torch.float32]
    for k in names:
        out[k].fill_(0.5)
    w = torch.ones_like(out[names[0]], requires_grad=True)
    loss = (out[names[0]] * w).sum()
    out[names[1]].neg_()
    out[names[2]].detach_()
    loss.backward()
    assert bool((w.grad == 0.5).all())
    out[names[1]].mul_(w if out[names[1]].shape == w.shape else 2.0)
    assert bool((out[names[1]] == -0.5 * (1 if out[names[1]].shape == w.shape else 2)).all())
    assert bool((out[names[0]] == 0.5).all()) and bool((out[names[2]] == 0.5).all())
