"""A field read on another stream than the simulation's: the tensor's readers on the caller's
stream come after the copy that fills it, and that copy after the readers of its memory."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_field_read_on_another_stream():
    import torch

    from paper_2304_11165_amd import rd

    shape = (40, 41, 48)
    img = np.ones(shape, np.uint8)
    c0, c1 = (torch.rand(shape, device="cuda") for _ in range(2))
    side = torch.cuda.Stream()
    s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp32")
    s.add_species(1.0)
    torch.cuda.synchronize()
    s.bind(stream=side)
    s.set_field(0, c0)
    out = torch.zeros(shape, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(50_000_000)  # a bounded wait of some 20 ms before the copy
    assert torch.equal(s.get_field(0, out).cpu(), c0.cpu())
    s.set_field(0, c1)
    torch.cuda.synchronize()
    torch.cuda._sleep(50_000_000)
    before = out.clone()  # reads the old field on the current stream ...
    after = s.get_field(0, out).clone()  # ... before it is overwritten
    assert torch.equal(before, c0) and torch.equal(after, c1)
