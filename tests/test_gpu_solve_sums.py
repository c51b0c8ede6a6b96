"""Sums of the steady-state solver over block lists around its dispatch edges: up to 4096
blocks one workgroup sums all rows, above that ranges of rows and a ticket.  The batch of one
geometry always takes the one-workgroup form, so both must reach the same tortuosity (each
to a relative residual of 1e-8, i.e. within 2e-6 of the exact value in tau)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rd():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2304_11165_amd import rd as rdmod

    return rdmod


# blocks per axis (z, y, x): 4096, 4097 (ragged last range), 4352, and more rows per range
# than one pass of a workgroup's threads takes (66049 blocks: 259 rows)
@pytest.mark.parametrize("blocks", [(16, 16, 16), (1, 17, 241), (16, 16, 17), (1, 257, 257)])
def test_sums_agree(rd, blocks):
    shape = tuple(8 * b for b in blocks)
    rng = np.random.default_rng(sum(blocks))
    img = (rng.random(shape) < 0.7).astype(np.uint8)
    img[::8, ::8, ::8] = 1  # every block is stored
    g = rd.Geometry(img, None, 1.0, 8)
    assert g.stats()["n_blocks"] == int(np.prod(blocks))
    axis = 2 if blocks[0] > 1 else 1
    s = rd.Sim(g, "fp32")
    s.add_species(1.0)
    s.bind(features=rd.RD_WS_SOLVER)
    one = s.steady_state(axis, 1e-8)
    tau, rel, _ = rd.Batch([g], "fp32").bind().tortuosity(axis, 1e-8)
    assert one["converged"] and rel[0] <= 1e-8
    assert abs(one["tau"] - tau[0]) <= 4e-6 * tau[0]
    again = s.steady_state(axis, 1e-8)  # a second solve starts from a clean ticket
    assert again["tau"] == one["tau"] and again["iters"] == one["iters"]
