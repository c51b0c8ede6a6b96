"""Copies between dense fields and block storage (8^3: two planes per wave up to 2048 blocks,
eight above) and the one-launch finish of the FP64 sums, around the sizes where their dispatch
changes: part blocks at the box edges, list lengths around 4096 rows (one workgroup) and above
(ranges and a ticket, which must be back at 0 for the next sum)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rd():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2304_11165_amd import rd as rdmod

    return rdmod


@pytest.mark.parametrize("layout", ["blocks", "compact"])
@pytest.mark.parametrize("storage", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (7, 9, 8), (17, 8, 33), (40, 41, 263), (64, 128, 128), (5, 22, 5457)])
def test_round_trip(rd, shape, storage, layout):
    import torch

    rng = np.random.default_rng(1)
    img = (rng.random(shape) < 0.6).astype(np.uint8)
    img.flat[0] = 1
    s = rd.Sim(rd.Geometry(img, None, 1.0, 8), storage)
    s.add_species(1.0)
    s.set_dirichlet(0, 2, 0.25)
    s.set_dirichlet(0, 3, 0.5)  # the higher face wins where a box is one voxel thick
    s.set_layout(layout)
    s.bind()
    f = torch.as_tensor(rng.random(shape, dtype=np.float32), device="cuda").bfloat16().float()  # exact in BF16
    s.set_field(0, f)
    want = f.cpu().numpy() * img
    want[:, 0][img[:, 0] != 0] = 0.25
    want[:, -1][img[:, -1] != 0] = 0.5
    assert np.array_equal(s.get_field(0).cpu().numpy(), want)


# rows of the balance: one per four blocks; of the region mass: one per block
@pytest.mark.parametrize("blocks", [(16, 16, 16), (1, 17, 241), (16, 32, 32), (5, 41, 81)])
def test_sums_repeat(rd, blocks):
    shape = tuple(8 * b for b in blocks)
    img = (np.random.default_rng(2).random(shape) < 0.5).astype(np.uint8)
    s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp32")
    s.add_species(1.0)
    s.set_dirichlet(0, 0, 1.0)
    s.bind()
    c = np.random.default_rng(4).random(shape, dtype=np.float32) * img
    s.set_field(0, c)
    c[:, :, 0] = img[:, :, 0]
    free = c.astype(np.float64)
    free[:, :, 0] = 0.0
    region = [1, shape[2] - 1, 0, shape[1], 0, shape[0]]
    inside = c.astype(np.float64)[:, :, 1:-1].sum()
    jump = ((c[:, :, 0].astype(np.float64) - c[:, :, 1]) * img[:, :, 0] * img[:, :, 1]).sum()
    for _ in range(3):
        b = s.balance(0)
        assert b["mass"] == pytest.approx(free.sum(), rel=1e-12)
        assert b["inflow"][0] == pytest.approx(jump, rel=1e-12) and not b["inflow"][1:].any()
        assert s.region_mass(0, region) == pytest.approx(inside, rel=1e-12)
        assert s.plane_flux(0, 0, 0) == pytest.approx(jump, rel=1e-12)


def test_adjoint_block_edges(rd):
    """The adjoint's blocks are each visited once whatever the list length (8^3, in an order
    over the XCDs) -- the gradients equal those of 4^3 blocks up to the order of FP64 sums."""
    for blocks in [(1, 4, 63), (3, 5, 17), (2, 9, 16)]:
        shape = tuple(8 * b for b in blocks)
        img = (np.random.default_rng(6).random(shape) < 0.6).astype(np.uint8)
        out = []
        for edge in (8, 4):
            s = rd.Sim(rd.Geometry(img, None, 1.0, edge), "fp32")
            s.add_species(0.8)
            s.add_reaction(0, -1, 0.02)
            s.set_dirichlet(0, 0, 1.0)
            s.bind(features=rd.RD_WS_ADJOINT, checkpoint_slots=6)
            s.set_field(0, np.random.default_rng(8).random(shape, dtype=np.float32) * img)
            out.append(s.adjoint(np.zeros(shape, np.float32), 8, 0.1, 3))
        assert out[0] == pytest.approx(out[1], rel=1e-11)
