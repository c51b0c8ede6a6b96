"""The order of the step's workgroups over the XCDs (list order, contiguous eighths, runs of
64 groups) around the sizes where it changes: every block is stepped exactly once, so the
fields equal those of the persistent kernel, which walks the list itself, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rd():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2304_11165_amd import rd as rdmod

    return rdmod


def _run(rd, img, edge, kernel, xcd, layout="blocks", factor=None):
    s = rd.Sim(rd.Geometry(img, None, 1.0, edge), "fp32")
    s.add_species(1.0)
    s.set_dirichlet(0, 0, 1.0)
    if layout == "compact":
        s.set_layout("compact")
    if edge == 8:
        s.set_kernel(kernel)
    s.set_launch(graph_steps=4, use_graph=True, xcd_map=xcd)
    s.bind(features=rd.RD_WS_DIFFUSIVITY if factor is not None else 0)
    if factor is not None:
        s.set_diffusivity(factor)
    rng = np.random.default_rng(5)
    s.set_field(0, rng.random(img.shape, dtype=np.float32) * img)
    s.step(0.1, 5)
    return s.get_field(0).cpu().numpy()


# 8^3 blocks: 63, 64 and 65 groups of four, one eighth of 512 groups, more than that, ragged
@pytest.mark.parametrize("blocks", [(1, 4, 63), (4, 8, 8), (1, 4, 65), (1, 128, 128), (1, 128, 129), (3, 71, 83)])
def test_orders_agree(rd, blocks):
    shape = tuple(8 * b for b in blocks)
    img = (np.random.default_rng(3).random(shape) < 0.6).astype(np.uint8)
    want = _run(rd, img, 8, "persistent", False)
    for kernel in ("block", "column", "column_xch"):
        for xcd in (False, True):
            assert np.array_equal(_run(rd, img, 8, kernel, xcd), want), (kernel, xcd)
    assert np.array_equal(_run(rd, img, 8, "column_lanes", False, "compact"), want)
    small = img[:, : 8 * min(blocks[1], 40)]
    want = _run(rd, small, 8, "persistent", False)
    assert np.array_equal(_run(rd, small, 4, None, False), want)
    e = np.random.default_rng(7).random(small.shape, dtype=np.float32)
    want = _run(rd, small, 8, "block", False, factor=e)  # one thread per slot
    for xcd in (False, True):
        assert np.array_equal(_run(rd, small, 8, "column_xch", xcd, factor=e), want)
