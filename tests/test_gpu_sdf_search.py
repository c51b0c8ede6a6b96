"""The signed distance's line passes (outward search) and its row pass (64-voxel chunks):
row lengths around the chunk size, lines in every direction, features many chunks away,
rows and planes without any; bit for bit against the oracle (squared distances are
integers)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rd():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2304_11165_amd import rd as rdmod

    return rdmod


def _image(shape, kind):
    rng = np.random.default_rng(hash(shape) % 1000)
    img = np.ones(shape, np.uint8)
    if kind == "corner":  # one feature voxel at the end of every axis
        img[-1, -1, -1] = 0
    elif kind == "two":
        img.flat[0] = 0
        img.flat[img.size // 2] = 0
    elif kind == "half":
        img[: (shape[0] + 1) // 2, : (shape[1] + 1) // 2] = 0
    else:
        img = (rng.random(shape) < {"sparse": 0.01, "dense": 0.5}[kind]).astype(np.uint8)
    return img


@pytest.mark.parametrize("kind", ["corner", "two", "half", "sparse", "dense"])
@pytest.mark.parametrize("shape", [(3, 5, 63), (2, 3, 64), (3, 2, 65), (2, 9, 128), (1, 2, 193), (5, 3, 300),
                                   (2, 301, 3), (301, 2, 3), (17, 31, 9), (33, 34, 35)])
def test_search_edges(rd, oracle_mod, shape, kind):
    img = _image(shape, kind)
    for im in (img, 1 - img):
        got = rd.sdf_from_image(im, 0.7).cpu().numpy()
        want = oracle_mod.signed_distance(im, 0.7)
        assert np.array_equal(got, want)
