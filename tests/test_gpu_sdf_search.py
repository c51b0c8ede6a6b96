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


# Flat and thin images whose passes need 2^24 workgroups or more (2^32 threads, more than one
# dimension of a grid holds), up to the limit of 32768 voxels an edge: planes of the other
# phase 64 voxels apart, so that the distances are known.
@pytest.mark.parametrize("shape,axis", [((32768, 1, 32768), 0), ((1, 32768, 32768), 1), ((8192, 8192, 1), 0)])
def test_search_flat_images(rd, shape, axis):
    import torch

    img = torch.ones(shape, dtype=torch.uint8, device="cuda")
    img.movedim(axis, 0)[::64] = 0
    got = rd.sdf_from_image(img, 0.5)
    k = torch.arange(shape[axis], device="cuda")
    near = torch.minimum(k % 64, torch.where(k // 64 * 64 + 64 < shape[axis], 64 - k % 64, k))
    want = torch.where(k % 64 == 0, -0.25, 0.5 * (near.double() - 0.5)).float()
    want = want.reshape([-1 if a == axis else 1 for a in range(3)])
    for z in range(0, shape[0], 4096):
        assert bool((got[z : z + 4096] == (want[z : z + 4096] if axis == 0 else want)).all())


# Lines searched with summaries of 64 and 512 rows: lengths around their multiples, both axes,
# features at the ends, in the middle and hundreds of rows apart.
@pytest.mark.parametrize("kind", ["corner", "two", "half", "sparse", "far"])
@pytest.mark.parametrize("n", [513, 575, 577, 1024, 1031, 2049])
def test_search_long_lines(rd, oracle_mod, n, kind):
    for shape in ((n, 3, 70), (2, n, 9), (n, n // 8 + 1, 1)):
        if kind == "far":
            img = np.ones(shape, np.uint8)
            img.flat[np.random.default_rng(n).integers(0, img.size, 5)] = 0
        else:
            img = _image(shape, kind)
        for im in (img, 1 - img):
            got = rd.sdf_from_image(im, 0.7).cpu().numpy()
            assert np.array_equal(got, oracle_mod.signed_distance(im, 0.7)), shape
