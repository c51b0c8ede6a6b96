"""Short block lists, which the column kernels hand to the workgroup-per-block kernel, around
the lengths where that ends (1024 blocks with one species, 1792 with more), and the rounding
conversions of 16-bit stores: every kernel gives the fields of the persistent kernel, which
does not change with the length, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rd():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2304_11165_amd import rd as rdmod

    return rdmod


def _run(rd, img, storage, species, kernel, fused=0):
    s = rd.Sim(rd.Geometry(img, None, 1.0, 8), storage)
    for i in range(species):
        s.add_species(1.0 - 0.25 * i)
        s.set_dirichlet(i, i, 0.5)
    if species > 1:
        s.add_reaction(0, 1, 0.125)
    s.set_rounding(1, seed=11)
    s.set_kernel(kernel, 8)
    if fused:
        s.set_fused_steps(fused)
    s.bind()
    rng = np.random.default_rng(5)
    for i in range(species):
        s.set_field(i, rng.random(img.shape, dtype=np.float32) * img)
    s.step(0.0625, 5)
    return [s.get_field(i).cpu().numpy() for i in range(species)]


@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("species,blocks", [(1, (1, 1, 1)), (1, (4, 16, 16)), (1, (5, 5, 41)),
                                            (2, (1, 1, 3)), (2, (7, 16, 16)), (2, (1, 11, 163))])
def test_lengths_agree(rd, storage, species, blocks):
    shape = tuple(8 * b for b in blocks)
    img = (np.random.default_rng(3).random(shape) < 0.6).astype(np.uint8)
    want = _run(rd, img, storage, species, "persistent")
    for kernel, fused in (("column", 0), ("column_xch", 0), ("column_xch", 4)):
        got = _run(rd, img, storage, species, kernel, fused)
        assert all(np.array_equal(g, w) for g, w in zip(got, want)), (kernel, fused)


# A step without diffusion rounds every voxel by itself, with random bits of its own: a voxel
# in FP16's normal range rounds alike in waves that hold only such values and zeros (the
# conversion instruction) and in waves that also hold smaller or larger ones (in software).
@pytest.mark.parametrize("kernel", ["block", "column", "persistent"])
def test_fp16_mixed_waves(rd, kernel):
    shape = (8, 64, 80)
    rng = np.random.default_rng(9)
    normal = np.exp2(rng.uniform(-13.5, 15.9, shape)).astype(np.float32)
    normal[rng.random(shape) < 0.2] = 0.0
    small = np.exp2(rng.uniform(-24.0, -14.5, shape)).astype(np.float32)
    other = rng.random(shape) < 0.3

    def run(field):
        s = rd.Sim(rd.Geometry(np.ones(shape, dtype=np.uint8), None, 1.0, 8), "fp16")
        s.add_species(0.0)
        s.add_reaction(0, -1, 0.25)
        s.set_rounding(1, seed=3)
        s.set_kernel(kernel, 8)
        s.bind()
        s.set_field(0, field)
        s.step(0.0625, 1)
        return s.get_field(0).cpu().numpy(), np.asarray(field, dtype=np.float16).astype(np.float64)

    a, a0 = run(np.where(other, 0.0, normal).astype(np.float32))
    b, b0 = run(np.where(other, small, normal).astype(np.float32))
    assert np.array_equal(a[~other], b[~other])
    for got, c in ((a, a0), (b, b0)):  # one of the two stored neighbours of the exact result
        exact = c * (1.0 - 0.25 * 0.0625)
        gap = np.maximum(np.exp2(np.floor(np.log2(np.maximum(exact, 2.0 ** -30))) - 10), 2.0 ** -24)
        assert np.all(np.abs(got - exact) < gap * (1.0 + 2.0 ** -10))


# More workgroups than seven per compute unit: a fused launch's grid stays within what is
# resident at once, whatever scalar registers its kernel uses.
def test_fused_grid_resident(rd):
    img = np.ones((8, 8 * 89, 8 * 89), dtype=np.uint8)  # 1981 groups of four blocks
    want = _run(rd, img, "fp32", 1, "persistent")
    got = _run(rd, img, "fp32", 1, "column", 4)
    assert np.array_equal(got[0], want[0])
