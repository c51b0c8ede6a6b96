"""Two steps per launch against one step per launch of the persistent kernel, bit for bit:
boxes that end one voxel into a block, missing neighbour and edge blocks, walls, held faces,
odd step counts and graphs whose number of launches has to be made even; lists on both
sides of the length from which every form is paired (1024 blocks)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rd():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2304_11165_amd import rd as rdmod

    return rdmod


def _image(shape, fill, blocks):
    rng = np.random.default_rng(shape[0] * 7 + shape[2])
    img = rng.random(shape) < fill
    nb = [-(-n // 8) for n in shape]
    keep = rng.random(nb) < blocks
    keep[0, 0, 0] = True
    for ax in range(3):
        keep = keep.repeat(8, ax)
    img &= keep[: shape[0], : shape[1], : shape[2]]
    img[0, 0, 0] = True
    return img.astype(np.uint8)


def _run(rd, img, species, storage, sround, kernel, steps, gs, graph=True, xcd=False):
    s = rd.Sim(rd.Geometry(img, None, 1.0, 8), storage)
    s.add_species(1.0)
    s.add_reaction(0, -1, 0.0625)
    s.set_robin(0, 0.125)
    s.set_dirichlet(0, 0, 1.0)
    s.set_dirichlet(0, 3, 0.25)
    s.set_dirichlet(0, 5, 0.75)
    if species > 1:
        s.add_species(0.5)
        s.add_reaction(0, 1, 0.125)
        s.add_reaction(1, 0, 0.25)
        s.set_dirichlet(1, 1, 0.5)
        s.set_dirichlet(1, 4, 1.0)
    s.set_kernel(kernel, 8)
    s.set_launch(graph_steps=gs, use_graph=graph, xcd_map=xcd)
    s.set_rounding(sround, seed=7)
    s.bind()
    rng = np.random.default_rng(5)
    for i in range(species):
        s.set_field(i, rng.random(img.shape, dtype=np.float32) * img)
    out = []
    for n in steps:
        s.step(0.0625, n)
        out += [s.get_field(i).cpu().numpy() for i in range(species)]
    return out


@pytest.mark.parametrize("species", [1, 2])
@pytest.mark.parametrize("storage,sround", [("fp32", 0), ("fp32", 1), ("bf16", 0), ("bf16", 1), ("fp16", 0),
                                            ("fp16", 1)])
@pytest.mark.parametrize("shape,fill,blocks", [((8, 8, 8), 0.7, 1.0), ((1, 1, 1), 1.0, 1.0), ((9, 17, 25), 0.9, 1.0),
                                               ((40, 33, 41), 0.6, 0.6), ((88, 97, 105), 0.6, 0.6),
                                               ((90, 97, 104), 1.0, 0.9)])
def test_pairs_agree(rd, species, storage, sround, shape, fill, blocks):
    img = _image(shape, fill, blocks)
    steps = (2, 1, 5, 8)
    want = _run(rd, img, species, storage, sround, "persistent", steps, 8, False)
    for kernel, gs, graph, xcd in (("column", 8, False, False), ("column_xch", 2, True, False),
                                   ("column", 6, True, True), ("column", 4, True, False)):
        got = _run(rd, img, species, storage, sround, kernel, steps, gs, graph, xcd)
        assert all(np.array_equal(g, w) for g, w in zip(got, want)), (kernel, gs, graph)


# The adjoint keeps the last segment's states and recomputes the others', two steps per launch
# with the column kernels: any segment length (odd and even, one segment, single steps) gives
# the same states, hence the same sums, as single steps of the workgroup kernel.
@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("shape", [(9, 17, 25), (88, 97, 105)])
def test_adjoint_states(rd, storage, shape):
    img = _image(shape, 0.7, 0.9)
    rng = np.random.default_rng(2)
    c0 = rng.random(shape, dtype=np.float32) * img
    target = rng.random(shape, dtype=np.float32) * img

    def run(kernel, every):
        import torch

        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), storage)
        s.add_species(1.0)
        s.add_reaction(0, -1, 0.0625)
        s.set_dirichlet(0, 0, 1.0)
        s.set_kernel(kernel, 8)
        s.bind(features=rd.RD_WS_ADJOINT, checkpoint_slots=-(-9 // every) + every - 1)
        s.set_field(0, c0)
        got = s.adjoint(torch.as_tensor(target, device="cuda"), 9, 0.0625, every)
        return [float(v) for v in got], s.get_field(0).cpu().numpy()

    want = run("block", 4)
    for every in (1, 2, 3, 4, 9):
        got = run("column", every)
        assert got[0] == want[0] and np.array_equal(got[1], want[1]), every


# The same with a diffusivity factor (zeros among its values), against the kernel with one
# thread per slot, and the gradient with respect to the factor.
@pytest.mark.parametrize("storage,sround", [("fp32", 0), ("fp32", 1), ("bf16", 0), ("bf16", 1), ("fp16", 1)])
@pytest.mark.parametrize("shape,fill,blocks", [((8, 8, 8), 0.7, 1.0), ((1, 1, 1), 1.0, 1.0), ((9, 17, 25), 0.9, 1.0),
                                               ((40, 33, 41), 0.6, 0.6), ((90, 97, 104), 1.0, 0.9)])
def test_factor_pairs(rd, storage, sround, shape, fill, blocks):
    img = _image(shape, fill, blocks)
    rng = np.random.default_rng(8)
    e = rng.random(shape, dtype=np.float32)
    e[rng.random(shape) < 0.1] = 0.0
    c0 = rng.random(shape, dtype=np.float32) * img

    def run(kernel, steps, gs):
        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), storage)
        s.add_species(1.0)
        s.add_reaction(0, -1, 0.0625)
        s.set_robin(0, 0.125)
        s.set_dirichlet(0, 0, 1.0)
        s.set_dirichlet(0, 3, 0.25)
        s.set_dirichlet(0, 5, 0.75)
        s.set_kernel(kernel, 8)
        s.set_launch(graph_steps=gs, use_graph=True, xcd_map=False)
        s.set_rounding(sround, seed=7)
        s.bind(features=rd.RD_WS_DIFFUSIVITY)
        s.set_diffusivity(e)
        s.set_field(0, c0)
        out = []
        for n in steps:
            s.step(0.0625, n)
            out.append(s.get_field(0).cpu().numpy())
        return out

    want = run("block", (2, 1, 5, 8), 8)
    for kernel, gs in (("column", 4), ("column_xch", 6)):
        got = run(kernel, (2, 1, 5, 8), gs)
        assert all(np.array_equal(g, w) for g, w in zip(got, want)), kernel


@pytest.mark.parametrize("shape", [(9, 17, 25), (40, 33, 41)])
def test_adjoint_factor_states(rd, shape):
    import torch

    img = _image(shape, 0.7, 0.9)
    rng = np.random.default_rng(2)
    c0, target = (rng.random(shape, dtype=np.float32) * img for _ in range(2))
    e = rng.random(shape, dtype=np.float32)

    def run(every):
        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp32")
        s.add_species(1.0)
        s.add_reaction(0, -1, 0.0625)
        s.set_dirichlet(0, 0, 1.0)
        s.set_kernel("column", 8)
        s.bind(features=rd.RD_WS_ADJOINT | rd.RD_WS_DIFFUSIVITY, checkpoint_slots=-(-9 // every) + every - 1)
        s.set_diffusivity(e)
        s.set_field(0, c0)
        loss, gD, gk, ge = s.adjoint_factor(torch.as_tensor(target, device="cuda"), 9, 0.0625, every)
        return (loss, gD, gk), ge.cpu().numpy(), s.get_field(0).cpu().numpy()

    want = run(1)  # single steps only
    for every in (2, 4, 9):
        got = run(every)
        assert got[0] == want[0] and np.array_equal(got[1], want[1]) and np.array_equal(got[2], want[2]), every


# Direct launches inside a caller's own graph: an even number of steps leaves the two field
# buffers as they were, so that each replay goes on from the last one.
@pytest.mark.parametrize("factor", [False, True])
@pytest.mark.parametrize("steps", [2, 4, 6])
def test_callers_graph(rd, steps, factor):
    import torch

    shape = (24, 40, 33)
    img = _image(shape, 0.8, 0.9)
    rng = np.random.default_rng(6)
    c0 = rng.random(shape, dtype=np.float32) * img
    e = rng.random(shape, dtype=np.float32)

    def sim(stream):
        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp32")
        s.add_species(1.0)
        s.set_dirichlet(0, 1, 1.0)
        s.set_kernel("column", 8)
        s.set_launch(graph_steps=16, use_graph=False, xcd_map=False)
        s.bind(features=rd.RD_WS_DIFFUSIVITY if factor else 0, stream=stream)
        if factor:
            s.set_diffusivity(e)
        s.set_field(0, c0)
        torch.cuda.synchronize()
        return s

    eager = sim(torch.cuda.current_stream())
    side = torch.cuda.Stream()
    s = sim(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        s.step(0.0625, steps)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        eager.step(0.0625, steps)
        want = eager.get_field(0).cpu().numpy()
        assert np.array_equal(s.get_field(0).cpu().numpy(), want)
        torch.cuda.synchronize()


# The same with eager work on the captured simulation itself between the replays: an even
# number of steps leaves the buffers as they were eagerly, too (direct launches, a replayed
# graph of the library with direct launches after it), from the capture on.
@pytest.mark.parametrize("factor", [False, True])
@pytest.mark.parametrize("captured,between", [(2, 2), (4, 6), (2, 18), (6, 22)])
def test_replay_after_eager_steps(rd, captured, between, factor):
    import torch

    shape = (24, 40, 33)
    img = _image(shape, 0.8, 0.9)
    rng = np.random.default_rng(6)
    c0 = rng.random(shape, dtype=np.float32) * img
    e = rng.random(shape, dtype=np.float32)

    def sim(stream, kernel):
        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp32")
        s.add_species(1.0)
        s.set_dirichlet(0, 1, 1.0)
        s.set_kernel(kernel, 8)
        s.set_launch(graph_steps=16, use_graph=True, xcd_map=False)
        s.bind(features=rd.RD_WS_DIFFUSIVITY if factor else 0, stream=stream)
        if factor:
            s.set_diffusivity(e)
        s.set_field(0, c0)
        torch.cuda.synchronize()
        return s

    single = sim(torch.cuda.current_stream(), "block")
    side = torch.cuda.Stream()
    s = sim(side, "column")
    for n in (2, 1):
        s.step(0.0625, n)
        single.step(0.0625, n)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        s.step(0.0625, captured)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        s.step(0.0625, between)
        torch.cuda.synchronize()
        single.step(0.0625, captured + between)
        want = single.get_field(0).cpu().numpy()
        with torch.cuda.stream(side):  # the copy to the host waits for the simulation's stream
            got = s.get_field(0).cpu().numpy()
        assert np.array_equal(got, want)


# An adjoint leaves the buffers as its number of steps does, whatever its segments: here 8
# steps in segments of 5 (5 + 3), 3 (3 + 3 + 2) and 8.
@pytest.mark.parametrize("factor", [False, True])
@pytest.mark.parametrize("every", [3, 5, 8])
def test_replay_after_adjoint(rd, every, factor):
    import torch

    shape = (24, 40, 33)
    img = _image(shape, 0.8, 0.9)
    rng = np.random.default_rng(6)
    c0, target, e = (rng.random(shape, dtype=np.float32) * img for _ in range(3))
    target = torch.as_tensor(target, device="cuda")

    def sim(stream, kernel, features=0):
        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp32")
        s.add_species(1.0)
        s.set_dirichlet(0, 1, 1.0)
        s.set_kernel(kernel, 8)
        s.bind(features=features | (rd.RD_WS_DIFFUSIVITY if factor else 0), stream=stream,
               checkpoint_slots=-(-8 // every) + every - 1 if features else 0)
        if factor:
            s.set_diffusivity(e)
        s.set_field(0, c0)
        torch.cuda.synchronize()
        return s

    single = sim(torch.cuda.current_stream(), "block")
    side = torch.cuda.Stream()
    s = sim(side, "column", rd.RD_WS_ADJOINT)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        s.step(0.0625, 4)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            s.adjoint(target, 8, 0.0625, every)
        torch.cuda.synchronize()
        single.step(0.0625, 4 + 8)
        want = single.get_field(0).cpu().numpy()
        with torch.cuda.stream(side):
            got = s.get_field(0).cpu().numpy()
        assert np.array_equal(got, want)


# A captured copy of the field (or into it) holds the buffer's address as captured steps do.
@pytest.mark.parametrize("call", ["get", "set"])
@pytest.mark.parametrize("between", [2, 6, 18])
def test_replay_of_copies(rd, between, call):
    import torch

    shape = (24, 40, 33)
    img = _image(shape, 0.8, 0.9)
    rng = np.random.default_rng(6)
    c0, c1 = (torch.as_tensor(rng.random(shape, dtype=np.float32) * img, device="cuda") for _ in range(2))

    def sim(stream, kernel):
        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp32")
        s.add_species(1.0)
        s.set_kernel(kernel, 8)
        s.set_launch(graph_steps=16, use_graph=True, xcd_map=False)
        s.bind(stream=stream)
        s.set_field(0, c0)
        torch.cuda.synchronize()
        return s

    single = sim(torch.cuda.current_stream(), "block")
    side = torch.cuda.Stream()
    s = sim(side, "column")
    out = torch.zeros(shape, device="cuda")
    act = torch.as_tensor(img, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        s.get_field(0, out) if call == "get" else s.set_field(0, c1)
    for _ in range(2):
        s.step(0.0625, between)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        single.step(0.0625, between)
        if call == "set":
            single.set_field(0, c1)
            s.step(0.0625, between)
            single.step(0.0625, between)
            s.get_field(0, out)
        torch.cuda.synchronize()
        assert torch.equal(out * act, single.get_field(0) * act)
