"""The autotuning cache keeps apart what launches other kernels under the same setting: the
rounding (pairs of 16-bit steps depend on it) and a diffusivity factor."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_key_covers_rounding_and_factor(tmp_path):
    from paper_2304_11165_amd import rd

    img = (np.random.default_rng(1).random((24, 32, 40)) < 0.7).astype(np.uint8)
    cache = tmp_path / "tune.txt"

    def tuned(sround, factor, sink=0.0):
        s = rd.Sim(rd.Geometry(img, None, 1.0, 8), "fp16")
        s.add_species(1.0)
        s.set_rounding(sround, seed=1)
        s.bind(features=rd.RD_WS_DIFFUSIVITY)
        if factor:
            s.set_diffusivity(np.ones(img.shape, np.float32))
        if sink:
            s.set_sink(0, sink)
            s.set_sink_band(np.zeros(img.shape, np.float32), 1.0)
        s.autotune(0.0625, 8, cache_path=cache)
        return s.last_tune_from_cache

    forms = [(0, False), (1, False), (0, True), (1, True), (0, False, 0.5)]
    assert [tuned(*f) for f in forms] == [False] * 5
    assert [tuned(*f) for f in forms] == [True] * 5
    assert len(cache.read_text().splitlines()) == 5
