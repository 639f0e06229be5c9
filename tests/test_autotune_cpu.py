"""The autotuner's cache (CPU): a launch chosen with another build of the
library is not applied, one chosen with this build is."""
import json
import types

import pytest
import torch  # noqa: F401  (before the library: both have to find one HIP runtime)

from paper_1010_3816_amd import autotune, binding


class _Grid:
    """What tune_grid asks of a grid, with the launches it sets."""

    def __init__(self):
        props = types.SimpleNamespace(name="gpu", gcnArchName="gfx950", multi_processor_count=256)
        self.torch = types.SimpleNamespace(cuda=types.SimpleNamespace(get_device_properties=lambda d: props))
        self.device, self.nr, self.ntheta, self.handle, self.stream = 0, 1600, 128, None, None
        self.params = types.SimpleNamespace(coef_mode=binding.TEUK_COEF_KERR)
        self.now, self.calls = (2, 4, 0, 0), []

    def tile(self):
        return self.now[:2]

    def block_launch(self):
        return self.now[2:]

    def set_tile(self, r, w):
        self.now = (r, w) + self.now[2:]
        self.calls.append(self.now)

    def set_block_launch(self, k, c):
        self.now = self.now[:2] + (k, c)


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "launch.json"
    monkeypatch.setenv("TEUK_TUNE_CACHE", str(path))
    return path


def test_entry_of_another_build_is_not_applied(cache, monkeypatch):
    # the default launch is the fastest now; the file holds another one, from an
    # earlier version of the library, under the keys without and with a build
    stale = {"rows": 16, "waves": 2, "block": 0, "cols": 0, "ms": 1.0}
    cache.write_text(json.dumps({"grid|gfx950/256cu|1600x128": stale,
                                 "grid|gfx950/256cu|0123456789abcdef|1600x128": stale}))
    g = _Grid()
    monkeypatch.setattr(autotune, "_time", lambda *a: 1.0 if g.now == (2, 4, 0, 0) else 2.0)
    out = autotune.tune_grid(g)
    assert "cached" not in out and g.now == (2, 4, 0, 0)
    # and the choice of this build is applied without timing anything
    monkeypatch.setattr(autotune, "_time", lambda *a: pytest.fail("timed"))
    h = _Grid()
    assert autotune.tune_grid(h)["cached"] and h.now == (2, 4, 0, 0) and len(h.calls) == 1


def test_heights_fill_rounds_of_the_passes_strips(cache, monkeypatch):
    g = _Grid()
    monkeypatch.setattr(autotune, "_time", lambda *a: 1.0)
    tried = {e["rows"] for e in autotune.tune_grid(g, use_cache=False)["table"]}
    assert set(autotune.round_rows(1600, 128, 256, 58)) <= tried
