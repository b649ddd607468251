"""The shipped tuning cache is what the present autotuner writes: every entry
tried the present candidates and chose among them."""
import json

import pytest

pytest.importorskip("torch")
from paper_1710_03197_amd import autotune as at  # noqa: E402

ENTRIES = json.load(open(at.SHIPPED_CACHE))


@pytest.mark.parametrize("key", sorted(ENTRIES))
def test_entry_is_the_tuners(key):
    entry = ENTRIES[key]
    d = int(key.split("|")[1][1:])
    shapes = len(at.TILE_CANDIDATES[d])
    assert set(entry) == {"options", "ms_pair", "default_ms_pair", "tried"}
    if d == 2:  # (every 2D candidate makes a plan; in 3D some tiles are refused)
        assert entry["tried"] == (shapes * len(at.CHUNK_CANDIDATES) + len(at.SAMPLE_CANDIDATES) +
                                  len(at.FFT_GROUP_CANDIDATES) + len(at.RADIX_CANDIDATES) + 2)
    opt = dict(entry["options"])
    assert tuple(opt.pop("tile")) in at.TILE_CANDIDATES[d]
    assert opt.pop("grid_chunk") in at.CHUNK_CANDIDATES
    assert opt.pop("fft_groups") in at.FFT_GROUP_CANDIDATES
    assert opt.pop("fft_radix", 1) in at.RADIX_CANDIDATES
    assert opt.pop("fuse_reduce", 1) in (1, 2)
    assert opt.pop("grid_waves", 1) == 1 or d == 3
    for name, value in opt.items():
        assert {name: value} in at.SAMPLE_CANDIDATES, name
