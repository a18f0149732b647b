"""The weight loads that run ahead of their use stay inside the stored weights.

The offsets below are the kernels' own rules (host/device functions), run over every load of
a workgroup: the layers, K blocks and waves of the residual network, and the class tiles that
a wave of the plain networks visits, with the ones past the last that its prefetch names."""
import numpy as np
import pytest

from tests import _internal

BODY = """
extern "C" unsigned weight_at(unsigned l, unsigned wave, unsigned kb, unsigned nb) { return res_weight_at(l, wave, kb, nb); }
extern "C" unsigned bias_row(unsigned l, unsigned nb) { return res_bias_row(l, nb); }
extern "C" unsigned tile_of(unsigned ct, unsigned classes) { return class_tile(ct, classes); }
extern "C" unsigned turn_count(unsigned w, unsigned tiles, unsigned cols) { return turns(w, tiles, cols); }
extern "C" unsigned turn_of(unsigned i, unsigned w, unsigned tiles, unsigned cols) { return turn_tile(i, w, tiles, cols); }
extern "C" unsigned column_of(unsigned i, unsigned w, unsigned tiles, unsigned cols) { return turn_column(i, w, tiles, cols); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _internal.compile_host(str(tmp_path_factory.mktemp("internal")), BODY)


@pytest.mark.parametrize("nb", [1, 2, 6, 16])
def test_residual_network(lib, nb):
    layers = 2 * nb
    seen = set()
    for wave in range(8):
        loads = [(0, 0), (0, 1)]                       # the tile's start
        for l in range(layers):
            loads += [(l, kb + 2) for kb in range(14)] + [(l + 1, 1), (l + 1, 0)]
        for l, kb in loads:
            at = lib.weight_at(l, wave, kb, nb)
            assert at % 4096 == 0 and at + 4096 <= layers * 512 * 512 * 2, (l, wave, kb)
            if l < layers:
                seen.add(at)
    assert len(seen) == layers * 128                   # every 4 KB piece has its own place
    for l in range(layers + 1):                        # the next layer's biases, once per layer
        row = lib.bias_row(l, nb)
        assert 1 <= row < 1 + layers and (l == layers or row == 1 + l)


@pytest.mark.parametrize("C", [33, 48, 49, 64, 65, 144, 256, 257, 387, 512])
def test_plain_network_class_tiles(lib, C):
    stored = 2 * -(-C // 32)
    visited = []
    for wave in range(8):
        ct, named = wave, [wave]                       # loaded before the first tile
        while ct < -(-C // 16):
            visited.append(lib.tile_of(ct, C))
            ct += 8
            named.append(ct)                           # loaded during the tile before
        assert all(0 <= lib.tile_of(t, C) < stored for t in named), (wave, named)
    assert sorted(visited) == list(np.arange(-(-C // 16)))


@pytest.mark.parametrize("C", [33, 48, 49, 64, 65, 112, 113, 128, 129, 144, 256, 257, 387, 512])
def test_turns_over_the_class_tiles(lib, C):
    """Eight waves that share class tiles by turns (four header columns): every tile meets every
    column once, no wave has two turns more than another, and the tile named ahead is stored."""
    tiles, cols, stored = -(-C // 16), 4, 2 * -(-C // 32)
    seen, count = [], []
    for wave in range(8):
        n = lib.turn_count(wave, tiles, cols)
        count.append(n)
        for i in range(n + 1):
            tile = lib.turn_of(i, wave, tiles, cols)
            assert 0 <= lib.tile_of(tile, C) < stored
            if i < n:
                assert tile < tiles
                seen += [(tile, c) for c in (range(cols) if i < tiles // 8 else [lib.column_of(i, wave, tiles, cols)])]
    assert sorted(seen) == [(t, c) for t in range(tiles) for c in range(cols)]
    assert max(count) - min(count) <= 1
