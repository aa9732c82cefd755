"""CPU test of the byte offsets that the FP16 odd step and the two-step passes
take their links from (kernels.hpp link_at and link_base): for every link of the
lattices they must be those of the tiled slots, below 4 GiB, at the nodes around tile
edges and up to the largest state."""
import random

import pytest

TILE = 2048


def _slot(pops, i, n):
    """Element of population i (from 1) of node n (kernels.hpp tiled)."""
    return ((((n // TILE) * pops) + i - 1) * TILE) + n % TILE


def _offsets(pops, size, i, io, n, m):
    """link_at and link_base with slot i of node m, slot io of node n."""
    tile = TILE * size
    apart = abs(i - io) * tile
    base = (min(i, io) - 1) * tile
    byte = m * size
    at = byte + (byte // tile) * ((pops - 1) * tile) + (apart if i > io else 0)
    own = _slot(pops, 1, n) * size + (apart if io > i else 0)
    assert byte // tile < 1 << 24 and (pops - 1) * tile < 1 << 24  # a 24-bit multiply
    assert max(at, own) < 1 << 32
    return base + at, base + own


@pytest.mark.parametrize("size", [2, 4, 8])
@pytest.mark.parametrize("pops", [18, 14, 6])
def test_link_offsets_are_those_of_the_tiled_slots(pops, size):
    rng = random.Random(pops * 10 + size)
    most = (1 << 32) // (pops * size) // TILE * TILE  # nodes of a 4 GiB region
    nodes = [0, 1, TILE - 1, TILE, TILE + 1, most // 2, most - TILE, most - 1]
    nodes += [rng.randrange(most) for _ in range(200)]
    for i in range(1, pops + 1):
        for io in range(1, pops + 1):
            if i == io:
                continue
            for n, m in zip(nodes, rng.sample(nodes, len(nodes))):
                at, own = _offsets(pops, size, i, io, n, m)
                assert at == _slot(pops, i, m) * size and own == _slot(pops, io, n) * size
