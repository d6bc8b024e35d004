"""The tile lists of an ordered sweep (kListWords and make_lists in paper_1905_12799_amd/csrc/kmeans_lloyd.hip), as a model: how they are
packed, what a slab meets, and how the step that a key holds becomes a tile again (steps_to_tiles there).  test_gpu_ordered.py shows
which lists occur."""
import os
import re

import numpy as np
import pytest

SOURCE = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1905_12799_amd", "csrc", "kmeans_lloyd.hip")).read()
HEAD = int(re.search(r"kListHead = (\d+);", SOURCE).group(1))
ALL_MORE = int(re.search(r"kAllMore = (0x[0-9a-f]+)u;", SOURCE).group(1), 16)
MAX_TILES = int(re.search(r"kListMaxTiles = (\d+);", SOURCE).group(1))


def list_entry(head, more, e):
    return ((head if e < HEAD or e == 15 else more) >> (4 * (e if e < HEAD else (7 if e == 15 else e - HEAD)))) & 15


def pack(masks, n_tiles, others_longest=1):
    """The words of one unit: `masks` names the tiles of its eight slots, `others_longest` is the longest list of the units that are
    packed with it.  Returns head [8], more [8] (None: not written) and the length."""
    longest = max(max(bin(m).count("1") for m in masks), 1)
    if longest > HEAD and longest == n_tiles - 1:
        longest = n_tiles
    everything = (1 << n_tiles) - 1
    wave = max(longest, others_longest)
    heads, mores = [], []
    for m in masks:
        m = everything if longest == n_tiles else m
        m |= (everything & ~m) << 16

        def take():
            nonlocal m
            e = ((m & -m).bit_length() - 1) & 15                     # (none left: 15)
            m &= m - 1 if m else 0
            return e

        head, more = (longest - 1) << 28, 0
        for i in range(min(HEAD, wave)):
            head |= take() << (4 * i)
        if wave > HEAD:
            for i in range(8):
                more |= take() << (4 * i)
        heads.append(head & 0xFFFFFFFF)
        mores.append(more if wave > HEAD else None)
    return heads, mores, longest


def read(heads, mores, n_tiles):
    """The tiles that each slot meets, step by step."""
    n = (heads[0] >> 28) + 1
    out = []
    for head, more in zip(heads, mores):
        if n > HEAD:
            more = ALL_MORE if n == n_tiles else more
        out.append([list_entry(head, more, e) for e in range(n)])
    return out


@pytest.mark.parametrize("n_tiles", range(3, MAX_TILES + 1))
def test_lists_of_every_length(n_tiles):
    """Every slot meets the tiles of its list, each once, in as many steps as the longest list takes; a list of all tiles is them in order."""
    rng = np.random.default_rng(n_tiles)
    met = set()
    for longest in range(1, n_tiles + 1):
        for others in (1, HEAD, n_tiles):
            lengths = rng.integers(0, longest + 1, 8)
            lengths[rng.integers(8)] = longest
            masks = [sum(1 << int(t) for t in rng.choice(n_tiles, n, replace=False)) for n in lengths]
            heads, mores, packed = pack(masks, n_tiles, others)
            steps = read(heads, mores, n_tiles)
            met.add(len(steps[0]))
            assert packed == len(steps[0]) and packed in (longest, n_tiles) and (packed == longest or longest == n_tiles - 1 > HEAD - 1)
            for mask, tiles in zip(masks, steps):
                assert len(set(tiles)) == len(tiles) == packed and max(tiles) < n_tiles
                assert all(mask >> t & 1 == 0 or t in tiles for t in range(n_tiles))
            if packed == n_tiles:
                assert all(tiles == list(range(n_tiles)) for tiles in steps)
    assert met >= set(range(1, min(HEAD, n_tiles) + 1)) | {n_tiles}


def key_bits(indices):
    return (indices - 1).bit_length() if indices > 1 else 0


@pytest.mark.parametrize("S", [1, 2, 4, 8])
def test_a_step_becomes_the_tile_its_slot_met(S):
    """Keys of every step, quad of the run and row, over anything in the bits above: the index within the run that comes out."""
    rng = np.random.default_rng(S)
    shift = {1: 2, 2: 3, 4: 4, 8: 5}[S]
    tile_mask = (15 << shift) & 127
    final = 0x3F if S == 1 else 0x7F
    for n_tiles in range(3, {1: 16, 2: 16, 4: 8, 8: 4}[S] + 1):
        for longest in range(1, n_tiles + 1):
            masks = [sum(1 << int(t) for t in rng.choice(n_tiles, longest, replace=False)) for _ in range(8)]
            heads, mores, _ = pack(masks, n_tiles)
            steps = read(heads, mores, n_tiles)
            n_it = len(steps[0])
            bits = 7 if S == 8 else key_bits(4 * S * n_it)
            assert 4 * S * n_it <= 1 << bits
            for hl in (0, 1):                                        # the half-wave owns slots 4 hl .. 4 hl + 3
                for a in range(4):
                    for step in range(n_it):
                        row = int(rng.integers(4))
                        quad = 4 * a if S >= 4 else (4 * (a & 1) if S == 2 else 0)       # (key_index: bit 4, the half, is added later at S = 8)
                        key = (int(rng.integers(1 << 24)) << bits) | (step << shift) | quad | row
                        m1 = key
                        if n_it <= HEAD or not (S < 8 and n_it == n_tiles):
                            at = ((m1 >> shift) & ((((1 << bits) - 1) >> shift))) if bits > shift else 0
                            # the slot is picked by the key's own bits
                            slot = a if S == 1 else ((2 * (a >> 1) + (m1 >> 2 & 1)) if S == 2 else (m1 >> 2 & 1) + 2 * (m1 >> 3 & 1))
                            assert slot == a
                            tile = list_entry(heads[4 * hl + slot], ALL_MORE if n_it == n_tiles else mores[4 * hl + slot], at)
                            m1 = ((tile << shift) & tile_mask) | (m1 & ~tile_mask)
                        else:
                            m1 &= (1 << bits) - 1
                        want = (steps[4 * hl + a][step] << shift) | quad | row
                        assert m1 & final == want & final == want
