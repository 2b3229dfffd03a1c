"""Bricks whose level 1 holds more same-level references than the symbols
above L_0 fill dwords.  In the paired front kernel the replaying wave lists
those references over the decoding wave's copy of the symbols (436 dwords),
from its start on, while the decoding wave is at the L_0 symbols: it must not
copy these any more."""
import numpy as np
import pytest

COPIED = 436  # dwords of packed symbols that the decoding wave copies


def brick(seed):
    """Up to z = 12: groups of 4^3 voxels shifted by 2, so that all children
    of a 4^3 block but the last equal their lower neighbours.  Above: noise on
    part of the blocks of 2^3, for many L_0 symbols."""
    rng = np.random.default_rng(seed)
    v = np.ones((32, 32, 32), np.uint32)
    g = rng.integers(2, 14, (4, 9, 9)).astype(np.uint32)
    s = (np.arange(32) + 2) // 4
    v[:12] = g[np.ix_(s[:12], s, s)]
    noise = rng.integers(1, 9, (16, 8, 16)).astype(np.uint32)
    v[12:28, :8, :16] = noise
    return v


def ranges(orc, v):
    """(dwords of the symbols above L_0, dwords of the reference list, dwords
    of all symbols, palette entries)"""
    sym, cum, pal = orc.brick_symbols(v)
    c0, c1, c2, c3 = (int(c) for c in cum[:4])
    seg, seg2 = sym[c2:c1], sym[c3:c2]
    # expanded level-2 nodes: level 2's operations without the stop bit, after
    # its deltas (one for each operation 5)
    d = next(d for d in range(seg2.size % 8, seg2.size, 8) if np.count_nonzero((seg2[d:] & 7) == 5) == d)
    E = np.count_nonzero(seg2[d:] < 8)
    ops = (seg[seg.size - 8 * E:] & 7).reshape(E, 8)
    k = np.arange(8)
    nref = sum(np.count_nonzero((ops == a + 1) & (((k >> a) & 1) == 0)) for a in range(3))
    return c1 / 8, nref / 2, c0 / 8, len(pal)


@pytest.mark.parametrize("seed", [1, 2])
def test_references_reach_behind_the_copied_symbols(orc, seed):
    upper, refs, every, P = ranges(orc, brick(seed))
    assert upper + 8 < refs and upper + 8 < COPIED and every > refs and P <= 252


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 7, 300])
def test_small_batches_of_such_bricks(orc, n):
    from gpu_util import gpu_decode, gpu_decode_uniform
    import paper_2308_16619_amd as csv
    vol = np.concatenate([brick(s) for s in range(8)], axis=2)
    blob = csv.encode_volume(vol)
    pool = csv.Pool()
    pool.add_volume(blob)
    ids = np.arange(n, dtype=np.uint32) % 8
    print("[gpu-test] %d full-LOD requests" % n, flush=True)
    want = orc.decode_bricks(blob, ids, np.zeros(n, np.uint8))
    np.testing.assert_array_equal(gpu_decode_uniform(pool, ids, 0), want)
    lods = (np.arange(n) % 3).astype(np.uint8)
    got, _ = gpu_decode(pool, ids, lods)
    np.testing.assert_array_equal(got, orc.decode_bricks(blob, ids, lods))
