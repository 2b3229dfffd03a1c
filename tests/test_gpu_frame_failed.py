"""GPU: a frame that fails after its keys were given blocks (its bricks do not
fit the pool's memory budget for decoding) leaves a cache from which the next
frames serve what they decode themselves."""
import numpy as np
import pytest

import synth
from gpu_util import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stats", [True, False])
def test_frames_after_a_failed_one(orc, stats):
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = orc.encode_volume(synth.cells(n=256, grid=19, seed=2), scale_bits=10, lane_k=64)
    nb = 4 * 512

    def pool_of(budget):
        pool = csv.Pool(hbm_budget=budget)
        for _ in range(4):
            pool.add_volume(blob)
        return pool

    def frame(cache, ids, lods):
        return cache.frame(torch.from_numpy(ids.view(np.int32)).cuda(), torch.from_numpy(lods).cuda(), stats=stats)[0]

    rng = np.random.default_rng(5)
    few = rng.permutation(nb)[:700].astype(np.uint32)
    few_lods = rng.integers(0, 5, few.size).astype(np.uint8)
    free = pool_of(0)
    c = csv.FrameCache(free, 512 << 20, few.size)
    frame(c, few, few_lods)
    torch.cuda.synchronize()
    c.close()
    pool = pool_of(free.info()["device_bytes"] + (1 << 20))  # room for 700 bricks, not for all
    cache = csv.FrameCache(pool, 1 << 30, 5 * nb)
    every = np.tile(np.arange(nb, dtype=np.uint32), 5)
    every_lods = np.repeat(np.arange(5, dtype=np.uint8), nb)
    with pytest.raises(csv.CsvError) as e:
        frame(cache, every, every_lods)
    assert e.value.code == csv.CSV_ENOMEM
    for part in (slice(0, 700), slice(200, 600), slice(0, 650)):
        ids, lods = few[part].copy(), few_lods[part].copy()
        slots = frame(cache, ids, lods)
        torch.cuda.synchronize()
        slots = slots.cpu().numpy()
        assert (slots >= 0).all()
        for k in range(0, ids.size, 37):
            n = (32 >> int(lods[k])) ** 3
            np.testing.assert_array_equal(cache.read(slots[k], n),
                                          orc.decode_brick(blob, int(ids[k]) % 512, int(lods[k])).ravel())
    cache.close()
