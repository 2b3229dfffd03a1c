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


def test_a_frame_captured_after_a_failed_one(orc):
    # the graph's own reset has not run when the next frame is a call
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = orc.encode_volume(synth.cells(n=256, grid=19, seed=2), scale_bits=10, lane_k=64)
    pool = csv.Pool()
    pool.add_volume(blob)
    rng = np.random.default_rng(6)
    n = 300
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    lods = torch.zeros(n, dtype=torch.uint8, device="cuda")
    slots = torch.zeros(n, dtype=torch.int64, device="cuda")
    cache = csv.FrameCache(pool, 256 << 20, n)
    limited = csv.Pool(hbm_budget=pool.info()["device_bytes"] + (64 << 10))  # no room for a decode's buffers
    limited.add_volume(blob)
    failing = csv.FrameCache(limited, 256 << 20, n)

    def fill():
        ids.copy_(torch.from_numpy(rng.integers(0, 512, n).astype(np.int32)))
        lods.copy_(torch.from_numpy(rng.integers(0, 5, n).astype(np.uint8)))
        slots.fill_(-2)
        torch.cuda.synchronize()

    def check(c):
        torch.cuda.synchronize()
        i, t, at = ids.cpu().numpy(), lods.cpu().numpy(), slots.cpu().numpy()
        assert (at >= 0).all()
        for k in range(0, n, 29):
            size = (32 >> int(t[k])) ** 3
            np.testing.assert_array_equal(c.read(at[k], size), orc.decode_brick(blob, int(i[k]), int(t[k])).ravel())

    fill()
    for _ in range(2):
        with pytest.raises(csv.CsvError):
            failing.frame(ids, lods, slots=slots, stats=False)
    failing.close()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        cache.frame(ids, lods, slots=slots, stream=s, stats=False)  # the stream's decode buffers
    check(cache)
    fresh = torch.cuda.Stream()  # a stream without buffers, in a capture: refused after the frame's keys have their blocks
    with pytest.raises(csv.CsvError):
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=fresh):
            cache.frame(ids, lods, slots=slots, stream=fresh, stats=False)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        cache.frame(ids, lods, slots=slots, stream=s, stats=False)
    fill()
    with torch.cuda.stream(s):
        cache.frame(ids, lods, slots=slots, stream=s, stats=False)
    check(cache)
    for _ in range(3):
        fill()
        g.replay()
        check(cache)
    cache.close()
