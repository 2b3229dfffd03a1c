"""GPU: memory budgets of pools whose bricks take other kernels than those of
32^3 rANS bricks."""
import numpy as np
import pytest

import synth
from gpu_util import torch_cuda

pytestmark = pytest.mark.gpu
ARENA = 82560  # bytes of a workgroup of the leaf kernel for large palettes


def pool_of(csv, blob, budget=0):
    pool = csv.Pool(hbm_budget=budget)
    pool.add_volume(blob)
    return pool


def decode(pool, n, n_bricks, edge=32):
    torch = torch_cuda()
    ids = torch.arange(n, dtype=torch.int32, device="cuda") % n_bricks
    out = torch.full((n * edge ** 3,), -1, dtype=torch.int32, device="cuda")
    print("[gpu-test] %d bricks of edge %d" % (n, edge), flush=True)
    pool.decode(ids, out, lod=0)
    torch.cuda.synchronize()
    assert pool.last_error() == (0, 0)
    return out.cpu().numpy().view(np.uint32)


def raw_blob(csv, seed):
    """Raw 32^3 bricks, one with a large palette."""
    vol = synth.cells(n=64, grid=8, seed=seed)
    vol[:32, :32, :32] = np.random.default_rng(seed).integers(1, 3000, (32, 32, 32)).astype(np.uint32)
    return csv.encode_volume(vol, coding=1)


def test_batches_that_grow_within_a_budget(orc):
    # raw 32^3 bricks: the budget holds the slots and 12 arenas
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = raw_blob(csv, 4)
    pool = pool_of(csv, blob)
    before = pool.info()["device_bytes"]
    decode(pool, 1, 8)
    every = pool.info()["device_bytes"] - before  # 1,024 slots, 4 arenas per CU
    arenas = 4 * torch.cuda.get_device_properties(0).multi_processor_count * ARENA
    assert every > arenas
    pool = pool_of(csv, blob, before + every - arenas + 12 * ARENA + ARENA // 2)
    want = orc.decode_bricks(blob, np.arange(12) % 8, np.zeros(12, np.uint8))
    for n in (8, 9, 12):
        np.testing.assert_array_equal(decode(pool, n, 8), want[:n * 32768])


def test_small_batches_leave_the_budget_to_others(orc):
    # a budget of what an unlimited pool takes for a stream: small batches on
    # several streams and a second volume fit
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = raw_blob(csv, 5)
    pool = pool_of(csv, blob)
    decode(pool, 1, 8)
    pool = pool_of(csv, blob, pool.info()["device_bytes"] + ARENA // 4)
    want = orc.decode_bricks(blob, np.arange(4), np.zeros(4, np.uint8))
    for s in [torch.cuda.Stream() for _ in range(3)]:
        with torch.cuda.stream(s):
            np.testing.assert_array_equal(decode(pool, 4, 8), want)
    assert pool.add_volume(blob) == 8


@pytest.mark.parametrize("budget", [0, 1 << 30])
def test_captured_after_a_smaller_batch(orc, budget):
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = raw_blob(csv, 6)
    pool = pool_of(csv, blob, budget)
    want = orc.decode_bricks(blob, np.arange(8), np.zeros(8, np.uint8)).reshape(8, -1)
    n = 50
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    out = torch.empty((n, 32768), dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        pool.decode(ids[:3], out)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    print("[gpu-test] captured", flush=True)
    with torch.cuda.graph(g, stream=s):
        pool.decode(ids, out, stream=s)
    rng = np.random.default_rng(6)
    for _ in range(3):
        now = rng.integers(0, 8, n).astype(np.int32)
        ids.copy_(torch.from_numpy(now))
        out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert pool.last_error() == (0, 0)
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want[now])


def volume64(seed):
    vol = synth.cells(n=128, grid=9, seed=seed)
    vol[:20, :20, :20] = np.random.default_rng(seed).integers(1, 1 << 30, (20, 20, 20)).astype(np.uint32)
    vol[:64, 64:, :64] = 5
    return vol


def workgroup_bytes(blob, n_bricks):
    """What a 64^3 request needs where a workgroup decodes it in memory: a
    byte per symbol, five bytes per node, four per parent of the finest level."""
    rs = (128 + 8 * (n_bricks + 1) + 15) & ~15
    c0 = max(int(np.frombuffer(blob, np.uint32, 4, rs + int(i))[3]) for i in np.frombuffer(blob, np.uint64, n_bricks, 128))
    nodes = sum(8 ** k for k in range(7))
    up = lambda v: (v + 255) & ~255  # noqa: E731
    return up(c0 + 16) + up(4 * nodes) + up(nodes) + up(4 * 8 ** 5)


@pytest.mark.parametrize("coding", [0, 1])
@pytest.mark.parametrize("n", [1, 5])
def test_edge64_within_a_budget(orc, coding, n):
    import paper_2308_16619_amd as csv
    blob = csv.encode_volume(volume64(7), brick_log2=6, coding=coding)
    base = pool_of(csv, blob).info()["device_bytes"]
    want = orc.decode_bricks(blob, np.arange(n), np.zeros(n, np.uint8))
    pool = pool_of(csv, blob, base + 64 + n * workgroup_bytes(blob, 8))
    np.testing.assert_array_equal(decode(pool, n, 8, 64), want)
    # a budget below one request's slot
    pool = pool_of(csv, blob, base + (100 << 10))
    with pytest.raises(csv.CsvError) as e:
        decode(pool, n, 8, 64)
    assert e.value.code == csv.CSV_ENOMEM


@pytest.mark.parametrize("coding", [0, 1])
def test_edge64_captured(orc, coding):
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = csv.encode_volume(volume64(8), brick_log2=6, coding=coding)
    pool = pool_of(csv, blob)
    want = orc.decode_bricks(blob, np.arange(8), np.zeros(8, np.uint8)).reshape(8, -1)
    n = 12
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    out = torch.empty((n, 64 ** 3), dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        pool.decode(ids, out)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    print("[gpu-test] captured", flush=True)
    with torch.cuda.graph(g, stream=s):
        pool.decode(ids, out, stream=s)
    rng = np.random.default_rng(8)
    for _ in range(3):
        now = rng.integers(0, 8, n).astype(np.int32)
        ids.copy_(torch.from_numpy(now))
        out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert pool.last_error() == (0, 0)
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want[now])
    fresh = pool_of(csv, blob)
    with pytest.raises(csv.CsvError) as e:  # no slots on this stream, and they cannot be made in a capture
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=s):
            fresh.decode(ids, out, stream=s)
    assert e.value.code == csv.CSV_EBUSY
