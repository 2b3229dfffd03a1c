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


def test_batches_that_grow_within_a_budget(orc):
    # raw 32^3 bricks: the budget holds the slots and 12 arenas
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    vol = synth.cells(n=64, grid=8, seed=4)
    vol[:32, :32, :32] = np.random.default_rng(4).integers(1, 3000, (32, 32, 32)).astype(np.uint32)
    blob = csv.encode_volume(vol, coding=1)
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
