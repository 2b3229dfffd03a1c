"""GPU: the frame cache's lists over several workgroups.  Keys take their
places with one counter step per wave and workgroup, so request counts on
both sides of a wave and of a workgroup, with duplicates, unknown ids and
levels that are not stored, must give the counts of a host model over sets,
one block per distinct key, and every block the decode of its brick."""
import numpy as np
import pytest

import synth
from gpu_util import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 65, 255, 257, 1025, 9001])
def test_counts_and_blocks(orc, n):
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = orc.encode_volume(synth.cells(n=256, grid=19, seed=2), scale_bits=10, lane_k=64)
    pool = csv.Pool()
    for _ in range(5):
        pool.add_volume(blob)
    nb = 5 * 512
    cache = csv.FrameCache(pool, 512 << 20, n)
    rng = np.random.default_rng(n)
    last = set()
    for f in range(4):
        ids = rng.integers(0, nb + 3, n).astype(np.uint32)
        lods = rng.choice(7, n, p=[.3, .2, .2, .1, .1, .05, .05]).astype(np.uint8)
        if f == 3:
            lods[:] = 5  # nothing stored: every key of the last frame leaves
        ok = (ids < nb) & (lods < 5)
        keys = set(zip(ids[ok].tolist(), lods[ok].tolist()))
        slots, st = cache.frame(torch.from_numpy(ids.view(np.int32)).cuda(), torch.from_numpy(lods).cuda())
        slots = slots.cpu().numpy()
        assert (st["frame"], st["distinct"], st["decoded"]) == (f + 1, len(keys), len(keys - last))
        assert (st["hits"], st["evicted"], st["rebuilt"]) == (len(keys & last), len(last - keys), 0)
        assert ((slots >= 0) == ok).all()
        at = {}
        for i, t, s in zip(ids[ok].tolist(), lods[ok].tolist(), slots[ok].tolist()):
            assert at.setdefault((i, t), s) == s
        iv = sorted((s, s + (32 >> t) ** 3) for (_, t), s in at.items())
        assert all(a[1] <= b[0] for a, b in zip(iv, iv[1:]))
        some = sorted(at)[:: max(1, len(at) // 40)]
        for i, t in some:
            size = (32 >> t) ** 3
            out = torch.empty(size, dtype=torch.int32, device="cuda")
            pool.decode(torch.tensor([i], dtype=torch.int32, device="cuda"), out, lod=t)
            np.testing.assert_array_equal(cache.read(at[i, t], size), out.cpu().numpy().view(np.uint32))
        last = keys
    cache.close()
