"""Bricks of edge 2..16 and raw 32^3 bricks through the front kernel, where
its paths part: the number of rANS states per brick, batches larger than the
waves or slots there are, stream captures and tight memory budgets."""
import numpy as np
import pytest

import synth
from gpu_util import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def csvlib():
    torch_cuda()
    import paper_2308_16619_amd as csv
    csv.lib()
    return csv


def log(msg):
    print("[gpu-test] " + msg, flush=True)


def volume(n, seed):
    vol = synth.cells(n=n, grid=max(2, n // 7), seed=seed)
    vol[:16, :16, :16] = np.random.default_rng(seed).integers(1, 2000, (16, 16, 16)).astype(np.uint32)  # u16 indices
    vol[:16, 16:32, :16] = 3
    return vol


def full(csv, pool, n_ids, edge, lod):
    torch = torch_cuda()
    ids = torch.arange(n_ids, dtype=torch.int32, device="cuda")
    out = torch.full((n_ids * (edge >> lod) ** 3,), -1, dtype=torch.int32, device="cuda")
    pool.decode(ids, out, lod=lod)
    torch.cuda.synchronize()
    assert pool.last_error() == (0, 0)
    return out.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("lane_k,lane_max", [(64, 64), (8, 64), (16, 32), (64, 16), (8, 8), (8, 4), (1, 1), (1, 64)])
@pytest.mark.parametrize("N", [2, 3, 4])
def test_states_per_brick(csvlib, orc, N, lane_k, lane_max):
    # 1 .. 64 states: blocks of 8 steps with 64, 32, 16 or 8 states, their
    # remainders, and single steps with fewer
    blob = csvlib.encode_volume(volume(48, 5), brick_log2=N, lane_k=lane_k, lane_max=lane_max)
    B = csvlib.blob_info(blob)["n_bricks"]
    pool = csvlib.Pool()
    pool.add_volume(blob)
    for lod in (0, 1):
        log("edge %d, lane_k %d, lane_max %d, lod %d" % (1 << N, lane_k, lane_max, lod))
        np.testing.assert_array_equal(full(csvlib, pool, B, 1 << N, lod), orc.decode_bricks(blob, np.arange(B), [lod] * B))


@pytest.mark.parametrize("N,coding,n", [(4, 0, 20001), (2, 1, 70001), (5, 1, 8193), (5, 1, 17000)])
def test_batches_larger_than_the_scratch(csvlib, orc, N, coding, n):
    torch = torch_cuda()
    blob = csvlib.encode_volume(volume(64, 6), brick_log2=N, coding=coding)
    B = csvlib.blob_info(blob)["n_bricks"]
    pool = csvlib.Pool()
    pool.add_volume(blob)
    ids = np.random.default_rng(n).integers(0, B, n).astype(np.uint32)
    lod = 1
    want = orc.decode_bricks(blob, np.arange(B), [lod] * B).reshape(B, -1)
    out = torch.full((n, want.shape[1]), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(n, dtype=torch.int32, device="cuda")
    ids[n - 2] = B + 7  # a failure in the last chunk is named by its index in the call
    log("edge %d, %d requests" % (1 << N, n))
    pool.decode(torch.from_numpy(ids.view(np.int32)).cuda(), out, lod=lod, status=st)
    torch.cuda.synchronize()
    assert pool.last_error() == (csvlib.CSV_ERANGE, n - 2)
    ok = np.arange(n) != n - 2
    got = out.cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got[ok], want[ids[ok]])
    assert (got[n - 2] == 0).all()
    np.testing.assert_array_equal(st.cpu().numpy(), np.where(ok, 0, csvlib.CSV_ERANGE))


@pytest.mark.parametrize("N,warm,n", [(4, 2100, 9000), (5, 2100, 5000)])
def test_captured_after_a_smaller_batch(csvlib, orc, N, warm, n):
    torch = torch_cuda()
    blob = csvlib.encode_volume(volume(64, 7), brick_log2=N, coding=1)
    B = csvlib.blob_info(blob)["n_bricks"]
    pool = csvlib.Pool()
    pool.add_volume(blob)
    lod = 1
    want = orc.decode_bricks(blob, np.arange(B), [lod] * B).reshape(B, -1)
    rng = np.random.default_rng(3)
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    out = torch.empty((n, want.shape[1]), dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        pool.decode(ids[:warm], out, lod=lod)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    log("edge %d captured" % (1 << N))
    with torch.cuda.graph(g, stream=s):
        pool.decode(ids, out, lod=lod, stream=s)
    for k in range(3):
        now = rng.integers(0, B, n).astype(np.int32)
        ids.copy_(torch.from_numpy(now))
        out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert pool.last_error() == (0, 0)
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want[now])


@pytest.mark.parametrize("N,coding,n", [(1, 0, 1), (3, 0, 40), (4, 0, 1), (5, 1, 1), (5, 1, 8)])
def test_tight_memory_budget(csvlib, orc, N, coding, n):
    # the scratch a workgroup per request used to need (a byte per symbol,
    # five bytes per node and four per parent of the finest level) is enough
    blob = csvlib.encode_volume(volume(64, 8), brick_log2=N, coding=coding)
    info = csvlib.blob_info(blob)
    B = info["n_bricks"]
    free = csvlib.Pool()
    free.add_volume(blob)
    nodes = sum(8 ** k for k in range(N + 1))
    rs = (128 + 8 * (B + 1) + 15) & ~15
    idx = np.frombuffer(blob, np.uint64, B + 1, 128)
    c0 = max(int(np.frombuffer(blob, np.uint32, 4, rs + int(i))[3]) for i in idx[:-1])
    up = lambda v: (v + 255) & ~255  # noqa: E731
    group = up(c0 + 16) + up(4 * nodes) + up(nodes) + up(4 * 8 ** (N - 1))
    pool = csvlib.Pool(0, hbm_budget=free.info()["device_bytes"] + 64 + n * group)
    pool.add_volume(blob)
    log("edge %d, %d requests, %d bytes each" % (1 << N, n, group))
    np.testing.assert_array_equal(full(csvlib, pool, n, 1 << N, 0), orc.decode_bricks(blob, np.arange(n), [0] * n))


def volume64(seed):
    """128^3: cells; a patch of many labels (palette near 8,000), a
    checkerboard, a uniform brick and one of 17 random labels (many deltas)."""
    vol = synth.cells(n=128, grid=9, seed=seed)
    rng = np.random.default_rng(seed)
    vol[:20, :20, :20] = rng.integers(1, 1 << 30, (20, 20, 20)).astype(np.uint32)
    z, y, x = np.indices((64, 64, 64))
    vol[:64, :64, 64:] = np.where((x + y + z) % 2 == 0, 7, 9)
    vol[:64, 64:, :64] = 5
    vol[64:, :64, :64] = np.repeat(rng.integers(1, 18, (32, 64, 64)).astype(np.uint32), 2, 0)
    return vol


@pytest.mark.parametrize("lane_max", [64, 16, 2])
def test_edge64_every_lod(csvlib, orc, lane_max):
    torch = torch_cuda()
    v1, v2 = volume64(21), synth.cells(n=100, grid=6, seed=22)
    b1 = csvlib.encode_volume(v1, brick_log2=6, lane_max=lane_max)
    b2 = csvlib.encode_volume(v2, brick_log2=6, coding=1)  # ragged: 100 = 64 + 36
    pool = csvlib.Pool()
    pool.add_volume(b1)
    assert pool.add_volume(b2) == 8
    for lod in range(6):
        log("edge 64, lane_max %d, lod %d" % (lane_max, lod))
        want = np.concatenate([orc.decode_bricks(b, np.arange(8), [lod] * 8) for b in (b1, b2)])
        np.testing.assert_array_equal(full(csvlib, pool, 16, 64, lod), want)
    # per-request levels at offsets that are not 16-byte aligned
    ids = np.arange(16).repeat(2).astype(np.uint32)
    lods = (np.arange(32) % 7).astype(np.uint8)
    off, tot = csvlib.output_offsets(lods, 6)
    off = off + np.arange(32, dtype=np.uint64) * 3
    out = torch.full((tot + 96,), -1, dtype=torch.int32, device="cuda")
    log("edge 64, mixed lods")
    pool.decode(torch.from_numpy(ids.view(np.int32)).cuda(), out, lods=torch.from_numpy(lods).cuda(),
                out_offsets=torch.from_numpy(off.view(np.int64)).cuda())
    torch.cuda.synchronize()
    assert pool.last_error() == (0, 0)
    got = out.cpu().numpy().view(np.uint32)
    for i, t, o in zip(ids, lods, off):
        want = orc.decode_brick(b1 if i < 8 else b2, int(i) % 8, int(t)).ravel()
        np.testing.assert_array_equal(got[int(o):int(o) + want.size], want)


@pytest.mark.parametrize("n", [1030, 2500])
def test_edge64_more_requests_than_slots(csvlib, orc, n):
    torch = torch_cuda()
    blob = csvlib.encode_volume(volume64(23), brick_log2=6)
    pool = csvlib.Pool()
    pool.add_volume(blob)
    ids = np.random.default_rng(n).integers(0, 8, n).astype(np.uint32)
    lods = np.where(np.arange(n) % 50 == 0, 0, 3).astype(np.uint8)
    off, tot = csvlib.output_offsets(lods, 6)
    out = torch.full((tot,), -1, dtype=torch.int32, device="cuda")
    log("edge 64, %d requests" % n)
    pool.decode(torch.from_numpy(ids.view(np.int32)).cuda(), out, lods=torch.from_numpy(lods).cuda(),
                out_offsets=torch.from_numpy(off.view(np.int64)).cuda())
    torch.cuda.synchronize()
    assert pool.last_error() == (0, 0)
    got = out.cpu().numpy().view(np.uint32)
    want = {(i, t): orc.decode_brick(blob, i, t).ravel() for i in range(8) for t in (0, 3)}
    for i, t, o in zip(ids, lods, off):
        w = want[int(i), int(t)]
        np.testing.assert_array_equal(got[int(o):int(o) + w.size], w)


@pytest.mark.parametrize("nibble", [0x7, 0x8, 0x1, 0x2, 0x3])
def test_edge64_malformed_finest_level(csvlib, orc, nibble):
    # the first operation of level 0 of the checkerboard (its node lies in the
    # brick's corner): an unused code, a stop bit, references out of the brick
    torch = torch_cuda()
    blob = csvlib.encode_volume(volume64(24), brick_log2=6, coding=1)
    idx = np.frombuffer(blob, np.uint64, 9, 128)
    rs = (128 + 8 * 9 + 15) & ~15
    at = rs + int(idx[1])
    w = np.frombuffer(blob, np.uint32, 9, at)
    c0, c1 = int(w[3]), int(w[4])
    first = c0 - 8 * 32768  # every level-1 node is expanded
    assert first >= c1
    bad = bytearray(blob)
    byte = at + 4 * (9 + int(w[0])) + first // 2
    sh = 4 * (first & 1)
    bad[byte] = (bad[byte] & ~(0xF << sh)) | (nibble << sh)
    pool = csvlib.Pool()
    pool.add_volume(bytes(bad))
    out = torch.full((3, 64 ** 3), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(3, dtype=torch.int32, device="cuda")
    log("edge 64, malformed operation %d" % nibble)
    pool.decode(torch.tensor([0, 1, 4], dtype=torch.int32, device="cuda"), out, status=st)
    torch.cuda.synchronize()
    assert pool.last_error() == (csvlib.CSV_ECORRUPT, 1)
    assert st.tolist() == [0, csvlib.CSV_ECORRUPT, 0]
    got = out.cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got[1], 0)
    for k, i in ((0, 0), (2, 4)):
        np.testing.assert_array_equal(got[k], orc.decode_brick(blob, i, 0).ravel())


def test_edge64_large_palette_takes_the_generic_decoder(csvlib, orc):
    vol = volume64(25)
    vol[64:, 64:, 64:] = np.random.default_rng(1).integers(1, 1 << 30, (64, 64, 64)).astype(np.uint32)
    blob = csvlib.encode_volume(vol, brick_log2=6, coding=1)
    pool = csvlib.Pool()
    pool.add_volume(blob)
    log("edge 64, a palette of %d entries" % 64 ** 3)
    np.testing.assert_array_equal(full(csvlib, pool, 8, 64, 0), orc.decode_bricks(blob, np.arange(8), [0] * 8))
