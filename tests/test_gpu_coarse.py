"""GPU: requests of coarse levels of detail and small batches, where a decode
makes fewer launches or its later kernels find nothing to do."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_decode, torch_cuda

pytestmark = pytest.mark.gpu


def volume64(seed):
    """128^3: cells, a patch of many labels, a uniform 64^3 brick."""
    vol = synth.cells(n=128, grid=9, seed=seed)
    vol[:20, :20, :20] = np.random.default_rng(seed).integers(1, 1 << 30, (20, 20, 20)).astype(np.uint32)
    vol[:64, 64:, :64] = 5
    return vol


def decode_lods(csv, pool, ids, lods, status=False):
    torch = torch_cuda()
    off, tot = csv.output_offsets(lods, 6)
    out = torch.full((tot,), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(ids.size, dtype=torch.int32, device="cuda") if status else None
    pool.decode(torch.from_numpy(ids.view(np.int32)).cuda(), out, lods=torch.from_numpy(lods).cuda(),
                out_offsets=torch.from_numpy(off.view(np.int64)).cuda(), **({"status": st} if status else {}))
    torch.cuda.synchronize()
    return out.cpu().numpy().view(np.uint32), off, st


@pytest.mark.parametrize("n", [1, 512, 513, 1100])
@pytest.mark.parametrize("lane_max,tables", [(64, 1), (2, 1), (64, 3)])
def test_edge64_symbols_decoded_by_either_kernel(orc, n, lane_max, tables):
    # up to two requests per CU the upper kernel decodes the symbols, beyond
    # that a launch of its own; three volumes' tables do not fit LDS
    import paper_2308_16619_amd as csv
    blob = csv.encode_volume(volume64(31), brick_log2=6, lane_max=lane_max, scale_bits=11)
    pool = csv.Pool()
    for _ in range(tables):
        pool.add_volume(blob)
    rng = np.random.default_rng(n)
    ids = rng.integers(0, 8 * tables, n).astype(np.uint32)
    lods = np.where(np.arange(n) % 100 == 0, 0, rng.integers(1, 7, n)).astype(np.uint8)
    print("[gpu-test] edge 64, %d requests, %d states, %d volumes" % (n, lane_max, tables), flush=True)
    got, off, _ = decode_lods(csv, pool, ids, lods)
    assert pool.last_error() == (0, 0)
    want = {(i, t): orc.decode_brick(blob, i, t).ravel() for i in range(8) for t in range(7)}
    for i, t, o in zip(ids, lods, off):
        w = want[int(i) % 8, int(t)]
        np.testing.assert_array_equal(got[int(o):int(o) + w.size], w)


@pytest.mark.parametrize("n", [3, 700])
@pytest.mark.parametrize("labels", [100, 1 << 31])
@pytest.mark.parametrize("lod", [2, 3, 4, 5])
def test_edge64_one_coarse_level(orc, n, lod, labels):
    # by workgroups, and, many of them, by the front kernel (u8 or u16 indices)
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blobs = [csv.encode_volume(volume64(32 + c) % labels, brick_log2=6, coding=c) for c in (0, 1)]
    pool = csv.Pool()
    for b in blobs:
        pool.add_volume(b)
    ids = torch.arange(n, dtype=torch.int32, device="cuda") % 16
    out = torch.full((n, (64 >> lod) ** 3), -1, dtype=torch.int32, device="cuda")
    print("[gpu-test] edge 64, %d requests of level %d" % (n, lod), flush=True)
    pool.decode(ids, out, lod=lod)
    torch.cuda.synchronize()
    assert pool.last_error() == (0, 0)
    want = np.concatenate([orc.decode_bricks(b, np.arange(8), [lod] * 8).reshape(8, -1) for b in blobs])
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want[np.arange(n) % 16])


@pytest.mark.parametrize("n", [5, 600])
def test_edge64_malformed_states(orc, n):
    # a changed state of brick 1: found by whichever kernel decodes the symbols
    import paper_2308_16619_amd as csv
    blob = csv.encode_volume(volume64(33), brick_log2=6)
    rs = (128 + 8 * 9 + 15) & ~15
    at = rs + int(np.frombuffer(blob, np.uint64, 9, 128)[1])
    P = int(np.frombuffer(blob, np.uint32, 1, at)[0])
    bad = bytearray(blob)
    bad[at + 4 * (9 + P) + 1] ^= 0x5A
    pool = csv.Pool()
    pool.add_volume(bytes(bad))
    ids = (np.arange(n) % 5).astype(np.uint32)
    lods = np.where(np.arange(n) < 5, 0, 3).astype(np.uint8)
    print("[gpu-test] edge 64, malformed state among %d requests" % n, flush=True)
    got, off, st = decode_lods(csv, pool, ids, lods, status=True)
    st = st.cpu().numpy()
    assert st[1] == csv.CSV_ECORRUPT and pool.last_error()[0] == csv.CSV_ECORRUPT
    np.testing.assert_array_equal(got[int(off[1]):int(off[2])], 0)
    for k in (0, 2, 3, 4):
        assert st[k] == 0
        np.testing.assert_array_equal(got[int(off[k]):int(off[k]) + 64 ** 3], orc.decode_brick(blob, int(ids[k]), 0).ravel())


@pytest.mark.parametrize("n,plain", [(600, False), (600, True), (1500, False)])
def test_edge64_requests_out_of_range_among_many(orc, n, plain):
    # each is found once, by the kernel that serves its level
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = csv.encode_volume(volume64(36), brick_log2=6)
    pool = csv.Pool()
    pool.add_volume(blob)
    rng = np.random.default_rng(36)
    ids = rng.integers(0, 8, n).astype(np.uint32)
    lods = rng.integers(1, 7, n).astype(np.uint8)
    ids[[200, 300]] = [8, 1 << 31]
    lods[[200, 300]] = [1, 4]
    off, tot = csv.output_offsets(lods, 6)
    lods[[100, 599]] = [7, 255]
    out = torch.full((tot,), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(n, dtype=torch.int32, device="cuda")
    print("[gpu-test] edge 64, requests out of range, plain %s" % plain, flush=True)
    d = [torch.from_numpy(ids.view(np.int32)).cuda(), out]
    kw = {"lods": torch.from_numpy(lods).cuda(), "out_offsets": torch.from_numpy(off.view(np.int64)).cuda()}
    pool.decode(*d, **kw, **({"plain": True} if plain else {"status": st}))
    torch.cuda.synchronize()
    code, who = pool.last_error()
    assert code == csv.CSV_ERANGE and who in (100, 200, 300, 599)
    bad = np.isin(np.arange(n), (100, 200, 300, 599))
    if not plain:
        np.testing.assert_array_equal(st.cpu().numpy(), np.where(bad, csv.CSV_ERANGE, 0))
    got = out.cpu().numpy().view(np.uint32)
    for i in np.nonzero(~bad)[0]:
        w = orc.decode_brick(blob, int(ids[i]), int(lods[i])).ravel()
        np.testing.assert_array_equal(got[int(off[i]):int(off[i]) + w.size], w)


@pytest.mark.parametrize("n", [1025, 9300])
def test_edge64_levels_0_and_1_listed_from_many_requests(orc, n):
    # more requests than slots: none, some and only such levels (in chunks up
    # to the ninth, whose leaf workgroups take 8 runs)
    import paper_2308_16619_amd as csv
    blob = csv.encode_volume(volume64(37), brick_log2=6)
    pool = csv.Pool()
    pool.add_volume(blob)
    rng = np.random.default_rng(n)
    want = {(i, t): orc.decode_brick(blob, i, t).ravel() for i in range(8) for t in range(7)}
    for levels, p in (((3, 4, 5, 6), None), ((0, 1, 2, 5), (0.01, 0.3, 0.3, 0.39)), ((1,), None), ((0, 1), (0.005, 0.995))):
        ids = rng.integers(0, 8, n).astype(np.uint32)
        lods = rng.choice(levels, n, p=p).astype(np.uint8)
        lods[-1] = levels[0]
        print("[gpu-test] edge 64, %d requests of levels %s" % (n, levels), flush=True)
        got, off, _ = decode_lods(csv, pool, ids, lods)
        assert pool.last_error() == (0, 0)
        for i, t, o in zip(ids, lods, off):
            w = want[int(i), int(t)]
            assert np.array_equal(got[int(o):int(o) + w.size], w), (i, t, o)


def test_edge64_captured_with_more_requests_than_the_list_holds(orc):
    # the list cannot grow in a capture: chunks of all levels then
    torch = torch_cuda()
    import paper_2308_16619_amd as csv
    blob = csv.encode_volume(volume64(38), brick_log2=6)
    pool = csv.Pool()
    pool.add_volume(blob)
    n = 2100
    want = {(i, t): orc.decode_brick(blob, i, t).ravel() for i in range(8) for t in range(7)}
    rng = np.random.default_rng(38)
    lods = np.where(np.arange(n) % 300 == 0, 0, rng.integers(2, 7, n)).astype(np.uint8)
    off, tot = csv.output_offsets(lods, 6)
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    d_lods, d_off = torch.from_numpy(lods).cuda(), torch.from_numpy(off.view(np.int64)).cuda()
    out = torch.empty(tot, dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        pool.decode(ids[:1100], out, lods=d_lods[:1100], out_offsets=d_off[:1100], stream=s)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    print("[gpu-test] captured", flush=True)
    with torch.cuda.graph(g, stream=s):
        pool.decode(ids, out, lods=d_lods, out_offsets=d_off, stream=s)
    for _ in range(3):
        now = rng.integers(0, 8, n).astype(np.int32)
        ids.copy_(torch.from_numpy(now))
        out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert pool.last_error() == (0, 0)
        got = out.cpu().numpy().view(np.uint32)
        for i, t, o in zip(now, lods, off):
            w = want[int(i), int(t)]
            assert np.array_equal(got[int(o):int(o) + w.size], w), (i, t, o)


@pytest.mark.parametrize("coding", [0, 1])
@pytest.mark.parametrize("shape", [(2, 3, 0), (8, 3, 0), (8, 3, 1)])
def test_no_request_for_the_leaf_kernels_and_then_some(orc, coding, shape):
    # coarse levels by request leave the counters as full-LOD requests need them
    import paper_2308_16619_amd as csv
    vol = synth.cells(n=96, grid=9, seed=34)
    vol[:32, :32, :32] = np.random.default_rng(34).integers(1, 3000, (32, 32, 32)).astype(np.uint32)
    blob = csv.encode_volume(vol, coding=coding)
    pool = csv.Pool()
    pool.add_volume(blob)
    if coding == 0:
        pool.set_shape(shape)
    rng = np.random.default_rng(35)
    for k, levels in enumerate([(1, 2, 3, 4, 5), (0,), (5,), (4, 5), (0, 1, 2), (3,), (0,)]):
        n = 200 + k
        ids = rng.integers(0, 27, n).astype(np.uint32)
        lods = rng.choice(levels, n).astype(np.uint8)
        print("[gpu-test] coding %d, shape %s, levels %s" % (coding, shape, levels), flush=True)
        got, _ = gpu_decode(pool, ids, lods)
        np.testing.assert_array_equal(got, orc.decode_bricks(blob, ids, lods))
