"""The GPU compressor where its paths part: ragged volumes and row strides,
numbers of states per brick and symbols per block, records that do not fit
where they are usually written, bricks with few and many palette operations."""
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


def check(csvlib, orc, vol, **kw):
    opts = {"scale_bits": 10, "lane_k": 64, "lane_max": 64, **kw}
    print("[gpu-test] encode %s %s" % (vol.shape, opts), flush=True)
    got = csvlib.encode_volume_gpu(np.ascontiguousarray(vol), **opts)
    assert got == orc.encode_volume(vol, **opts)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 65), (65, 1, 1), (31, 33, 32), (32, 32, 33), (64, 40, 97),
                                   (33, 96, 129), (96, 31, 34)])
def test_ragged_volumes(csvlib, orc, shape):
    n = max(shape)
    vol = synth.cells(n=n, grid=max(2, n // 6), seed=n)[:shape[0], :shape[1], :shape[2]]
    check(csvlib, orc, vol, sample_stride=2)


@pytest.mark.parametrize("lane_k,lane_max,bits", [(64, 64, 8), (64, 32, 12), (1, 64, 10), (7, 16, 9), (64, 8, 11),
                                                  (3, 4, 10), (1, 2, 10), (1, 1, 12)])
def test_states_and_blocks(csvlib, orc, lane_k, lane_max, bits):
    # 40 labels a brick down to 1: from 0 symbols to thousands, so that last
    # blocks of 16 steps are whole, partial and the only one
    vol = synth.cells(n=96, grid=9, seed=bits + lane_k)
    vol[:32, :32, :32] = 4
    vol[32:64, :32, :32] = np.where(np.arange(32)[:, None, None] < 16, 4, 5)
    vol[:32, 32:64, :32][0, 0, 0] = 77
    check(csvlib, orc, vol, lane_k=lane_k, lane_max=lane_max, scale_bits=bits, sample_stride=1)


def test_records_larger_than_their_nibbles(csvlib, orc):
    # the only sampled brick is smooth, so that the tables give the others'
    # symbols up to 12 bits
    vol = np.random.default_rng(5).integers(1, 40, (96, 96, 128)).astype(np.uint32)
    vol[:32, :32, :32] = 1
    vol[:16, :32, :32] = 2
    check(csvlib, orc, vol, scale_bits=12)


@pytest.mark.parametrize("labels", [2, 17, 18, 60, 5000])
def test_palette_window(csvlib, orc, labels):
    # the last 17 entries: every label in it, one too many, most appended
    vol = np.random.default_rng(labels).integers(0, labels, (64, 64, 64)).astype(np.uint32)
    vol[32:] = np.repeat(np.repeat(np.repeat(vol[:16, :32, :32], 2, 0), 2, 1), 2, 2)
    check(csvlib, orc, vol, sample_stride=1)
    check(csvlib, orc, vol, tables=1)


def test_container_memory(csvlib, orc):
    # the library's own memory, the caller's, and a caller that has none;
    # sizes on both sides of the piecewise copy
    import ctypes
    torch = torch_cuda()
    L = csvlib.lib()
    for n, labels in ((64, 50), (160, 1 << 20)):
        vol = np.random.default_rng(n).integers(1, labels, (n, n, n)).astype(np.uint32)
        want = csvlib.encode_volume(vol)
        d = torch.from_numpy(vol.view(np.int32)).cuda()
        o = csvlib.EncodeOpts(5, 10, 64, 64, 0, 0, 2, 0)
        p, size = ctypes.c_void_p(), ctypes.c_size_t()
        print("[gpu-test] container of %d bytes" % len(want), flush=True)
        args = [ctypes.c_void_p(d.data_ptr()), n, n, n, ctypes.byref(o), 0, None]
        assert L.csv_encode_volume_gpu(*args, ctypes.byref(p), ctypes.byref(size)) == 0
        assert ctypes.string_at(p, size.value) == want
        L.csv_free(p)
        assert csvlib.encode_volume_gpu(d) == want
        none = csvlib._ALLOC(lambda size, ctx: None)
        assert L.csv_encode_volume_gpu_alloc(*args, none, None, ctypes.byref(size)) == csvlib.CSV_ENOMEM
    assert (len(want) >= 8 << 20) and csvlib.encode_volume_gpu(d) == want


@pytest.mark.parametrize("shape", [(5, 17, 33), (64, 64, 64), (64, 70, 96), (96, 128, 130), (128, 160, 161)])
def test_container_exits(csvlib, orc, shape):
    # containers of some KB to some 10 MB: with the state, in one copy when
    # the pinned buffer grows, in pieces; the second call finds it grown
    vol = np.random.default_rng(shape[2]).integers(1, 1 << 20, shape).astype(np.uint32)
    for _ in range(2):
        check(csvlib, orc, vol)
    check(csvlib, orc, vol[:3])


@pytest.mark.parametrize("by,bx", [(1, 1023), (32, 32), (25, 41), (41, 100)])
def test_sizes_scanned_per_workgroup_or_once(csvlib, orc, by, bx):
    # one brick short of, at, one past and well past the last count of bricks
    # whose sizes every workgroup scans itself
    vol = np.zeros((1, 32 * by, 32 * bx), np.uint32)
    rng = np.random.default_rng(bx)
    for y, x in zip(rng.integers(0, 32 * by, 4000), rng.integers(0, 32 * bx, 4000)):
        vol[0, y:y + 9, x:x + 5] = y + x
    check(csvlib, orc, vol)


@pytest.mark.parametrize("left,sample_stride", [(110, 0), (48, 3)])
def test_little_device_memory(csvlib, orc, left, sample_stride):
    # in batches of bricks, as the device has no room for all of them at once
    torch = torch_cuda()
    vol = synth.cells(n=192, grid=14, seed=31)
    vol[:96] = np.random.default_rng(31).integers(1, 1 << 30, (96, 192, 192)).astype(np.uint32)
    opts = {"scale_bits": 10, "lane_k": 64, "lane_max": 64, "sample_stride": sample_stride}
    want = orc.encode_volume(vol, **opts)
    dev = torch.from_numpy(vol.view(np.int32)).cuda()
    assert csvlib.encode_volume_gpu(dev, **opts) == want
    csvlib.encode_gpu_release(0)
    torch.cuda.empty_cache()
    fill = []
    while len(fill) < 8 and torch.cuda.mem_get_info()[0] >> 20 > left + 16:
        fill.append(torch.empty(torch.cuda.mem_get_info()[0] - (left << 20), dtype=torch.uint8, device="cuda"))
    now = torch.cuda.mem_get_info()[0] >> 20
    print("[gpu-test] %d MiB left" % now, flush=True)
    try:
        if now > left + 64:
            pytest.skip("the device's memory cannot be filled up")
        assert csvlib.encode_volume_gpu(dev, **opts) == want
        assert csvlib.encode_volume_gpu(dev[:33, :40, :50].contiguous(), **opts) == orc.encode_volume(
            np.ascontiguousarray(vol[:33, :40, :50]), **opts)
    finally:
        del fill
        torch.cuda.empty_cache()
        csvlib.encode_gpu_release(0)
    assert csvlib.encode_volume_gpu(dev, **opts) == want
