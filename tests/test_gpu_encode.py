"""GPU-side encoder (ecf8_encode_gpu, paper Section 3.1 on the device): the container it writes is
the CPU encoder's, byte for byte; the oracle's reader decodes it to the input and agrees on the
stream length; the GPU decoder round-trips it."""
import ctypes
import os
import subprocess
import sys
import time

import numpy as np
import pytest
import torch

from paper_2510_02676_amd import ecf8, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _rand_bytes(n, seed, conc=0.4):
    rng = np.random.default_rng(seed)
    p = rng.dirichlet(np.ones(16) * conc)
    e = rng.choice(16, size=n, p=p).astype(np.uint8)
    return ((rng.integers(0, 2, n, dtype=np.uint8) << 7) | (e << 3) | rng.integers(0, 8, n, dtype=np.uint8)).astype(np.uint8)


def _check_same(orc, x, rows, cols, oracle_read=True, **opts):
    d_x = torch.from_numpy(x).to(DEV)
    hdr, d_blob = ecf8.ecf8_encode_gpu(d_x, rows, cols, **opts)
    torch.cuda.synchronize()
    got = d_blob.cpu().numpy()
    want = ecf8.ecf8_encode(x, rows, cols, **opts)
    assert bytes(hdr) == bytes(want.header)
    w = want.numpy()
    assert got.size == w.size
    if not np.array_equal(got, w):
        bad = np.flatnonzero(got != w)
        raise AssertionError("GPU and CPU containers differ at %d bytes, first at offset %d (sections: cb %d lb %d st %d pl %d)"
                             % (bad.size, bad[0], hdr.off_chunk_bit, hdr.off_lane_bits, hdr.off_stream, hdr.off_plane))
    ecf8.blob_validate(got)
    if oracle_read:
        dec, bits = orc.container_decode(got)
        assert np.array_equal(dec, x.reshape(-1)) and bits == hdr.stream_bits
    out = ecf8.ecf8_decode(hdr, d_blob.clone())
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().reshape(-1), x.reshape(-1))


@pytest.mark.parametrize("lane_syms", [32, 64, 128])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 2047, 4097, 8193, 3 * 8192 + 77, 300_001, 1_000_003])
def test_same_container_as_the_cpu_encoder(orc, lane_syms, n):
    x = _rand_bytes(n, 13 * n + lane_syms)
    _check_same(orc, x, 1, n, lane_syms=lane_syms, max_code_len=15 if n % 2 else 0, table_mode=1 + (n % 3 == 0))


@pytest.mark.parametrize("opts", [dict(group_chunks=1), dict(group_chunks=4, lane_syms=32), dict(group_chunks=64),
                                  dict(max_code_len=4), dict(max_code_len=15, lane_syms=64, group_chunks=2)])
def test_layout_and_cap_options(orc, opts):
    x = _rand_bytes(2_300_017, 77)
    _check_same(orc, x, 1, x.size, **opts)


@pytest.mark.parametrize("lane_syms,rows,cols", [(32, 16, 128), (64, 64, 4096), (128, 48, 3584), (64, 160, 1024)])
def test_row_tiled_layout(orc, lane_syms, rows, cols):
    x = _rand_bytes(rows * cols, rows + cols)
    _check_same(orc, x, rows, cols, lane_syms=lane_syms, tile_rows=16)


@pytest.mark.parametrize("block", range(4))
def test_seeded_sweep_of_shapes_and_options(orc, block):
    """120 seeded combinations of size, lane_syms, group width, cap, table mode and exponent skew:
    the device writes the CPU encoder's container every time."""
    rng = np.random.default_rng(7000 + block)
    for i in range(30):
        lane_syms = int(rng.choice([32, 64, 128]))
        chunk = 64 * lane_syms
        n = max(1, int(rng.integers(1, 40)) * chunk + int(rng.integers(-chunk, chunk)) if i % 2 else int(rng.integers(1, 300_000)))
        x = _rand_bytes(n, int(rng.integers(1 << 30)), conc=float(rng.choice([0.05, 0.3, 2.0, 50.0])))
        _check_same(orc, x, 1, n, oracle_read=(i % 5 == 0), lane_syms=lane_syms,
                    group_chunks=int(rng.choice([1, 2, 8, 32, 64])), max_code_len=int(rng.choice([0, 15, 4, 10])),
                    table_mode=int(rng.choice([1, 2])))


@pytest.mark.parametrize("chunks,extra", [(1024, 0), (1024, 1), (2048, -1), (8192, 7), (65536, 0), (65536, 1), (65536 + 8192, 5)])
def test_many_chunks(chunks, extra):
    """Many tiles, each placed by what the ones before it have counted: powers of two, one chunk less and more."""
    n = chunks * 2048 + extra
    x = np.resize(_rand_bytes((1 << 20) + 12345, chunks + extra), n)
    opts = dict(lane_syms=32, max_code_len=15 if extra else 0)
    want = ecf8.ecf8_encode(x, 1, n, **opts)
    hdr, d_blob = ecf8.ecf8_encode_gpu(torch.from_numpy(x).to(DEV), 1, n, **opts)
    torch.cuda.synchronize()
    assert bytes(hdr) == bytes(want.header)
    assert torch.equal(d_blob.cpu(), torch.from_numpy(want.numpy()))


@pytest.mark.parametrize("opts", [dict(lane_syms=128, table_mode=1), dict(lane_syms=64, table_mode=2, max_code_len=15), dict(lane_syms=32, table_mode=1, group_chunks=1),
                                  dict(lane_syms=64, tile_rows=16, table_mode=2)])
def test_every_byte_of_the_blob_is_written(opts):
    """Into a poisoned buffer: the padding between sections, the plane past a ragged end and the dwords of the stream
    that chunks share hold what the CPU encoder's container holds, and nothing behind the blob is touched."""
    rows = 16 if "tile_rows" in opts else 1
    for n in ([4096, 16 * 4096] if rows == 16 else [1, 33, 2047, 8192, 8192 * 33 + 5, 300_001]):
        x = _rand_bytes(n, n + 5)
        want = ecf8.ecf8_encode(x, rows, n // rows, **opts)
        buf = torch.full((want.size + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
        hdr, _ = ecf8.ecf8_encode_gpu(torch.from_numpy(x).to(DEV), rows, n // rows, d_blob=buf, **opts)
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert bytes(hdr) == bytes(want.header)
        assert np.array_equal(got[:want.size], want.numpy()), n
        assert (got[want.size:] == 0xA5).all(), n


# One compute unit's waves take 4, 8 or 16 chunks of a tile, one each and then more each: either side of those borders, tiles of one chunk
@pytest.mark.parametrize("chunks", [1, 4, 5, 1024, 1025, 2048, 2049, 4096, 4097, 4129, 12289])
@pytest.mark.parametrize("extra", [0, 3])
def test_borders_of_tiles(chunks, extra):
    n = chunks * 2048 + extra
    x = np.resize(_rand_bytes((1 << 20) + 4321, chunks + extra, conc=2.0), n)
    for opts in (dict(lane_syms=32), dict(lane_syms=32, max_code_len=15, group_chunks=1)):
        want = ecf8.ecf8_encode(x, 1, n, **opts)
        buf = torch.full((want.size + 256,), 0xA5, dtype=torch.uint8, device=DEV)
        hdr, _ = ecf8.ecf8_encode_gpu(torch.from_numpy(x).to(DEV), 1, n, d_blob=buf, **opts)
        torch.cuda.synchronize()
        assert bytes(hdr) == bytes(want.header)
        assert torch.equal(buf[:want.size].cpu(), torch.from_numpy(want.numpy())) and bool((buf[want.size:] == 0xA5).all())


@pytest.mark.parametrize("lane_syms,cap,chunks,islands", [(32, 0, 40960, [(0, 170), (20011, 20400), (40930, 40960)]), (64, 15, 16500, [(2, 30), (8000, 8400), (16490, 16500)]),
                                                          (128, 15, 6200, [(0, 1), (3104, 3105), (6199, 6200)]), (128, 15, 6200, [(17, 18), (3135, 3136), (6197, 6198)])])
def test_chunks_that_do_not_fit_behind_the_others(lane_syms, cap, chunks, islands):
    """A wave packs its chunks of a tile one behind the other into an image that holds the average chunk some times over.  Islands of long
    codewords do not fit: several chunks of one wave, or a single chunk of 8192 codewords of ten bits, first, last and inside their tile."""
    E = 64 * lane_syms
    n = chunks * E - 37
    rng = np.random.default_rng(chunks + lane_syms)
    e = np.minimum(rng.geometric(0.5 if lane_syms == 128 else 0.98, n) - 1, 13).astype(np.uint8)
    for a, b in islands:
        e[a * E:b * E] = 14 if lane_syms == 128 else rng.integers(0, 16, e[a * E:b * E].size)
    x = (e << 3) | (rng.integers(0, 256, n, dtype=np.uint8) & 0x87)
    opts = dict(lane_syms=lane_syms, max_code_len=cap, group_chunks=1)
    want = ecf8.ecf8_encode(x, 1, n, **opts)
    assert lane_syms != 128 or want.header.code_len[14] >= 10
    hdr, d_blob = ecf8.ecf8_encode_gpu(torch.from_numpy(x).to(DEV), 1, n, **opts)
    torch.cuda.synchronize()
    assert bytes(hdr) == bytes(want.header)
    assert torch.equal(d_blob.cpu(), torch.from_numpy(want.numpy()))


def _us(call, n=10):
    """Host time of a call among others, in us."""
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(n):
        call()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / n * 1e6


def best_times(calls, rounds=12):
    """The least of some times of each call, taken in turn."""
    for call in calls:
        _us(call, 3)
    return [min(ts) for ts in zip(*[[_us(call) for call in calls] for _ in range(rounds)])]


@pytest.mark.parametrize("rows,cols,zeros,opts", [(14336, 7168, 0.75, {}), (16384, 16384, 0.5, {}), (16384, 16384, 0.5, dict(max_code_len=15)),
                                                  (16384, 16384, 0.5, dict(lane_syms=64, tile_rows=16))])
def test_unlike_chunks_are_encoded_as_fast_as_like_ones(rows, cols, zeros, opts):
    """Rows of zeros above the other weights, so that chunks differ in length and some do not fit behind the others of their wave, against as many zeros spread
    evenly over the columns.  Looked up symbol by symbol, the chunks that did not fit made it 1.6 to 2.9 times as long; packed as the others are, 1.02 to 1.19.  The
    limit lies between."""
    w = synth.make_weight(rows, cols, 1.8, 0.02, 1, 0, "block128", DEV).view(rows, cols)
    apart, spread = w.clone(), w
    apart[:int(zeros * rows)] = 0
    spread.view(rows, cols // 16, 16)[:, :, :int(zeros * 16)] = 0
    buf = torch.empty(rows * cols, dtype=torch.uint8, device=DEV)
    t_apart, t_spread = best_times([lambda x=x: ecf8.ecf8_encode_gpu(x, d_blob=buf, **opts) for x in (apart, spread)])
    print("%.1f us, zeros spread evenly %.1f" % (t_apart, t_spread))
    assert t_apart < 1.4 * t_spread


def _rows_equal(t, row):
    """Is every row of the flat tensor t (a whole number of rows) this row?  In pieces: t may be tens of GB."""
    n = row.numel()
    step = max(1, (1 << 28) // n) * n
    return all(bool((t[i:i + step].view(-1, n) == row).all()) for i in range(0, t.numel(), step))


@pytest.mark.parametrize("groups", [(1 << 17) + 3, (1 << 21) + 3])
def test_more_chunks_than_one_launch_takes(groups):
    """8.6 GB and 137 GB of weights, 32 symbols per lane: 2^22 and 2^26 chunks and some, the larger one with more than the 2^32
    work-items of a launch if each chunk had a wave of its own.  Every group of 32 chunks holds the same weights, whose code bits are a whole number of 16-byte units, so each section of the container is the CPU
    encoder's for one group over and over."""
    period = 32 * 2048
    n = groups * period
    rng = np.random.default_rng(1)
    e = np.full(period, 7, np.uint8)
    e[rng.choice(period, 4096, replace=False)] = np.repeat([8, 3], 2048)
    x = (e << 3) | (rng.integers(0, 256, period, dtype=np.uint8) & 0x87)
    opts = dict(lane_syms=32, table_mode=2)
    one = ecf8.ecf8_encode(x, 1, period, **opts)
    h1, b1 = one.header, torch.from_numpy(one.numpy().copy()).to(DEV)
    assert h1.stream_bits == period + 4096 and h1.stream_bits % 128 == 0
    size = n // period * (h1.stream_bits // 8 + h1.plane_bytes + 32 * 136) + (1 << 12)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < n + size + (4 << 30):
        pytest.skip("needs %d GB of device memory" % ((n + size) >> 30))
    d_x = torch.empty(n, dtype=torch.uint8, device=DEV)
    d_x[:period] = torch.from_numpy(x).to(DEV)
    done = period
    while done < n:
        more = min(done, n - done)
        d_x[done:done + more] = d_x[:more]
        done += more
    d_blob = torch.empty(size, dtype=torch.uint8, device=DEV)
    hdr, _ = ecf8.ecf8_encode_gpu(d_x, 1, n, d_blob=d_blob, **opts)
    torch.cuda.synchronize()
    assert list(hdr.code_len) == list(h1.code_len) and hdr.stream_bits == groups * h1.stream_bits and hdr.n_chunks == 32 * groups
    cb = d_blob[hdr.off_chunk_bit:hdr.off_chunk_bit + 8 * hdr.n_chunks].view(torch.int64).view(groups, 32)
    cb1 = b1[h1.off_chunk_bit:h1.off_chunk_bit + 8 * 32].view(torch.int64)
    assert torch.equal(cb, torch.arange(groups, device=DEV)[:, None] * h1.stream_bits + cb1)
    assert int(d_blob[hdr.off_chunk_bit + 8 * hdr.n_chunks:][:8].view(torch.int64)) == hdr.stream_bits
    for at, at1, nbytes in ((hdr.off_lane_bits, h1.off_lane_bits, 128 * 32), (hdr.off_stream, h1.off_stream, h1.stream_bits // 8),
                            (hdr.off_plane, h1.off_plane, h1.plane_bytes)):
        assert _rows_equal(d_blob[at:at + groups * nbytes], b1[at1:at1 + nbytes]), at
    del d_x, d_blob, cb
    torch.cuda.empty_cache()


def test_special_histograms(orc):
    fib = [1, 1]
    while len(fib) < 16:
        fib.append(fib[-1] + fib[-2])
    deep = np.repeat(np.arange(16, dtype=np.uint8) << 3, fib)
    np.random.default_rng(0).shuffle(deep)
    cases = [np.arange(256, dtype=np.uint8).repeat(40), np.full(5000, 0x80, dtype=np.uint8),
             np.array([0x38, 0xB8, 0x3C, 0x00], dtype=np.uint8), deep,
             np.concatenate([np.full(9000, 0x38, np.uint8), np.array([0x7F, 0xFF], np.uint8)])]
    for x in cases:
        for cap in (0, 15):
            _check_same(orc, x, 1, x.size, max_code_len=cap)


def _of_counts(counts, seed):
    """A tensor in which exponent s occurs counts[s] times, shuffled."""
    rng = np.random.default_rng(seed)
    e = np.repeat(np.arange(len(counts), dtype=np.uint8), counts)
    rng.shuffle(e)
    return (e << 3) | (rng.integers(0, 256, e.size, dtype=np.uint8) & 0x87)


@pytest.mark.parametrize("cap", [4, 5, 6, 7, 8, 11, 15])
def test_codes_of_equal_counts(cap):
    """The code is made on the device: of the many cheapest codes that equal counts and sums of counts allow it has to find the CPU encoder's."""
    rng = np.random.default_rng(cap)
    for i in range(40):
        m = int(rng.integers(1, 17))
        counts = np.zeros(16, np.int64)
        kind = [rng.integers(1, 3, m), 2 ** rng.integers(0, 9, m), np.sort(rng.integers(1, 2000, m)), np.maximum(1, (3000 * 0.55 ** np.arange(m)).astype(np.int64)),
                np.full(m, 7)][i % 5]
        counts[rng.choice(16, m, replace=False)] = kind
        x = _of_counts(counts, i)
        want = ecf8.ecf8_encode(x, 1, x.size, max_code_len=cap)
        hdr, blob = ecf8.ecf8_encode_gpu(torch.from_numpy(x).to(DEV), 1, x.size, max_code_len=cap)
        assert bytes(hdr) == bytes(want.header), (cap, list(counts))
        assert np.array_equal(blob.cpu().numpy(), want.numpy()), (cap, list(counts))


@pytest.mark.parametrize("chunks", [255, 256, 257, 511, 65537])
def test_borders_of_ranges(chunks):
    """A range of chunks per compute unit, of 256 at the most: one less and more than the compute units of a whole chip, of one chunk and two, of one range and two per
    compute unit; row-tiled, where no chunk is ragged, too."""
    x = np.resize(_rand_bytes((1 << 20) + 77, chunks, conc=1.0), chunks * 2048)
    for opts in (dict(lane_syms=32), dict(lane_syms=32, max_code_len=9), dict(lane_syms=32, tile_rows=16)):
        rows, n = (16, x.size) if "tile_rows" in opts else (1, x.size - 5)
        want = ecf8.ecf8_encode(x[:n], rows, n // rows, **opts)
        hdr, blob = ecf8.ecf8_encode_gpu(torch.from_numpy(x[:n]).to(DEV), rows, n // rows, **opts)
        assert bytes(hdr) == bytes(want.header)
        assert torch.equal(blob.cpu(), torch.from_numpy(want.numpy()))


def test_a_buffer_of_the_blobs_size_and_one_byte_less():
    """That the blob does not fit is found on the device; the next call is none the wiser."""
    x = _rand_bytes(300_001, 9)
    d_x, want = torch.from_numpy(x).to(DEV), ecf8.ecf8_encode(x, 1, x.size)
    for room in (want.size, want.size - 1, want.header.off_stream + want.header.plane_bytes, want.header.off_stream + want.header.plane_bytes - 1):
        buf = torch.full((want.size + 256,), 0xA5, dtype=torch.uint8, device=DEV)
        if room == want.size:
            hdr, blob = ecf8.ecf8_encode_gpu(d_x, 1, x.size, d_blob=buf[:room])
            assert bytes(hdr) == bytes(want.header) and np.array_equal(blob.cpu().numpy(), want.numpy())
        else:
            with pytest.raises(ecf8.Ecf8Error) as e:
                ecf8.ecf8_encode_gpu(d_x, 1, x.size, d_blob=buf[:room])
            assert e.value.code == ecf8.E_CAPACITY
        torch.cuda.synchronize()
        assert bool((buf[room:] == 0xA5).all())


def test_config0_and_a_full_size_matrix(orc):
    w = synth.make(synth.config0()[0], seed=0).numpy()
    _check_same(orc, w.reshape(-1), 1024, 1024)
    spec = synth.config1(0, 1)[4]                       # l0.gate, 14336 x 4096
    wd = synth.make(spec, 0, device=DEV)
    hdr, d_blob = ecf8.ecf8_encode_gpu(wd)
    want = ecf8.ecf8_encode(wd.cpu(), spec["rows"], spec["cols"])
    torch.cuda.synchronize()
    assert bytes(hdr) == bytes(want.header)
    assert torch.equal(d_blob.cpu(), torch.from_numpy(want.numpy()))
    assert torch.equal(ecf8.ecf8_decode(hdr, d_blob), wd)


def test_on_a_side_stream():
    """The histogram is read back behind work that is still queued on the caller's stream, which is not the default one."""
    x = torch.from_numpy(_rand_bytes(2_000_001, 3)).to(DEV)
    y = torch.from_numpy(_rand_bytes(2_000_001, 4, conc=3.0)).to(DEV)
    m = torch.randn(4096, 4096, device=DEV)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        z = x.clone()
        for _ in range(8):
            m = m @ m * 1e-3
        z.copy_(y)                                             # after milliseconds of products
        hdr, d_blob = ecf8.ecf8_encode_gpu(z, 1, z.numel())
        z.copy_(x)                                             # behind the encode on the same stream
    torch.cuda.synchronize()
    want = ecf8.ecf8_encode(y.cpu(), 1, y.numel())
    assert bytes(hdr) == bytes(want.header)
    assert torch.equal(d_blob.cpu(), torch.from_numpy(want.numpy()))


def test_argument_errors():
    d_x = torch.zeros(4096, dtype=torch.uint8, device=DEV)
    with pytest.raises(ecf8.Ecf8Error) as e:
        ecf8.ecf8_encode_gpu(d_x, 1, 4096, lane_syms=48)
    assert e.value.code == ecf8.E_ARG
    with pytest.raises(ecf8.Ecf8Error) as e:
        ecf8.ecf8_encode_gpu(d_x, 1, 4096, d_blob=torch.empty(512, dtype=torch.uint8, device=DEV))
    assert e.value.code == ecf8.E_CAPACITY
    with pytest.raises(ecf8.Ecf8Error) as e:
        ecf8.ecf8_encode_gpu(d_x, 1, 4096, d_blob=torch.empty(1 << 20, dtype=torch.uint8, device=DEV)[16:])
    assert e.value.code == ecf8.E_ALIGN
    with pytest.raises(ecf8.Ecf8Error):
        ecf8.ecf8_encode_gpu(d_x, 8, 512, lane_syms=64, tile_rows=16)


def test_histograms_of_calls_at_the_same_time():
    """Eight threads, each on a stream of its own with a long copy queued before each call: every call gets its own histogram."""
    import threading
    xs = [_rand_bytes(50_000 + 8192 * i, 900 + i) for i in range(8)]
    wants = [ecf8.ecf8_encode(x, 1, x.size) for x in xs]
    big = torch.zeros(1 << 28, dtype=torch.uint8, device=DEV)
    bad = []

    def work(i):
        s = torch.cuda.Stream()
        d_x = torch.from_numpy(xs[i]).to(DEV)
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            for k in range(12):
                if k % 4 == i % 4:
                    y = big.clone()
                    y.add_(1)
                hdr, d_blob = ecf8.ecf8_encode_gpu(d_x, 1, xs[i].size)
                s.synchronize()
                if bytes(hdr) != bytes(wants[i].header) or not np.array_equal(d_blob.cpu().numpy(), wants[i].numpy()):
                    bad.append((i, k))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_refused_while_the_stream_is_captured():
    x = torch.from_numpy(_rand_bytes(100_000, 5)).to(DEV)
    out = torch.empty(1 << 18, dtype=torch.uint8, device=DEV)
    z = torch.zeros(4, device=DEV)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        z.add_(1)
        with pytest.raises(ecf8.Ecf8Error):
            ecf8.ecf8_encode_gpu(x, 1, x.numel(), d_blob=out)
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert bool((z == k + 1).all())
    hdr, blob = ecf8.ecf8_encode_gpu(x, 1, x.numel(), d_blob=out)
    assert np.array_equal(blob.cpu().numpy(), ecf8.ecf8_encode(x.cpu().numpy(), 1, x.numel()).numpy())


class _Stream:
    """A stream by its handle, as the binding takes one."""
    def __init__(self, handle):
        self.cuda_stream = handle


def test_refused_on_the_null_stream_while_another_is_captured():
    """A blocking stream that is being captured keeps the null stream from being used.  The call says so, and leaves no error behind for the next one, which
    looks for errors of its launch, nor does it spoil the capture."""
    hip = ecf8._lib
    x = _rand_bytes(100_000, 6)
    want = ecf8.ecf8_encode(x, 1, x.size)
    d_x, d_blob, out = torch.from_numpy(x).to(DEV), want.to(DEV), torch.empty(1 << 18, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    cs, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(cs), 0) == 0
    assert hip.hipStreamBeginCapture(cs, 2) == 0                        # hipStreamCaptureModeRelaxed
    with pytest.raises(ecf8.Ecf8Error) as e:
        ecf8.ecf8_encode_gpu(d_x, 1, x.size, d_blob=out, stream=_Stream(None))
    left = hip.hipPeekAtLastError()
    assert hip.hipStreamEndCapture(cs, ctypes.byref(graph)) == 0
    y = ecf8.ecf8_decode(want.header, d_blob)
    hip.hipGraphDestroy(graph)
    hip.hipStreamDestroy(cs)
    torch.cuda.synchronize()
    assert e.value.code == ecf8.E_HIP and left == 0
    assert np.array_equal(y.cpu().numpy().reshape(-1), x)


FIRST_CALL = """
import ctypes, sys, threading
import numpy as np
import torch
from paper_2510_02676_amd import ecf8, ecfw
hip = ecf8._lib
xs = np.random.default_rng(7).integers(0, 256, 1 << 22, dtype=np.uint8)
blob, wide = ecf8.ecf8_encode(xs, 1, xs.size), ecfw.ecfw_encode(ecfw.FMT_E5M2, xs, 1, xs.size)
x = torch.from_numpy(xs).to("cuda:0")
outs = [torch.empty(1 << 23, dtype=torch.uint8, device="cuda:0") for _ in range(2 * 20)]
d_blob, y = blob.to("cuda:0"), torch.zeros_like(x)
streams = [torch.cuda.Stream() for _ in range(8)]
big = [torch.zeros(1 << 27, dtype=torch.float32, device="cuda:0") for _ in streams]
torch.cuda.synchronize()

class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle

for s, b in zip(streams, big):                                          # some 10 ms: the calls wait with the stream, not with their page
    with torch.cuda.stream(s):
        for _ in range(8):
            b.add_(1)
cs, graph, run = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
assert hip.hipStreamCreateWithFlags(ctypes.byref(cs), 1) == 0
assert hip.hipStreamBeginCapture(cs, 0) == 0                            # hipStreamCaptureModeGlobal
ecf8.ecf8_decode(blob.header, d_blob, y, stream=Stream(cs.value))
bad = []

def work(i):
    s = streams[i % 8]
    try:
        if i % 2:
            hdr, b = ecf8.ecf8_encode_gpu(x, 1, xs.size, d_blob=outs[i], stream=s)
        else:
            hdr, b = ecfw.ecfw_encode_gpu(ecfw.FMT_E5M2, x, 1, xs.size, d_blob=outs[i], stream=s)
        outs[i] = b
    except Exception as e:
        bad.append((i, str(e)))

threads = [threading.Thread(target=work, args=(i,)) for i in range(len(outs))]      # more calls at a time than pages are kept
for t in threads:
    t.start()
for t in threads:
    t.join()
assert not bad, bad
assert hip.hipStreamEndCapture(cs, ctypes.byref(graph)) == 0
assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, 0) == 0
for k in range(3):
    y.fill_(0xA5)
    torch.cuda.synchronize()
    assert hip.hipGraphLaunch(run, cs) == 0 and hip.hipStreamSynchronize(cs) == 0
    assert torch.equal(y, x), k
for i, b in enumerate(outs):
    assert np.array_equal(b.cpu().numpy(), (blob if i % 2 else wide).numpy()), i
print("capture and calls whole")
"""


def test_first_calls_while_another_thread_captures():
    """In a process of its own, where no call has left a page behind: calls of other threads get their pages while this one captures a stream in the mode
    that forbids allocations in all threads, and the graph replays."""
    r = subprocess.run([sys.executable, "-c", FIRST_CALL], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "capture and calls whole" in r.stdout, r.stdout + r.stderr


NO_PAGE = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)                     # in front of the runtime's own
import numpy as np
import torch
from paper_2510_02676_amd import ecf8, ecfw
xs = np.random.default_rng(8).integers(0, 256, 100_000, dtype=np.uint8)
x = torch.from_numpy(xs).to("cuda:0")
for k in range(3):
    hdr, b = ecf8.ecf8_encode_gpu(x, 1, xs.size)
    want = ecf8.ecf8_encode(xs, 1, xs.size)
    assert bytes(hdr) == bytes(want.header) and np.array_equal(b.cpu().numpy(), want.numpy())
    hdr, b = ecfw.ecfw_encode_gpu(ecfw.FMT_BF16, x.view(torch.int16), 1, xs.size // 2)
    want = ecfw.ecfw_encode(ecfw.FMT_BF16, xs.view(np.uint16), 1, xs.size // 2)
    assert bytes(hdr) == bytes(want.header) and np.array_equal(b.cpu().numpy(), want.numpy())
    assert np.array_equal(ecf8.ecf8_decode(*ecf8.ecf8_encode_gpu(x, 1, xs.size)).cpu().numpy().reshape(-1), xs)
assert ctypes.c_int.in_dll(shim, "refused").value >= 9
print("copied instead")
"""


def test_no_pinned_page(tmp_path):
    """Where the runtime refuses a page, the header is copied.  In a process of its own, whose first library answers for the runtime."""
    (tmp_path / "shim.c").write_text("int refused; int hipHostMalloc(void **p, unsigned long n, unsigned flags) { *p = 0; refused++; return 2; }\n")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.c")], check=True, timeout=60)
    r = subprocess.run([sys.executable, "-c", NO_PAGE, str(tmp_path / "shim.so")], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "copied instead" in r.stdout, r.stdout + r.stderr
