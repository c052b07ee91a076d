"""What the calls queue on the device, without one: a library in front of the runtime's answers for it and counts the launches."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>
int launches, fail_at = -1, last;
hipError_t hipGetDevice(int *d) { *d = 0; return 0; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int dev) { memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return 0; }
static dim3 grid_, block_; static size_t lds_; static hipStream_t stream_;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) { grid_ = g; block_ = b; lds_ = l; stream_ = s; return 0; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) { *g = grid_; *b = block_; *l = lds_; *s = stream_; return 0; }
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t s)
{
    return launches++ == fail_at ? (last = hipErrorLaunchFailure) : hipSuccess;
}
hipError_t hipGetLastError(void) { int e = last; last = 0; return e; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) { *st = hipStreamCaptureStatusNone; return 0; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *mode) { return 0; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags) { *p = aligned_alloc(4096, 4096); return 0; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned flags) { *d = h; return 0; }
hipError_t hipHostFree(void *p) { free(p); return 0; }
hipError_t hipStreamSynchronize(hipStream_t s) { return 0; }
"""

BEGIN = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)                     # in front of the runtime's own
def var(name): return ctypes.c_int.in_dll(shim, name)
from paper_2510_02676_amd import ecf8, ecfw
"""


def run_on_shim(tmp_path, code):
    (tmp_path / "shim.c").write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-I/opt/rocm/include", "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.c")], check=True, timeout=60)
    r = subprocess.run([sys.executable, "-c", BEGIN + code + "\nprint('as expected')", str(tmp_path / "shim.so")], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "as expected" in r.stdout, r.stdout + r.stderr


FAILED_LAUNCH = r"""
x, blob = 1 << 20, 1 << 21                                              # addresses that nothing looks at
lib = ecf8._lib
h8, hw = ecf8.Header(), ecfw.WHeader()
def e4m3(): return lib.ecf8_encode_gpu(x, 64, 4096, None, blob, 1 << 20, ctypes.byref(h8), None)
def wide(fmt):
    o = ecfw.WEncodeOpts(fmt=fmt)
    return lib.ecfw_encode_gpu(x, 64, 4096, ctypes.byref(o), blob, 1 << 20, ctypes.byref(hw), None)
for call in (e4m3, lambda: wide(ecfw.FMT_BF16), lambda: wide(ecfw.FMT_E5M2)):
    for k in range(4):
        var("launches").value, var("fail_at").value = 0, k if k < 3 else -1
        assert call() == ecf8.E_HIP                                     # with all three queued: the header never comes
        assert var("launches").value == min(k + 1, 3), (k, var("launches").value)
"""


def test_nothing_is_queued_behind_a_failed_launch(tmp_path):
    """A device encode is three kernels, each of which takes from the blob what the one before has written there, places to store at among it."""
    run_on_shim(tmp_path, FAILED_LAUNCH)


MANY_CHUNKS = r"""
lib = ecf8._lib
at = 1 << 20                                                            # an address that nothing looks at
def queued(total, call):
    var("launches").value = 0
    assert call(total) == 0
    return var("launches").value
def e4m3(total):
    i = ecf8.BatchInfo(total_chunks=total, lane_syms=32, max_code_len=7)
    return lib.ecf8_decode_batched(at, 7, ctypes.byref(i), None)
def wide(total, fmt, longest):
    i = ecfw.WBatchInfo(total_chunks=total, fmt=fmt, lane_syms=64, max_code_len=longest)
    return lib.ecfw_decode_batched(at, 7, ctypes.byref(i), None)
def group(total, M):
    i = ecf8.GemmGroupInfo(total_work=total, n_items=7, max_M=M)
    return lib.ecf8_gemm_fp8_grouped(at, ctypes.byref(i), None)
calls = [e4m3] + [lambda t, f=f, l=l: wide(t, f, l) for f in (ecfw.FMT_BF16, ecfw.FMT_E5M2) for l in (12, 16)] + [lambda t, M=M: group(t, M) for M in (1, 20, 64)]
for call in calls:
    assert [queued(t, call) for t in (1, (1 << 31) - 1, 1 << 31, (1 << 31) + 1, (1 << 32) - 1, 1 << 32, (1 << 32) + 1)] == [1, 1, 1, 2, 2, 2, 3]
# one tensor of more than that
n = ((1 << 31) + 1) * 2048
h = ecf8.ecf8_encode(__import__("numpy").zeros(2048, dtype="uint8"), 1, 2048, lane_syms=32).header
def header(n):
    g = ecf8.Header.from_buffer_copy(bytes(h))
    g.rows, g.cols, g.n_elem, g.n_chunks, g.plane_bytes = 1, n, n, -(-n // 2048), -(-n // 2048) * 1024
    g.total_size = g.off_plane + g.plane_bytes
    return g
big, most = header(n), header(1 << 42)
assert lib.ecf8_decode(ctypes.byref(big), at, at, n, None) == ecf8.E_FORMAT
assert queued(0, lambda _: lib.ecf8_decode(ctypes.byref(most), at, at, n, None)) == 1
w = ecfw.ecfw_encode(ecfw.FMT_BF16, __import__("numpy").zeros(4096, dtype="uint16"), 1, 4096).header
w.n_elem, w.n_chunks = ((1 << 31) + 1) * 4096, (1 << 31) + 1
assert lib.ecfw_decode(at, ctypes.byref(w), at, 4 * w.n_elem, 0, None) == ecf8.E_FORMAT
w.n_elem, w.n_chunks = (1 << 31) * 4096, 1 << 31
assert queued(0, lambda _: lib.ecfw_decode(at, ctypes.byref(w), at, 4 * w.n_elem, 0, None)) == 1
assert lib.ecf8_gemm_fp8_raw(at, 1 << 40, 1 << 20, at, 1, at, None) == ecf8.E_ARG
"""


def test_chunk_numbers_past_32_bits(tmp_path):
    """Kernels number chunks in 32 bits: a batch or a group of more than 2^31 is several launches, a tensor of more is refused."""
    run_on_shim(tmp_path, MANY_CHUNKS)
