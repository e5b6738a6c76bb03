"""Launches and allocations that the runtime refuses, on the CPU: the library
over a stand-in for the HIP runtime (device memory is host memory, kernels do
not run) in which they fail on request."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
struct dim3 { uint32_t x, y, z; };
static int fail = 0, launches = 0;
static size_t most = ~(size_t)0, bytes = 0;
static thread_local int sticky = 0;
static struct { dim3 g, b; size_t m; void *s; } cfg;
extern "C" {
void fake_fail(int on) { fail = on; }
void fake_most(size_t bytes) { most = bytes; }
int fake_launches() { return launches; }
size_t fake_bytes() { return bytes; }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, void *s) { cfg.g = g; cfg.b = b; cfg.m = m; cfg.s = s; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, void **s) { *g = cfg.g; *b = cfg.b; *m = cfg.m; *s = cfg.s; return 0; }
int hipLaunchKernel(const void *, dim3, dim3, void **, size_t, void *) {
    ++launches;
    if (fail) sticky = 9;  // hipErrorInvalidConfiguration
    return fail ? 9 : 0;
}
int hipGetLastError() { int e = sticky; sticky = 0; return e; }
const char *hipGetErrorString(int) { return "refused"; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 100000; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipSetDevice(int) { return 0; }
int hipMalloc(void **p, size_t n) { bytes += n; *p = n > most ? 0 : calloc(1, n ? n : 1); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
int hipHostFree(void *p) { free(p); return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return 0; }
int hipGetSymbolAddress(void **p, const void *) { static void *a = calloc(1, 64 << 20); *p = a; return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { memcpy(d, s, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *) { if (v) memset(d, v, n); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1; return 0; }
}
"""

SETUP = r"""
import ctypes, sys
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_1807_08804_amd as P
from tests.micro import MicroQuery

a = np.arange(20, dtype=np.int32)
g = P.Graph(np.arange(21, dtype=np.int32), (a + 1) % 20, a * 0, a * 0)
q = MicroQuery(2, [-1, 0], [-1, -1], [0], [1], [0])
assert rt.fake_launches() == 0


def status(f):
    try:
        f()
        return P.SGM_OK
    except P.SGMError as e:
        return e.code


"""

LAUNCHES = SETUP + r"""
calls = [lambda: g.match_query(q), lambda: g.match_batch([q, q]),
         lambda: g.match_query_noalloc(q, 16)]
# kernels that do not run leave zeroed results: no rows
assert [status(f) for f in calls] == [P.SGM_OK] * 3 and rt.fake_launches() >= 3
rt.fake_fail(1)
print("refused:", [status(f) for f in calls])
assert [status(f) for f in calls] == [P.SGM_EDEVICE] * 3
srv = P.Server(g)
assert srv.wait(srv.submit(q), q.n)[0] == P.SGM_EDEVICE
rt.fake_fail(0)
assert srv.wait(srv.submit(q), q.n)[0] == P.SGM_OK
srv.close()
print("again:", [status(f) for f in calls])
assert [status(f) for f in calls] == [P.SGM_OK] * 3
g.close()
print("ok")
"""


ALLOCATIONS = SETUP + r"""
for most in (1 << 29, 1 << 19, 4000):  # the output arena, slot memory, small buffers
    rt.fake_most(ctypes.c_size_t(most))
    for calls in range(3):
        assert status(lambda: g.match_query(q)) == P.SGM_EDEVICE
        assert status(lambda: g.match_batch([q, q])) == P.SGM_EDEVICE
    rt.fake_most(ctypes.c_size_t(1 << 62))
    assert status(lambda: g.match_query(q)) == P.SGM_OK
    g.close()
    g = P.Graph(np.arange(21, dtype=np.int32), (a + 1) % 20, a * 0, a * 0)
g.close()
print("ok")
"""


RERUNS = SETUP + r"""
# a root of more vertices than a regular list: served by the rerun thread
V = 70000
b = np.arange(V, dtype=np.int32)
g = P.Graph(np.arange(V + 1, dtype=np.int32), (b + 1) % V, b * 0, b * 0)
srv = P.Server(g)
q = MicroQuery(2, [-1, -1], [-1, -1], [0], [1], [0])
assert srv.wait(srv.submit(q), q.n)[0] == P.SGM_OK
rt.fake_fail(1)
assert srv.wait(srv.submit(q), q.n)[0] == P.SGM_EDEVICE
rt.fake_fail(0)
assert srv.wait(srv.submit(q), q.n)[0] == P.SGM_OK
srv.close()
g.close()
print("ok")
"""


def test_a_refused_rerun_is_an_error(tmp_path):
    """A served query whose rerun in a larger slot fails is reported, not
    answered with no rows."""
    run(tmp_path, RERUNS)


MEMORY = SETUP + r"""
rt.fake_bytes.restype = ctypes.c_size_t
V = 100000
at, size = np.zeros(V + 1, np.int32), {}
for out_only in (0, 1):
    b = rt.fake_bytes()
    P.Graph(at, a[:0], a[:0], np.zeros(V, np.int32), out_only=out_only).close()
    size[out_only] = rt.fake_bytes() - b
print(size)
assert size[1] + 36 * V <= size[0]
print("ok")
"""


def test_outgoing_graph_alone_holds_its_own_arrays(tmp_path):
    """The row extents and type order that the persistent kernel reads (36
    bytes a vertex and more) are not kept for a graph that never runs it."""
    run(tmp_path, MEMORY)


def run(tmp_path, script):
    src, lib = tmp_path / "fakehip.cpp", tmp_path / "libfakehip.so"
    src.write_text(RUNTIME)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    out = subprocess.run([sys.executable, "-c", script, str(lib)], cwd=ROOT, capture_output=True,
                         text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.endswith("ok\n"), out.stdout + out.stderr


def test_a_refused_allocation_stays_an_error(tmp_path):
    """A context whose buffers could not all be had is not used: every call
    reports it, until there is memory again."""
    run(tmp_path, ALLOCATIONS)


def test_a_refused_launch_is_an_error(tmp_path):
    """Results are read from the memory that the kernel writes: a launch that
    the runtime refuses ends the call with a device error (a batch, a served
    query and one without allocation too), and the next call is answered."""
    run(tmp_path, LAUNCHES)
