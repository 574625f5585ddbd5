"""The library's host code against a HIP runtime that launches nothing: a shared object whose symbols are found before those of
libamdhip64.  It keeps a list of what the library asks for (launches, copies, streams, events) and fails the call, or the allocation of
host memory, that it is told to.  Run in a process of its own (run()), since it stands in front of the real runtime."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <dlfcn.h>
#include <mutex>
#include <new>
struct Dim { uint32_t x, y, z; };
namespace {
struct Entry { char what; char name[160]; int64_t a, b, c; const void *stream; };
// what: K launch (a workgroups, b threads, c a word of the arguments), M copy, S stream made, E event made, R event a recorded, W wait for event a
Entry entries[1 << 16];
int64_t count = 0, fail_at = -1, calls = 0, allocations = 0, alloc_fail_at = -1, peek = 0;
bool capturing = false, counting = false;
int last = 0;
char failed = ' ';       // what the failing call was
intptr_t next_handle = 16;
Entry *add(char what, const void *stream) {
  Entry *e = &entries[count < (1 << 16) ? count++ : (1 << 16) - 1];
  std::memset(e, 0, sizeof *e);
  e->what = what; e->stream = stream;
  return e;
}
int result() { const int rc = fail_at >= 0 && calls++ == fail_at ? 719 : 0; if (rc) { last = rc; failed = count ? entries[count - 1].what : '?'; } return rc; }
}
extern "C" {
// the test's side
void fake_reset(int64_t fail, int64_t alloc_fail, int cap) { count = 0; calls = 0; allocations = 0; fail_at = fail; alloc_fail_at = alloc_fail; capturing = cap != 0; last = 0; failed = ' '; }
int fake_failed() { return failed; }
void fake_count_allocations(int on) { counting = on != 0; }
void fake_peek(int64_t word) { peek = word; }
int64_t fake_entries(Entry **e) { *e = entries; return count; }
int64_t fake_calls() { return calls; }
int64_t fake_allocations() { return allocations; }
// the library's side
int hipLaunchKernel(const void *f, Dim grid, Dim block, void **args, size_t, void *stream) {
  Entry *e = add('K', stream);
  Dl_info info;
  if (dladdr(f, &info) && info.dli_sname) std::snprintf(e->name, sizeof e->name, "%s", info.dli_sname);
  e->a = (int64_t)grid.x * grid.y * grid.z; e->b = block.x;
  std::memcpy(&e->c, static_cast<const char *>(args[0]) + peek, 8);
  if ((uint64_t)grid.x * block.x > 0xffffffffull || (uint64_t)grid.y * block.y > 0xffffffffull) { last = 9; return 9; }
  return result();
}
namespace { struct { Dim grid, block; size_t shared; void *stream; } config; }
int __hipPushCallConfiguration(Dim grid, Dim block, size_t shared, void *stream) { config = {grid, block, shared, stream}; return 0; }
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *shared, void **stream) {
  *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
  return 0;
}
int hipMemcpyAsync(void *, const void *, size_t, int, void *s) { add('M', s); return result(); }
int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, int, void *s) { add('M', s); return result(); }
int hipMemcpy(void *, const void *, size_t, int) { return result(); }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = (void *)(next_handle += 16); add('S', *s); return result(); }
int hipEventCreateWithFlags(void **e, unsigned) { *e = (void *)(next_handle += 16); add('E', nullptr); return result(); }
int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventRecord(void *e, void *s) { add('R', s)->a = (int64_t)e; return result(); }
int hipStreamWaitEvent(void *s, void *e, unsigned) { add('W', s)->a = (int64_t)e; return result(); }
int hipStreamIsCapturing(void *, int *status) { *status = capturing ? 1 : 0; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.f; return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { const int rc = last; last = 0; return rc; }
}
void *operator new(size_t n) {
  if (counting && allocations++ == alloc_fail_at) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
"""

PRELUDE = r"""
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
from paper_2309_06497_amd import binding as B
L = B.lib()
i64 = ctypes.c_int64
class Entry(ctypes.Structure):
    _fields_ = [("what", ctypes.c_char), ("name", ctypes.c_char * 160), ("a", i64), ("b", i64), ("c", i64), ("stream", ctypes.c_void_p)]
fake.fake_entries.restype = fake.fake_calls.restype = fake.fake_allocations.restype = i64
def reset(fail=-1, alloc_fail=-1, capturing=0):
    fake.fake_reset(i64(fail), i64(alloc_fail), int(capturing))
def entries():
    p = ctypes.POINTER(Entry)()
    return [p[k] for k in range(fake.fake_entries(ctypes.byref(p)))]
def launches(name=""):
    return [e for e in entries() if e.what == b"K" and name.encode() in e.name]
STREAM = 7 << 20                      # the caller's
def failing(call, limit=1 << 20):
    # the call with its first request to the runtime failing, its second one, and so on until it succeeds: what failed, and the code
    for k in range(limit):
        reset(fail=k)
        rc = call()
        if fake.fake_calls() <= k:
            assert rc == 0, rc
            return
        yield chr(fake.fake_failed()), rc
def out_of_memory(call, limit=1 << 20):
    # the same for allocations of host memory
    for k in range(limit):
        reset(alloc_fail=k)
        fake.fake_count_allocations(1)
        rc = call()
        fake.fake_count_allocations(0)
        if fake.fake_allocations() <= k:
            assert rc == 0, rc
            return
        yield rc
class Opt:
    # memory of the device is never touched: addresses that nothing lies at
    def __init__(self, shapes, block, freq=100, start=0, **kw):
        self.cfg = B.make_config(shapes, block, 0.999, 1e-12, kw.pop("r", 0.25), freq, start, **kw)
        self.n, self.handle = len(shapes), ctypes.c_void_p()
        nbytes = B.shampoo_workspace_bytes(self.cfg)
        rc = L.shampoo_create(ctypes.byref(self.cfg), ctypes.c_void_p(1 << 40), nbytes, ctypes.c_void_p(STREAM), ctypes.byref(self.handle))
        assert rc == 0, rc
    def pointers(self, where, skew=0):
        return (ctypes.c_void_p * self.n)(*[(where << 36) + (k << 28) + skew for k in range(self.n)])
    def step(self, t, where=1, skew=0):
        w, g = self.pointers(where), self.pointers(where + 1, skew)
        return L.shampoo_step(self.handle, w, g, 0.01, t, ctypes.c_void_p(STREAM))
    def timing(self, on):
        assert L.shampoo_set_timing(self.handle, int(on)) == 0
    def get(self, param, block, which, nbytes):
        return L.shampoo_get(self.handle, param, block, which, ctypes.c_void_p(1 << 39), nbytes, ctypes.c_void_p(STREAM))
def unjoined():
    # helper streams with work that the caller's stream does not wait for at the end of the list
    # clock[s]: for every stream, how much of its work stream s has waited for
    done, clock, at = {}, {}, {}
    for e in entries():
        s = e.stream
        own = clock.setdefault(s, {})
        if e.what in (b"K", b"M"):
            done[s] = own[s] = done.get(s, 0) + 1
        elif e.what == b"R":
            at[e.a] = dict(own)
        elif e.what == b"W":
            for k, v in at.get(e.a, {}).items():
                own[k] = max(own.get(k, 0), v)
    seen = clock.get(STREAM, {})
    return [s for s in done if s != STREAM and seen.get(s, 0) < done[s]]
"""


def build(folder):
    src, lib = os.path.join(folder, "fake_hip.cpp"), os.path.join(folder, "fake_hip.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", src, "-o", lib, "-ldl"], check=True)
    return lib


def run(lib, code):
    """Runs the code behind the prelude; returns what it prints, line by line."""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", CUDA_VISIBLE_DEVICES="", PYTHONPATH=ROOT)
    p = subprocess.run([sys.executable, "-c", PRELUDE + code, lib], env=env, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, (p.returncode, p.stdout[-2000:], p.stderr[-2000:])
    return p.stdout.split("\n")
