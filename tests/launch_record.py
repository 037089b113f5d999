"""A stand-in for the HIP runtime, for CPU tests of the library's host code: it
records the kernels that a call launches (names, grids, dynamic LDS) and can
fail a launch or an allocation or choose the fastest of several timed trials.
Nothing runs on a device.

`record(tmp_path, code)` runs `code` in a process of its own where `lib` is the
built library bound to the stand-in, `rec` the stand-in's controls, `bits`,
`p` and `q` whatever is passed in `env`; `code` fills the dict `out`, which is
returned.
"""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2504_03909_amd", "libhe_mi355x.so")

STUB = r"""
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>
struct Dim { uint32_t x, y, z; };
struct Launch { std::string name; uint32_t grid; uint64_t dyn, first, second; };
static std::map<const void *, std::string> names;
static std::vector<Launch> launches;
static std::map<void *, size_t> live;
static size_t total = 0, limit = ~(size_t)0;
static std::string fail_name;
static int last = 0, timed = 0, fastest = -1;
static struct { Dim g, b; size_t shm; void *s; } conf;
static void *handle;
static char scratch[256];
extern "C" {
// ---- controls
void rec_reset() { launches.clear(); timed = 0; }
int rec_count() { return (int)launches.size(); }
int rec_registered() { return (int)names.size(); }
const char *rec_name(int i) { return launches[i].name.c_str(); }
uint32_t rec_grid(int i) { return launches[i].grid; }
uint64_t rec_dyn(int i) { return launches[i].dyn; }
uint64_t rec_arg0(int i) { return launches[i].first; }
uint64_t rec_arg1(int i) { return launches[i].second; }
void rec_fail(const char *name) { fail_name = name; }
void rec_fastest(int trial) { fastest = trial; timed = 0; }
int rec_timed() { return timed; }
void rec_limit(uint64_t bytes) { limit = bytes; }
uint64_t rec_total() { return total; }
// ---- the runtime
void **__hipRegisterFatBinary(const void *) { return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *dev, unsigned, void *, void *, void *, void *,
                           int *) { names[host] = dev; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim g, Dim b, size_t shm, void *s) { conf = {g, b, shm, s}; return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *shm, void **s) {
  *g = conf.g; *b = conf.b; *shm = conf.shm; *s = conf.s;
  return 0;
}
int hipLaunchKernel(const void *fn, Dim g, Dim, void **args, size_t shm, void *) {
  Launch l{names.count(fn) ? names[fn] : "?", g.x, shm, 0, 0};
  const bool bad = !fail_name.empty() && l.name.find(fail_name) != std::string::npos;
  if (l.name.find("k_fill") != std::string::npos) {
    memcpy(&l.first, args[0], 8);
    memcpy(&l.second, args[1], 8);
  }
  if (bad) l.name = "failed " + l.name;
  launches.push_back(l);
  if (bad) last = 1;
  return bad ? 1 : 0;
}
int hipGetLastError() { const int e = last; last = 0; return e; }
const char *hipGetErrorString(int) { return "stand-in error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipMalloc(void **p, size_t n) {
  if (total + n > limit || !(*p = calloc(1, n ? n : 1))) return last = 2;
  total += n;
  live[*p] = n;
  return 0;
}
int hipFree(void *p) {
  if (p) { total -= live[p]; live.erase(p); free(p); }
  return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipEventCreate(void **e) { *e = &handle; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = timed++ == fastest ? 1.f : 2.f; return 0; }
int hipFuncGetAttributes(void *a, const void *) { memset(a, 0, 56); return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = scratch; return 0; }
// blocks per compute unit: one for a kernel whose name holds rec_single's text, else two
static std::string single;
void rec_single(const char *name) { single = name; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *fn, int, size_t) {
  *n = !single.empty() && names.count(fn) && names[fn].find(single) != std::string::npos ? 1 : 2;
  return 0;
}
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = &handle; return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = &handle; return 0; }
int hipGraphInstantiate(void **e, void *, void *, char *, size_t) { *e = &handle; return 0; }
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
}
"""

PRELUDE = r"""
import ctypes, json, sys
env = json.loads(sys.argv[3])
# loaded first and globally, so that the library's references find it before the real runtime
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
# the calls below pass addresses that are no device memory: never to a real runtime
assert rec.rec_registered() > 0, "the library is not bound to the stand-in"
u32, u64, vp = ctypes.c_uint32, ctypes.c_uint64, ctypes.c_void_p
rec.rec_name.restype = ctypes.c_char_p
for f in ("rec_dyn", "rec_arg0", "rec_arg1", "rec_total"):
    getattr(rec, f).restype = u64
rec.rec_limit.argtypes = [u64]
lib.he_last_error.restype = lib.he_ckks_last_error.restype = ctypes.c_char_p

def launches():
    return [(rec.rec_name(i).decode(), rec.rec_grid(i), rec.rec_dyn(i)) for i in range(rec.rec_count())]

def limbs(x, n):
    return (u32 * n)(*[(x >> (32 * i)) & 0xFFFFFFFF for i in range(n)])

def key(bits, p, q):
    h = vp()
    assert lib.he_key_import(u32(bits), limbs(p, bits // 64), limbs(q, bits // 64), ctypes.byref(h)) == 0
    return h

out = {}
"""


def record(tmp_path, code, **env):
    stub = os.path.join(str(tmp_path), "librec.so")
    if not os.path.exists(stub):
        src = os.path.join(str(tmp_path), "rec.cpp")
        with open(src, "w") as f:
            f.write(STUB)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", src, "-o", stub], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE + code + "\nprint(json.dumps(out))", stub, LIB, json.dumps(env)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.splitlines()[-1])
