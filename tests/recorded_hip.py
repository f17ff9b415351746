"""The library's host code on a HIP runtime that runs nothing and writes down what it is asked for: which kernels with
which grids go to which streams, and which events order them.  For tests of dispatch rules and of stream order without a
GPU.  The stand-in is compiled with gcc and loaded, in a child process, ahead of the library, whose HIP calls it takes."""
import json
import os
import subprocess
import sys

from conftest import ROOT

SOURCE = r"""
#include <stdarg.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
typedef void *P;
static char *text; static size_t used, room;
static void line(const char *f, ...) {
  if (room - used < 512) text = realloc(text, room = 2 * room + 4096);
  va_list a; va_start(a, f); used += vsnprintf(text + used, 512, f, a); va_end(a);
}
const char *recorded(void) { return used ? text : ""; }
void forget(void) { used = 0; }
int complete = 0;   /* what hipEventQuery says of every event */
int capturing = 0;  /* ... and hipStreamIsCapturing of every stream */
static struct { const void *f; const char *name; } kernels[4096]; static int n_kernels;
static uintptr_t next_handle = 0x100000;
static struct { dim3 g, b; size_t s; P st; } conf;
P *__hipRegisterFatBinary(const void *d) { static P h; return &h; }
void __hipUnregisterFatBinary(P *m) {}
void __hipRegisterFunction(P *m, const void *f, char *d, const char *name, unsigned t, P a, P b, P c, P e, int *w) {
  if (n_kernels < 4096) kernels[n_kernels].f = f, kernels[n_kernels++].name = name;
}
void __hipRegisterVar(P *m, P v, char *h, char *d, int ext, size_t size, int c, int g) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, P st) { conf.g = g; conf.b = b; conf.s = s; conf.st = st; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, P *st) { *g = conf.g; *b = conf.b; *s = conf.s; *st = conf.st; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, P *args, size_t s, P st) {
  const char *name = "?";
  for (int i = 0; i < n_kernels; ++i) if (kernels[i].f == f) name = kernels[i].name;
  line("launch %lu %u %u %u %.200s\n", (unsigned long)st, g.x, g.y, b.x, name);
  return 0;
}
int hipStreamCreateWithFlags(P *s, unsigned f) { *s = (P)(next_handle += 16); line("stream %lu\n", (unsigned long)*s); return 0; }
int hipEventCreateWithFlags(P *e, unsigned f) { *e = (P)(next_handle += 16); return 0; }
int hipEventRecord(P e, P s) { line("record %lu %lu\n", (unsigned long)e, (unsigned long)s); return 0; }
int hipStreamWaitEvent(P s, P e, unsigned f) { line("wait %lu %lu\n", (unsigned long)s, (unsigned long)e); return 0; }
int capture_mode = 0;  /* the thread's: global, as every thread begins */
int hipThreadExchangeStreamCaptureMode(int *m) { int had = capture_mode; capture_mode = *m; *m = had; return 0; }
int hipEventQuery(P e) { line("query %lu %d\n", (unsigned long)e, capture_mode); return complete ? 0 : 600; }
int hipStreamIsCapturing(P s, int *status) { *status = capturing; return 0; }
int hipHostMalloc(P *p, size_t n, unsigned f) { *p = calloc(1, n); return 0; }
int hipHostFree(P p) { free(p); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(P *p, const void *s) { *p = (P)0x7000000; return 0; }
int hipStreamBeginCapture(P s, int m) { return 0; }
int hipStreamEndCapture(P s, P *g) { *g = (P)(next_handle += 16); return 0; }
int hipGraphInstantiate(P *x, P g, P *n, char *l, size_t s) { *x = (P)(next_handle += 16); return 0; }
int hipGraphLaunch(P x, P s) { line("graph %lu\n", (unsigned long)s); return 0; }
int hipMemcpyAsync(P d, const void *s, size_t n, int k, P st) { return 0; }
#define NOTHING(name) int name() { return 0; }
NOTHING(hipGetLastError) NOTHING(hipDeviceSynchronize) NOTHING(hipStreamSynchronize) NOTHING(hipStreamDestroy)
NOTHING(hipEventDestroy) NOTHING(hipEventSynchronize) NOTHING(hipGraphDestroy) NOTHING(hipGraphExecDestroy)
"""

CHILD = r"""
import ctypes as C, json, sys
hip = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
hip.recorded.restype = C.c_char_p
lib = C.CDLL(sys.argv[2])
lib.apex_codec_row_bytes.restype = C.c_size_t
address = [1 << 40]

def memory(size=1 << 36):
    "An address that nothing looks behind."
    address[0] += size
    return address[0]

def call(name, *args):
    return getattr(lib, name)(*[C.c_float(a) if isinstance(a, float) else C.c_uint64(a or 0) if a is None or isinstance(a, int)
                                else a for a in args])

def take():
    "What has been recorded since the last time: lists of words."
    lines = [l.split() for l in hip.recorded().decode().splitlines()]
    hip.forget()
    return [[int(w) if w.isdigit() else w for w in l] for l in lines]

def launches(calls=None):
    return [dict(stream=c[1], grid=c[2], grid_y=c[3], block=c[4], kernel=c[5]) for c in (take() if calls is None else calls)
            if c[0] == "launch"]

class Config(C.Structure):
    _fields_ = [("capacity", C.c_uint64), ("max_slots", C.c_uint64), ("obs_bytes", C.c_uint32), ("act_bytes", C.c_uint32),
                ("alpha", C.c_float), ("eps", C.c_float), ("frac_bits", C.c_uint32), ("reserved", C.c_uint32),
                ("min_size", C.c_uint64)]

class Buffers(C.Structure):
    _fields_ = [(n, C.c_uint64) for n in "key slot mass weight obs act ret gacc".split()]

def replay(slots, obs_bytes, filled=None, act_bytes=4):
    h = C.c_void_p()
    assert call("apex_replay_create", C.byref(Config(slots, slots, obs_bytes, act_bytes, 0.6, 1e-6, 24, 0, 0)), memory(1 << 40),
                memory(), memory(), C.byref(h)) == 0
    if filled is None or filled:
        assert call("apex_replay_add", h, filled or slots, None, None, None, None, memory(), None, None) == 0
    take()
    return h

def pipeline(r, depth, nb, k):
    h, sets = C.c_void_p(), (Buffers * depth)(*[Buffers(*[memory() for _ in range(8)]) for _ in range(depth)])
    assert call("apex_pipeline_create", r, depth, sets, nb, k, C.byref(h)) == 0
    streams = [c[1] for c in take() if c[0] == "stream"]
    return h, streams

def steps(p, n, new_prio=True):
    return call("apex_pipeline_steps", p, n, 0.4, memory(), memory() if new_prio else None, None)

def add_begin(p, S, T, n=1, A=1):
    return call("apex_pipeline_add_begin", p, S, T, n, A, *[memory() for _ in range(10)])

def add_end(p):
    return call("apex_pipeline_add_end", p, 0, None, None)

def seen(calls, had):
    '''The work of the caller's streams (had: stream -> names) that each stream is ordered behind after `calls`, and a list of
    (launch, what it is ordered behind).'''
    after, events, out = {s: set(v) for s, v in had.items()}, {}, []
    for c in calls:
        if c[0] == "record":
            events[c[1]] = set(after.get(c[2], ()))
        elif c[0] == "wait":
            after.setdefault(c[1], set()).update(events[c[2]])
        elif c[0] == "mark":            # put in by a test: from here on the stream's latest work is c[2] alone
            after[c[1]] = {c[2]}
        elif c[0] == "launch":
            out.append((c, set(after.get(c[1], ()))))
    return after, out
"""


def run(tmp_path, body):
    """Runs `body` behind CHILD in a process of its own and returns what it leaves in `result`."""
    c, so = str(tmp_path / "recorded_hip.c"), str(tmp_path / "librecorded_hip.so")
    if not os.path.exists(so):
        with open(c, "w") as f:
            f.write(SOURCE)
        subprocess.check_call(["gcc", "-O1", "-w", "-shared", "-fPIC", "-o", so, c])
    lib = os.path.join(ROOT, "paper_1803_00933_amd", "libapex_replay.so")
    code = CHILD + "\n" + body + "\nprint(json.dumps(result))\n"
    r = subprocess.run([sys.executable, "-c", code, so, lib], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    return json.loads(r.stdout.splitlines()[-1])
