"""The loader's host side (csrc/kvh_loader.hip) over a HIP runtime of the test's own: what it enqueues where, and what it waits
for when a call of the runtime fails.  The file is compiled for the host alone; streams and events are numbers and every call
is written to a log, so nothing here touches a GPU."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LOADER = os.path.join(ROOT, "paper_2509_00105_amd", "csrc", "kvh_loader.hip")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")

RUNTIME = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string>
namespace kvh { struct DecodeParams; }
struct ihipStream_t;
static std::string journal;
static long next_handle = 100, calls, failing = -1, last_error;
static bool fails(const char* what, const void* a, const void* b) {
  char line[96];
  const bool bad = ++calls == failing;
  snprintf(line, sizeof line, "%s %ld %ld%s\n", what, (long)a, (long)b, bad ? " FAILED" : "");
  journal += line;
  if (bad) last_error = 1;
  return bad;
}
extern "C" {
char FATBIN[64];
const char* log_text() { return journal.c_str(); }
void log_clear(long fail_at) { journal.clear(); calls = last_error = 0; failing = fail_at; }
void restart() { next_handle = 100; log_clear(-1); }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)next_handle++; return 0; }
int hipStreamDestroy(void* s) { return fails("stream_destroy", s, 0); }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)next_handle++; return 0; }
int hipEventDestroy(void* e) { return fails("event_destroy", e, 0); }
int hipEventRecord(void* e, void* s) { return fails("record", s, e); }
int hipEventSynchronize(void* e) { return fails("event_sync", e, 0); }
int hipStreamWaitEvent(void* s, void* e, unsigned) { return fails("wait", s, e); }
int hipStreamSynchronize(void* s) { return fails("sync", s, 0); }
int hipGetLastError() { const int e = (int)last_error; last_error = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x100000; return 0; }
int hipPointerGetAttributes(int* at, const void*) { *at = 1; return 0; }  // hipMemoryTypeHost
struct Dim3 { uint32_t x, y, z; };
int hipLaunchKernel(const void*, Dim3 g, Dim3, void**, size_t, void* s) { return fails("copy", s, (void*)(size_t)g.x); }
static void* launch_stream;
static Dim3 launch_grid;
int __hipPushCallConfiguration(Dim3 g, Dim3, size_t, void* s) { launch_stream = s; launch_grid = g; return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* n, void** s) { *g = launch_grid; *b = {1, 1, 1}; *n = 0; *s = launch_stream; return 0; }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
size_t kvh_blob_size(int l, int n, int c, int) { return (size_t)l * n * c; }
int kvh_kept_tokens(int orig, int, int) { return orig; }
}
namespace kvh {
int launch_decode(DECODE_ARGS ihipStream_t* s) { return fails("decode", s, 0) ? -6 : 0; }
}
"""


@pytest.fixture(scope="module")
def loader(tmp_path_factory):
    d = tmp_path_factory.mktemp("loader")
    obj, so = str(d / "loader.o"), str(d / "loader.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "--cuda-host-only", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-c", "-o", obj, LOADER], check=True, stderr=subprocess.DEVNULL)
    undefined = subprocess.run(["nm", "-uC", obj], check=True, capture_output=True, text=True).stdout
    args = re.search(r"kvh::launch_decode\((.*)ihipStream_t\*\)", undefined).group(1).replace("kvh::", "")
    text = RUNTIME.replace("FATBIN", re.search(r"__hip_fatbin\w*", undefined).group(0)).replace("DECODE_ARGS", args)
    (d / "runtime.cpp").write_text(text)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-o", so, obj, str(d / "runtime.cpp")], check=True)
    lib = ctypes.CDLL(so)
    lib.log_text.restype = ctypes.c_char_p
    lib.kvh_loader_slot_bytes.restype = ctypes.c_size_t
    return lib


class View(ctypes.Structure):
    _fields_ = [("k", ctypes.c_void_p), ("v", ctypes.c_void_p), ("layer_stride", ctypes.c_int64), ("token_stride", ctypes.c_int64)]


ITEM = np.dtype([("blob_host", "<u8"), ("n_tokens", "<i4"), ("level", "<i4"), ("dst_token0", "<i8"), ("page_table", "<u8"),
                 ("orig_tokens", "<i4"), ("sink", "<i4"), ("window", "<i4"), ("compact", "<i4")], align=True)
COMPUTE = 7  # the caller's stream


class Session:
    """A loader of two slots that hold 4 blobs of 16 KiB each."""

    def __init__(self, lib, slot=4 * 16384):
        self.lib, self.ld = lib, ctypes.c_void_p()
        lib.restart()
        assert lib.kvh_loader_create(ctypes.byref(self.ld), ctypes.c_void_p(0x10000), ctypes.c_size_t(2 * (1536 + slot)), 2) == 0

    def log(self):
        return [ln.split() for ln in self.lib.log_text().decode().splitlines()]

    def run(self, blobs, fail_at=-1, stream=COMPUTE, tokens=16):
        items = np.zeros(blobs, dtype=ITEM)
        items["blob_host"], items["n_tokens"] = 0x20000, tokens
        view = View(0x30000, 0x30000, 1024 * 1024, 1024)
        self.lib.log_clear(ctypes.c_long(fail_at))
        rc = self.lib.kvh_loader_run(self.ld, ctypes.c_void_p(items.ctypes.data), blobs, 1, 1, 1024, ctypes.byref(view), 16, None, ctypes.c_void_p(stream))
        return rc, self.log()

    def destroy(self):
        self.lib.log_clear(ctypes.c_long(-1))
        assert self.lib.kvh_loader_destroy(self.ld) == 0
        return self.log()


def left_running(log):
    """Streams with a copy or a decode that neither the event of its slot (recorded behind the decode, which has waited for the copy)
    nor a wait for the stream covers."""
    running, last = set(), None
    for what, a, _, *failed in log:
        if failed:
            continue
        if what in ("copy", "decode"):
            running.add(a)
            last = what
        elif what == "sync":
            running.discard(a)
        elif what == "record" and a == str(COMPUTE) and last == "decode":
            running.clear()
    return running


@pytest.mark.parametrize("blobs", (1, 4, 5, 11))
def test_a_failed_run_leaves_no_work_on_a_slot(loader, blobs):
    """Whichever call of the runtime fails, an error comes back and nothing still reads or writes a slot that a later run, maybe on
    another stream, would take as free."""
    s = Session(loader)
    rc, whole = s.run(blobs)
    assert rc == 0 and sum(w == "decode" for w, *_ in whole) == -(-blobs // 4)
    for fail_at in range(1, len(whole) + 1):
        s = Session(loader)
        rc, log = s.run(blobs, fail_at)
        assert rc == (-6 if whole[fail_at - 1][0] == "decode" else rc) != 0 and log[:fail_at - 1] == whole[:fail_at - 1], (fail_at, whole[fail_at - 1])
        assert not left_running(log), (fail_at, log)


def test_runs_of_one_group_stay_on_the_callers_stream(loader):
    s = Session(loader)
    for blobs, streams in ((4, {str(COMPUTE)}), (1, {str(COMPUTE)})):
        rc, log = s.run(blobs)
        assert rc == 0 and [w for w, *_ in log] == ["copy", "decode", "record"] and {a for _, a, _ in log} == streams
    assert s.run(1)[1][0][:2] == ["wait", str(COMPUTE)]  # both slots have been used: the copy waits until this one is free
    rc, log = s.run(5)
    assert rc == 0 and len({a for w, a, _ in log if w == "copy"}) == 1 and {a for w, a, _ in log if w == "copy"} != {str(COMPUTE)}


def test_destroy_waits_for_the_copies_first(loader):
    s = Session(loader)
    s.run(3)
    what = [w for w, *_ in s.destroy()]
    assert what[:2] == ["sync", "event_sync"] and what.count("stream_destroy") == 1 and what.count("event_destroy") == 5


def test_blocks_of_a_copy(loader):
    """A block for each tile of 16 KiB up to 16, 48 for groups above 12 MiB, and one that writes the descriptors.  Between them lies
    what is slower than either: 32 blobs of 0.37 MB in groups of 4 took 351 us with 16 blocks, 360 to 445 with 24 and 32, 378 with 48."""
    s = Session(loader, slot=16 << 20)
    grid = lambda blobs, tokens: [int(b) for w, _, b in s.run(blobs, tokens=tokens)[1] if w == "copy"]
    assert grid(1, 1) == [2] and grid(4, 16) == [5] and grid(32, 16) == [17] and grid(3, 256 * 16) == [17]
    assert grid(1, 768 * 16) == [17] and grid(1, 768 * 16 + 1) == [49] and grid(4, 256 * 16) == [49] and grid(5, 256 * 16) == [49, 17]
