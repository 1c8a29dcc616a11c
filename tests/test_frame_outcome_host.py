"""Host side of a plain frame's outcome, without a GPU: the library runs over a stand-in HIP runtime
with two devices whose kernels do nothing, and what it asks of the runtime is recorded.  A wait for a
frame asks the frame's own device; and a stamp slot whose last frame may still be queued on another
stream is not given to a frame before that stream has drained, whatever was rendered in between."""
import subprocess
import sys
import tempfile
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent

RUNTIME = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cstddef>
static thread_local int device = 0;
static void note(const char* what, const void* stream) { std::printf("%s dev%d stream%zu\n", what, device, (size_t)stream); std::fflush(stdout); }
extern "C" {
struct dim3_ { unsigned x, y, z; };
int hipGetDeviceCount(int* n) { *n = 2; return 0; }
int hipSetDevice(int d) { device = d; return 0; }
int hipGetSymbolAddress(void** p, const void*) { static char w[512]; *p = w + 256 - (size_t)w % 256; return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = std::aligned_alloc(256, (n + 255) / 256 * 256); return 0; }
int hipHostFree(void* p) { std::free(p); return 0; }
int hipMalloc(void** p, size_t n) { *p = std::aligned_alloc(256, (n + 255) / 256 * 256); return 0; }
int hipFree(void* p) { std::free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { std::memcpy(d, s, n); return 0; }
int hipGetLastError() { return 0; }
int hipDeviceSynchronize() { return 0; }
static thread_local struct { dim3_ grid, block; size_t shared; void* stream; } call;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t n, void* st) { call = {g, b, n, st}; return 0; }
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* n, void** st) {
    *g = call.grid, *b = call.block, *n = call.shared, *st = call.stream;
    return 0;
}
int hipLaunchKernel(const void*, dim3_, dim3_, void**, size_t, void* st) { note("launch", st); return 0; }
int hipStreamSynchronize(void* st) { note("synchronize", st); return 0; }
int hipStreamQuery(void* st) { note("query", st); return 0; }
}
"""

PROGRAM = r"""
import ctypes as C, sys
C.CDLL(sys.argv[1], C.RTLD_GLOBAL)          # before the library: its calls bind here
import numpy as np
import paper_2608_15785_amd as rgs
from paper_2608_15785_amd import _binding as B
import workloads as wl

sc = wl.config_scene("small", n=300)
cam = wl.config_camera("small", width=64, height=48)
cc = B.camera_struct(cam)
img = np.zeros((3, 48, 64), np.float32)

def workspace(path):
    n = rgs.workspace_size(300, 64, 48, path, 5000)
    buf = np.zeros(n + 256, np.uint8)
    return buf, buf.ctypes.data + (-buf.ctypes.data) % 256, n

def render(ctx, ds, path, ws):
    assert B.lib.rgs_render(ctx.handle, ds.handle, C.byref(cc), 64, 48, B.PATHS[path], ws[1], ws[2],
                            img.ctypes.data, None) == 0

def mark(text):
    print("--", text, flush=True)
"""


def run(body):
    with tempfile.TemporaryDirectory() as d:
        src, lib = Path(d) / "runtime.cpp", Path(d) / "runtime.so"
        src.write_text(RUNTIME)
        subprocess.run(["g++", "-shared", "-fPIC", "-std=c++17", "-w", str(src), "-o", str(lib)], check=True)
        r = subprocess.run([sys.executable, "-c", PROGRAM + body, str(lib)], cwd=ROOT, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return r.stdout.split("-- asked\n")[1].split("--")[0].split("\n")[:-1]


@pytest.mark.parametrize("call", ["rgs_frame_outcome(ctx.handle, ws[1], None, 300)",
                                  "rgs_workspace_check(ctx.handle, ws[1], None, 300)"])
def test_waits_ask_the_contexts_device(call):
    """A context of device 1 on the default stream, asked while device 0 is current."""
    asked = run(f"""
ctx, other = B.Context(1, 0), B.Context(0, 0)
ds, ws = B.DeviceScene(ctx, sc, ("plain",)), workspace("plain")
render(ctx, ds, "plain", ws)
B.DeviceScene(other, sc, ("plain",))        # leaves device 0 current
mark("asked")
B.lib.{call}
mark("end")
""")
    assert asked and all("dev1" in line for line in asked)


@pytest.mark.parametrize("between", ["", "render(ctx, ds, 'fast', ws)", "ctx.set_stream(5); render(ctx, ds, 'fast', ws)"])
def test_a_slot_changes_streams_after_its_frame(between):
    """A plain frame on stream 7, perhaps another path's frame into its workspace (which retires
    the record), then a plain frame on stream 9: stream 7 drains first, or the slot is another."""
    asked = run(f"""
ctx = B.Context(0, 7)
ds = B.DeviceScene(ctx, sc, ("plain", "fast"))
spaces = [workspace("plain") for _ in range(9)]
ws = spaces[0]
for w in spaces[:8]:
    render(ctx, ds, "plain", w)             # every slot in use on stream 7
{between}
ctx.set_stream(9)
mark("asked")
render(ctx, ds, "plain", spaces[8])
mark("end")
""")
    assert asked[0].startswith("synchronize") and asked[0].endswith("stream7")
    assert len(asked) > 4 and all(line == "launch dev0 stream9" for line in asked[1:])


def test_a_free_slot_needs_no_wait():
    asked = run("""
ctx = B.Context(0, 7)
ds = B.DeviceScene(ctx, sc, ("plain", "fast"))
ws = workspace("plain")
render(ctx, ds, "plain", ws)
render(ctx, ds, "fast", ws)
ctx.set_stream(9)
mark("asked")
render(ctx, ds, "plain", ws)
mark("end")
""")
    assert len(asked) > 3 and all(line == "launch dev0 stream9" for line in asked)
