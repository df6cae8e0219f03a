"""The workspace's two sizes on the host: ctx.hip is linked with stand-ins for the HIP calls, whose device has room for `limit`
bytes."""
import os
import subprocess

from paper_2405_14917_amd import build

PROGRAM = r"""
#include <cstdlib>

#include "slim_internal.h"

static size_t limit;
static int mallocs, frees, syncs;
extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  ++mallocs;
  *p = bytes <= limit ? malloc(64) : nullptr;
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { ++frees; free(p); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++syncs; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "out of memory"; }
}

static void either(slim_ctx& ctx, size_t full, size_t base) {
  bool has_full = false;
  mallocs = frees = syncs = 0;
  const int st = slim_ws_reserve_either(&ctx, full, base, has_full);
  printf("%d %d %zu %d %d %d\n", st, (int)has_full, ctx.ws_bytes, mallocs, frees, (int)(ctx.err[0] != 0));
}

int main() {
  slim_ctx ctx;
  limit = 600;
  either(ctx, 1000, 500);      // refused, then the base
  either(ctx, 1000, 500);      // not asked for again
  either(ctx, 1200, 500);
  either(ctx, 580, 500);       // less than what was refused
  either(ctx, 1000, 590);      // the base grows
  limit = 2000;
  either(ctx, 1000, 590);      // still remembered ...
  printf("%d\n", (int)slim_ws_reserve(&ctx, 1100));      // ... until as much is there
  either(ctx, 1000, 590);
  either(ctx, 1500, 590);
  slim_ctx theirs;             // a caller's workspace is not asked of the device at all
  theirs.ws_external = true;
  theirs.ws_bytes = 700;
  either(theirs, 1000, 500);
  either(theirs, 600, 500);
  either(theirs, 1000, 800);
  return 0;
}
"""


def test_a_refused_workspace_is_remembered(tmp_path):
    src, exe = tmp_path / "t.hip", tmp_path / "t"
    src.write_text(PROGRAM)
    objs = []
    for f in (str(src), os.path.join(build.CSRC, "ctx.hip")):
        objs.append(str(tmp_path / (os.path.basename(f) + ".o")))
        subprocess.run([build.hipcc(), "--offload-host-only", "-O1", "-fPIC", "-std=c++17", "-I" + build.INCLUDE, "-I" + build.CSRC, "-c", f, "-o", objs[-1]],
                       check=True)
    subprocess.run(["g++", *objs, "-o", str(exe), "-pthread", "-Wl,--unresolved-symbols=ignore-in-object-files"], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    # status, full size, bytes held, allocations asked for, given up, an error text left behind
    assert out[:12] == ["0 0 500 2 0 0", "0 0 500 0 0 0", "0 0 500 0 0 0", "0 1 580 1 1 0", "0 0 590 1 1 0", "0 0 590 0 0 0", "0", "0 1 1100 0 0 0",
                        "0 1 1500 1 1 0", "0 0 700 0 0 0", "0 1 700 0 0 0", "-3 0 700 0 0 1"]
