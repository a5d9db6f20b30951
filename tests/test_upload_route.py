"""Which way a staging buffer is uploaded (by a kernel or by the runtime's copy), and what callers are told of launches.  The library runs in a
small program that answers the HIP calls in the runtime's place: no GPU is needed, and memory that no kernel may touch can be named."""
import os
import shutil
import subprocess

import pytest

from paper_2508_15919_amd import binding as hb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include "hfxattn.h"

struct Memory { char* at; size_t size; int type, device; char* on_gpu; };
static Memory memory[2];                      // the staging buffer and the descriptor
static int current, stream_device, launches, copies, pending, fail_launch;

static const Memory* find(const void* p) {
  for (const Memory& m : memory)
    if (m.type != hipMemoryTypeUnregistered && (char*)p >= m.at && (char*)p < m.at + m.size) return &m;
  return nullptr;
}

extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) {      // the runtime's reads through the handle
  if ((uintptr_t)s < 4096) std::abort();
  *d = stream_device;
  return hipSuccess;
}
hipError_t hipPeekAtLastError(void) { return (hipError_t)pending; }
hipError_t hipGetLastError(void) { int e = pending; pending = 0; return (hipError_t)e; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof *a);
  if (const Memory* m = find(p)) {
    a->type = (hipMemoryType)m->type;
    a->device = m->device;
    a->devicePointer = m->on_gpu + ((char*)p - m->at);
  }
  return hipSuccess;
}
hipError_t hipDrvPointerGetAttributes(unsigned n, hipPointer_attribute* which, void** data, hipDeviceptr_t p) {
  const Memory* m = find(p);
  for (unsigned i = 0; i < n; ++i) switch (which[i]) {
    case HIP_POINTER_ATTRIBUTE_MEMORY_TYPE: *(unsigned*)data[i] = m ? m->type : 0; break;
    case HIP_POINTER_ATTRIBUTE_DEVICE_POINTER: *(void**)data[i] = m ? m->on_gpu + ((char*)p - m->at) : nullptr; break;
    case HIP_POINTER_ATTRIBUTE_DEVICE_ORDINAL: *(int*)data[i] = m ? m->device : -2; break;
    case HIP_POINTER_ATTRIBUTE_RANGE_START_ADDR: *(void**)data[i] = m ? m->at : nullptr; break;
    case HIP_POINTER_ATTRIBUTE_RANGE_SIZE: *(size_t*)data[i] = m ? m->size : 0; break;
    default: return hipErrorInvalidValue;
  }
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* q) { *g = *b = dim3(1); *s = 0; *q = nullptr; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char scratch[256]; *p = scratch; return hipSuccess; }
static bool page_list;
static int32_t launched[6];                   // what a launch of the page copy carries
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t) {
  if (page_list) std::memcpy(launched, args[0], sizeof launched);
  if (fail_launch) return (hipError_t)(pending = hipErrorInvalidConfiguration);
  ++launches;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { ++copies; return hipSuccess; }
}

// staging: type, bytes of it that are known; descriptor: type, device, bytes; current device, the stream's device; pending error; a
// launch fails; the call after building; the stream's handle
int main(int, char** v) {
  static const int32_t kind[3] = {0, 0, 1}, q_len[3] = {1, 1, 20}, ctx[3] = {40, 33, 20}, indptr[4] = {0, 3, 6, 8}, pages[8] = {0, 1, 2, 3, 4, 5, 6, 7};
  const hfx_shape shape = {4, 2, 64, 16, 8, 0.f};
  size_t host_bytes, device_bytes, ws;
  if (hfx_batch_desc_sizes(&shape, 3, kind, q_len, ctx, &host_bytes, &device_bytes, &ws)) return 1;
  char* host = (char*)aligned_alloc(4096, 1 << 20);
  char* dev = (char*)aligned_alloc(4096, 1 << 20);
  auto bytes = [&](const char* s) { return std::strcmp(s, "all") ? (size_t)std::atoi(s) : device_bytes; };
  const bool elsewhere = std::atoi(v[1]) == 9;          // pinned, but at another address on the GPU
  memory[0] = Memory{host, bytes(v[2]), elsewhere ? (int)hipMemoryTypeHost : std::atoi(v[1]), 0, elsewhere ? host + 4096 : host};
  memory[1] = Memory{dev, bytes(v[5]), std::atoi(v[3]), std::atoi(v[4]), dev};
  current = std::atoi(v[6]);
  stream_device = std::atoi(v[7]);
  pending = std::atoi(v[8]);
  fail_launch = std::atoi(v[9]);
  char* any = dev + (1 << 19);
  int32_t ids[2] = {2, 3};
  const std::string what = v[10];
  void* stream = (void*)(uintptr_t)std::atoi(v[11]);
  hfx_status st = 0;
  if (what == "build") st = hfx_build_batch_desc(&shape, 3, kind, q_len, ctx, indptr, pages, host, host_bytes, dev, device_bytes, stream);
  else hfx_fill_batch_desc(&shape, 3, kind, q_len, ctx, indptr, pages, host, host_bytes);
  if (what == "attention") st = hfx_mixed_paged_attention(&shape, any, any, host, dev, any, 1 << 18, any, stream);
  if (what == "static") st = hfx_mixed_paged_attention_static(&shape, any, any, host, dev, any, stream);
  if (what == "gather") st = hfx_gather_kv(&shape, any, host, dev, 0, any, any, stream);
  if (what == "gather unaligned") st = hfx_gather_kv(&shape, any, host, dev, 0, any + 2, any, stream);
  if (what == "append") st = hfx_append_kv(&shape, any, any, any, host, dev, stream);
  if (what == "pages") st = hfx_copy_pages(&shape, any, any + 4096, 8, 2, ids, ids, host, dev, 4096, stream);
  if (what == "shared pages") {                 // the list of source pages lies in the staging buffer, between what is written there
    int32_t* stage = (int32_t*)host;
    const int32_t to[3] = {50, 60, 70};
    for (int i = 0; i < 3; ++i) stage[1 + i] = 1 + i;
    page_list = true;
    st = hfx_copy_pages(&shape, any, any + 4096, 100, 3, stage + 1, to, host, dev, 4096, stream);
    for (int i = 0; i < 6; ++i) std::printf("%d/%d ", stage[i], launched[i]);
  }
  std::printf("%d %s pending %d\n", st, launches && copies ? "copy and kernel" : launches ? "kernel" : copies ? "copy" : "nothing", pending);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    if not os.path.exists(hb.LIB_PATH):
        from paper_2508_15919_amd import build
        build.build()
    d = tmp_path_factory.mktemp("upload")
    src, exe = d / "upload.cpp", d / "upload"
    src.write_text(PROGRAM)
    lib = os.path.dirname(hb.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe), "-L", lib, f"-l:{os.path.basename(hb.LIB_PATH)}", f"-Wl,-rpath,{lib}:/opt/rocm/lib",
                    "-Wl,--allow-shlib-undefined"], check=True)

    def call(host=1, host_bytes="all", dev=2, device=0, dev_bytes="all", current=0, stream=0, pending=0, fail=0, entry="build", handle=4096):
        args = [host, host_bytes, dev, device, dev_bytes, current, stream, pending, fail, entry, handle]
        return subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout.strip()
    return call


UNKNOWN, PINNED, DEVICE, MANAGED, PINNED_ELSEWHERE = 0, 1, 2, 3, 9


@pytest.mark.parametrize("what,route", [
    ({}, "kernel"), ({"device": 1, "current": 1, "stream": 1}, "kernel"),
    # staging memory that the GPU does not see, or not under this address, or not all of it
    ({"host": UNKNOWN}, "copy"), ({"host": MANAGED}, "copy"), ({"host": PINNED_ELSEWHERE}, "copy"), ({"host_bytes": 256}, "copy"),
    # a destination that is no device memory, too small a piece of it, or another GPU's than the stream's
    ({"dev": UNKNOWN}, "copy"), ({"dev": PINNED}, "copy"), ({"dev": MANAGED}, "copy"), ({"dev_bytes": 256}, "copy"),
    ({"device": 1}, "copy"), ({"stream": 1}, "copy"), ({"stream": 1, "device": 1}, "copy"), ({"current": 1}, "copy")])
def test_a_kernel_uploads_only_between_memory_it_may_touch(program, what, route):
    """Everything else is left to the runtime's copy, which takes it or refuses it: a kernel that is handed a wrong address faults the GPU."""
    assert program(**what) == f"0 {route} pending 0"


ENTRIES = ["build", "attention", "static", "gather", "gather unaligned", "append", "pages"]


@pytest.mark.parametrize("entry", ENTRIES)
def test_an_unread_error_of_an_earlier_call_is_left_alone(program, entry):
    """The thread's last error may be of any call before and unread (hipErrorInvalidDevice here): a call of the library that enqueues its work
    says so, and the error is there for whoever looks for it."""
    assert program(pending=101, entry=entry) == "0 kernel pending 101"


@pytest.mark.parametrize("entry", ENTRIES)
def test_a_failed_launch_is_reported(program, entry):
    assert program(fail=1, entry=entry) == f"{hb.HFX_ERR_DEVICE} nothing pending 0"


def test_an_unread_error_does_not_disturb_the_runtimes_copy(program):
    assert program(host=UNKNOWN, pending=101) == "0 copy pending 101"
    assert program(host=UNKNOWN, pending=101, entry="pages") == "0 copy and kernel pending 101"


@pytest.mark.parametrize("handle", [0, 1, 2])       # the default stream, hipStreamLegacy, hipStreamPerThread
@pytest.mark.parametrize("entry", ENTRIES)
def test_streams_that_are_named_and_not_made(program, handle, entry):
    assert program(handle=handle, entry=entry) == "0 kernel pending 0"


def test_page_ids_are_read_once(program):
    """Ids that change while they are put down (here by that itself) do not get past the check: 60 and 70 are pages of the destination alone."""
    assert program(entry="shared pages") == "1/1 50/50 2/2 60/60 3/3 70/70 0 kernel pending 0"
