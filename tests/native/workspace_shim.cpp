// The HIP calls that the workspace makes, on host memory with a limit, and the
// prompt attention's launches, which only note how they were called: linked
// with bellman_api.cpp for tests/test_workspace.py, so that an allocation that
// fails can be had without a GPU.
#include <stdlib.h>

#include "../../paper_2510_15330_amd/csrc/internal.h"

namespace {
size_t g_limit = 0, g_used = 0;      // bytes the device has, and has given
size_t g_asked[8];                   // sizes asked for since the last reset
int g_calls = 0;
int g_split = -1;                    // of the last prompt attention launched
}  // namespace

namespace bellman {
void launch_prefill_prep(const PrefillArgs&, hipStream_t) {}
void launch_prefill_attn(const PrefillArgs& a, hipStream_t) { g_split = a.split; }
int device_error_word(int, int32_t** p) {
    static int32_t word = 0;
    *p = &word;
    return 0;
}
}  // namespace bellman

extern "C" {

void ws_device(size_t limit) {
    g_limit = limit;
    g_used = 0;
    g_calls = 0;
}
int ws_calls(size_t* asked) {
    const int n = g_calls;
    for (int i = 0; i < n && i < 8; ++i) asked[i] = g_asked[i];
    g_calls = 0;
    return n;
}

int ws_split(void) {
    const int s = g_split;
    g_split = -1;
    return s;
}

hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
    if (g_calls < 8) g_asked[g_calls] = bytes;
    ++g_calls;
    if (g_used + bytes > g_limit) return hipErrorOutOfMemory;
    g_used += bytes;
    *p = malloc(1);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int* dev) {
    *dev = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* cs) {
    *cs = hipStreamCaptureStatusNone;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "out of memory"; }

}
