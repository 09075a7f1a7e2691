// Stands in for the HIP runtime under libsdnn (loaded ahead of it by tests/routes.py): launches are written to a log and
// nothing runs, so that what a call launches, copies or refuses can be checked on a machine without a GPU, at sizes that
// need no memory.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <cxxabi.h>
#include <hip/hip_runtime.h>

static std::string text;
static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m; // the library registers its kernels before this file's own statics are set up
    return m;
}

extern "C" {
const char *stub_log() { return text.c_str(); }
void stub_clear() { text.clear(); }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *)
{
    int status = 0;
    char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::string s = status == 0 ? plain : name;
    free(plain);
    if (s.compare(0, 5, "void ") == 0) s.erase(0, 5);
    names()[fn] = s.substr(0, s.find('('));
}
static struct { dim3 g, b; size_t lds; hipStream_t s; } call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { call = {g, b, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = call.g; *b = call.b; *lds = call.lds; *s = call.s;
    return hipSuccess;
}
static char arg[92]; // the start of the first argument of the last launch of an LDS forward
static char long_arg[80]; // the same for k_fwd_long: the whole argument
const char *stub_arg() { return arg; }
const char *stub_long_arg() { return long_arg; }
hipError_t hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **args, size_t lds, hipStream_t)
{
    // what the runtime refuses: 2^32 work items in a dimension, more LDS than a workgroup can have
    if ((unsigned long long)g.x * b.x >= 1ull << 32 || g.y > 65535 || g.z > 65535 || g.x == 0 || g.y == 0 || g.z == 0 || lds > 160 * 1024)
        return hipErrorInvalidConfiguration;
    if (names()[fn].compare(0, 9, "k_fwd_lds") == 0) memcpy(arg, args[0], sizeof arg);
    if (names()[fn].compare(0, 11, "k_fwd_long<") == 0) memcpy(long_arg, args[0], sizeof long_arg);
    char line[512];
    snprintf(line, sizeof line, "%s %u %u %u\n", names()[fn].c_str(), g.x, g.y, g.z);
    text += line;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *, const void *, size_t bytes, hipMemcpyKind, hipStream_t)
{
    text += "memcpy " + std::to_string(bytes) + "\n";
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
static int capture;
void stub_capture(int on) { capture = on; } // every stream is being captured
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
static int cus = 256;
void stub_cus(int n) { cus = n; } // nets that are created from now on
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { p->multiProcessorCount = cus; return hipSuccess; } // the header appends the version
const char *hipGetErrorString(hipError_t e) { return e == hipErrorInvalidConfiguration ? "invalid configuration" : "no error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = (void *)((size_t)1 << 44); return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 8; return hipSuccess; }
}
