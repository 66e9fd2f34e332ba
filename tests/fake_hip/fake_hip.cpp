// A stand-in for the HIP runtime calls of the host code, for tests of what the
// library does with devices, streams and memory where no GPU is there: it has
// 8 devices, records the calls, launches nothing and copies nothing.  Loaded
// with RTLD_GLOBAL before the library, so that the library's references bind to
// it.  fake_fail() makes the next calls of one name return an error.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>

namespace {
using hipError = int;
using Handle = void *;
struct Dim3 {
    uint32_t x, y, z;
};
std::mutex mu;
std::string text;
std::map<std::string, std::pair<int, int>> fails;   // name -> (error, calls left)
thread_local int device = 0;
thread_local Dim3 cfg_grid, cfg_block;
thread_local size_t cfg_shm;
thread_local Handle cfg_stream;
int capturing = 0;
uintptr_t next_handle = 0x1000;

hipError called(const char *name, const std::string &args = "")
{
    std::lock_guard<std::mutex> lock(mu);
    text += std::string(name) + "@" + std::to_string(device) + (args.empty() ? "" : " " + args) + "\n";
    auto f = fails.find(name);
    if (f == fails.end() || f->second.second == 0) return 0;
    --f->second.second;
    return f->second.first;
}
hipError made(const char *name, Handle *out, const std::string &args = "")
{
    const hipError e = called(name, args);
    if (e == 0) *out = (Handle)(next_handle += 0x1000);
    return e;
}
// address space only: nothing reads or writes it
hipError allocated(const char *name, Handle *out, size_t bytes)
{
    const hipError e = called(name, std::to_string(bytes));
    if (e == 0) *out = (Handle)(next_handle += (bytes + 0xfff) / 0x1000 * 0x1000 + 0x1000);
    return e;
}
std::string hex(const void *p)
{
    char b[32];
    std::snprintf(b, sizeof(b), "%p", p);
    return b;
}
}  // namespace

extern "C" {
const char *fake_log() { return text.c_str(); }
void fake_clear() { text.clear(); }
void fake_fail(const char *name, int error, int calls) { fails[name] = {error, calls}; }
void fake_capturing(int on) { capturing = on; }

hipError __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shm, Handle s)
{
    cfg_grid = g;
    cfg_block = b;
    cfg_shm = shm;
    cfg_stream = s;
    return 0;
}
hipError __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *shm, Handle *s)
{
    *g = cfg_grid;
    *b = cfg_block;
    *shm = cfg_shm;
    *s = cfg_stream;
    return 0;
}
hipError hipLaunchKernel(const void *, Dim3 g, Dim3 b, void **, size_t shm, Handle)
{
    return called("hipLaunchKernel", std::to_string(g.x) + " " + std::to_string(b.x) + " " +
                                         std::to_string(shm));
}
hipError hipGetDevice(int *d)
{
    *d = device;
    return 0;
}
hipError hipSetDevice(int d)
{
    device = d;
    return called("hipSetDevice");
}
hipError hipDeviceSynchronize() { return called("hipDeviceSynchronize"); }
hipError hipGetLastError() { return 0; }
const char *hipGetErrorString(hipError) { return "fake"; }
hipError hipMalloc(Handle *p, size_t n) { return allocated("hipMalloc", p, n); }
hipError hipFree(Handle p) { return called("hipFree", hex(p)); }
hipError hipMallocAsync(Handle *p, size_t n, Handle) { return allocated("hipMallocAsync", p, n); }
hipError hipMallocFromPoolAsync(Handle *p, size_t n, Handle, Handle)
{
    return allocated("hipMallocFromPoolAsync", p, n);
}
hipError hipFreeAsync(Handle p, Handle) { return called("hipFreeAsync", hex(p)); }
hipError hipDeviceGetDefaultMemPool(Handle *p, int) { return made("hipDeviceGetDefaultMemPool", p); }
hipError hipMemPoolCreate(Handle *p, const void *) { return made("hipMemPoolCreate", p); }
hipError hipMemPoolSetAttribute(Handle, int, void *) { return called("hipMemPoolSetAttribute"); }
hipError hipMemPoolTrimTo(Handle, size_t n) { return called("hipMemPoolTrimTo", std::to_string(n)); }
hipError hipMemcpy(Handle, const void *, size_t, int) { return called("hipMemcpy"); }
hipError hipMemcpyAsync(Handle, const void *, size_t, int, Handle) { return called("hipMemcpyAsync"); }
hipError hipStreamCreateWithFlags(Handle *s, unsigned) { return made("hipStreamCreateWithFlags", s); }
hipError hipStreamSynchronize(Handle) { return called("hipStreamSynchronize"); }
hipError hipStreamWaitEvent(Handle, Handle, unsigned) { return called("hipStreamWaitEvent"); }
hipError hipStreamIsCapturing(Handle, int *st)
{
    *st = capturing;
    return called("hipStreamIsCapturing");
}
hipError hipEventCreate(Handle *e) { return made("hipEventCreate", e); }
hipError hipEventCreateWithFlags(Handle *e, unsigned) { return made("hipEventCreateWithFlags", e); }
hipError hipEventDestroy(Handle) { return called("hipEventDestroy"); }
hipError hipEventRecord(Handle, Handle) { return called("hipEventRecord"); }
hipError hipEventSynchronize(Handle) { return called("hipEventSynchronize"); }
}
