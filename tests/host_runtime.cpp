// A HIP runtime for tests of the library's host code where there is no GPU: device memory is host memory, a launch does nothing but
// count, streams keep no order.  It refuses what a caller can get wrong (a stream it does not know, a copy between device addresses that
// lie in no allocation) and, as the real one does, keeps the error of a refused call until it is asked for.
#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <iterator>
#include <map>
#include <mutex>
#include <thread>

namespace {
constexpr int kInvalidValue = 1, kInvalidHandle = 400, kNotFound = 500, kUnsupported = 801, kDeviceToDevice = 3;
struct Dim {
    uint32_t x, y, z;
};
std::mutex mu;
std::condition_variable launched;
std::map<uintptr_t, size_t> allocations;
std::map<uintptr_t, int64_t> streams;  // launches on each; the null stream is always there
uintptr_t next_handle = 0x1000;
thread_local int last_error = 0;
int64_t launches_of_other_threads = 0;
std::thread::id caller;
const void* awaited_src = nullptr;
int64_t awaited_launches = 0;
bool seen = false;

int result(int e)
{
    if (e) last_error = e;
    return e;
}
bool known(const void* p, size_t bytes)
{
    auto it = allocations.upper_bound((uintptr_t)p);
    if (it == allocations.begin()) return false;
    --it;
    return (uintptr_t)p + bytes <= it->first + it->second;
}
bool stream_ok(const void* s) { return !s || streams.count((uintptr_t)s); }
int launch(void* s)
{
    std::lock_guard<std::mutex> g(mu);
    if (!stream_ok(s)) return result(kInvalidHandle);
    ++streams[(uintptr_t)s];
    if (std::this_thread::get_id() != caller) {
        ++launches_of_other_threads;
        launched.notify_all();
    }
    return 0;
}
thread_local struct {
    Dim grid, block;
    size_t lds;
    void* stream;
} pushed;
}  // namespace

extern "C" {
// ---- what a test asks for
void host_runtime_caller() { caller = std::this_thread::get_id(); }
// The next copy from `src` waits until a thread other than the caller's has launched something (5 s at most).
void host_runtime_await_launch(const void* src)
{
    std::lock_guard<std::mutex> g(mu);
    awaited_src = src;
    awaited_launches = launches_of_other_threads;
    seen = false;
}
int host_runtime_saw_launch() { return seen; }
int64_t host_runtime_launches()  // of all streams
{
    std::lock_guard<std::mutex> g(mu);
    int64_t n = 0;
    for (auto& s : streams) n += s.second;
    return n;
}

// ---- the runtime
int hipMalloc(void** p, size_t bytes)
{
    std::lock_guard<std::mutex> g(mu);
    *p = calloc(1, bytes);
    allocations[(uintptr_t)*p] = bytes;
    return 0;
}
int hipFree(void* p)
{
    std::lock_guard<std::mutex> g(mu);
    allocations.erase((uintptr_t)p);
    free(p);
    return 0;
}
int hipMemGetAddressRange(void** base, size_t* size, void* p)
{
    std::lock_guard<std::mutex> g(mu);
    if (!known(p, 1)) return result(kNotFound);
    auto it = std::prev(allocations.upper_bound((uintptr_t)p));
    *base = (void*)it->first;
    *size = it->second;
    return 0;
}
int hipMemcpy(void* dst, const void* src, size_t bytes, int)
{
    memmove(dst, src, bytes);
    return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int kind, void* s)
{
    std::unique_lock<std::mutex> lk(mu);
    if (!stream_ok(s)) return result(kInvalidHandle);
    if (kind == kDeviceToDevice && !(known(dst, bytes) && known(src, bytes))) return result(kInvalidValue);
    if (src == awaited_src) {
        awaited_src = nullptr;
        seen = launched.wait_for(lk, std::chrono::seconds(5), [] { return launches_of_other_threads > awaited_launches; });
    }
    lk.unlock();
    memmove(dst, src, bytes);
    return 0;
}
int hipMemset(void* p, int v, size_t bytes)
{
    memset(p, v, bytes);
    return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned)
{
    std::lock_guard<std::mutex> g(mu);
    *s = (void*)(next_handle += 16);
    streams[(uintptr_t)*s] = 0;
    return 0;
}
int hipStreamDestroy(void* s)
{
    std::lock_guard<std::mutex> g(mu);
    return result(streams.erase((uintptr_t)s) ? 0 : kInvalidHandle);
}
int hipStreamSynchronize(void* s)
{
    std::lock_guard<std::mutex> g(mu);
    return result(stream_ok(s) ? 0 : kInvalidHandle);
}
int hipStreamWaitEvent(void* s, void*, unsigned) { return hipStreamSynchronize(s); }
int hipEventRecord(void*, void* s) { return hipStreamSynchronize(s); }
int hipEventCreateWithFlags(void** e, unsigned)
{
    std::lock_guard<std::mutex> g(mu);
    *e = (void*)(next_handle += 16);
    return 0;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*)
{
    *ms = 0.f;
    return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipGetDevice(int* d)
{
    *d = 0;
    return 0;
}
int hipSetDevice(int) { return 0; }
int hipGetLastError()
{
    const int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int e) { return e ? "refused" : "no error"; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void* s) { return launch(s); }
int hipExtLaunchKernel(const void*, Dim, Dim, void**, size_t, void* s, void*, void*, int) { return launch(s); }
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void* s)
{
    pushed = {grid, block, lds, s};
    return 0;
}
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* lds, void** s)
{
    *grid = pushed.grid;
    *block = pushed.block;
    *lds = pushed.lds;
    *s = pushed.stream;
    return 0;
}
void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
// not offered: graphs and module variables
int hipGetSymbolAddress(void**, const void*) { return result(kUnsupported); }
int hipGraphDestroy(void*) { return result(kUnsupported); }
int hipGraphExecDestroy(void*) { return result(kUnsupported); }
int hipGraphInstantiate(void**, void*, void*, char*, size_t) { return result(kUnsupported); }
int hipGraphLaunch(void*, void*) { return result(kUnsupported); }
int hipStreamBeginCapture(void*, int) { return result(kUnsupported); }
int hipStreamEndCapture(void*, void**) { return result(kUnsupported); }
}
