// Stands in for the HIP runtime under libwap.so where there is no GPU: every call the library makes on its launching paths is
// written down and answered with success, and nothing runs.  Loaded with RTLD_GLOBAL before the library, whose references then
// bind here.  Events count as complete as soon as they are recorded, or, after recorder_hold(1), never.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

namespace {
std::mutex mu;
std::vector<std::string> lines;
std::map<const void*, std::string> names;
std::map<const void*, int> limits;
std::set<const void*> recorded;
bool hold = false;
size_t handles = 0;
thread_local dim3 cfg_grid, cfg_block;
thread_local size_t cfg_smem;
thread_local hipStream_t cfg_stream;

void note(const char* fmt, const char* a, const void* b, long c, long d, long e = 0) {
    char line[1024];
    std::snprintf(line, sizeof line, fmt, a, b, c, d, e);
    lines.push_back(line);
}
void* handle() { return reinterpret_cast<void*>(0x1000 + 16 * ++handles); }
}  // namespace

extern "C" {
int recorder_count() { return (int)lines.size(); }
const char* recorder_line(int i) { return lines[i].c_str(); }
void recorder_hold(int on) { hold = on != 0; }

void** __hipRegisterFatBinary(const void*) {
    static void* module = nullptr;
    return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[fn] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t smem, hipStream_t st) {
    cfg_grid = grid; cfg_block = block; cfg_smem = smem; cfg_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* smem, hipStream_t* st) {
    *grid = cfg_grid; *block = cfg_block; *smem = cfg_smem; *st = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3, void**, size_t smem, hipStream_t st) {
    std::lock_guard<std::mutex> lock(mu);
    note("launch %s %p %ld %ld %ld", names[fn].c_str(), st, (long)smem, limits.count(fn) ? (long)limits[fn] : 65536L, (long)grid.x);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* fn, hipFuncAttribute, int value) {
    std::lock_guard<std::mutex> lock(mu);
    limits[fn] = value;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorder"; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = 0; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    std::lock_guard<std::mutex> lock(mu);
    *s = (hipStream_t)handle();
    note("stream %s%p %ld %ld", "", *s, 0, 0);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) {
    std::lock_guard<std::mutex> lock(mu);
    note("wait %s%p %ld %ld", "", s, 0, 0);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    std::lock_guard<std::mutex> lock(mu);
    *e = (hipEvent_t)handle();
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::mutex> lock(mu);
    recorded.insert(e);
    note("record %s%p %ld %ld", "", s, 0, 0);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    std::lock_guard<std::mutex> lock(mu);
    return hold && recorded.count(e) ? hipErrorNotReady : hipSuccess;
}
}
