// The workspace memory (csrc/workspace.h) against a scripted HIP runtime: each
// call is recorded, and returns what the scenario says.  Prints, line by line,
// the calls made and the state reached.
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../paper_2607_24377_amd/csrc/workspace.h"

static std::vector<std::string> g_calls;
static std::map<std::string, hipError_t> g_result;  // of calls that fail
static hipError_t g_last = hipSuccess;              // the runtime's last error
static int g_live = 0;                              // allocations not freed

static hipError_t called(const char* name) {
    g_calls.push_back(name);
    const auto it = g_result.find(name);
    const hipError_t e = it == g_result.end() ? hipSuccess : it->second;
    if (e != hipSuccess) g_last = e;
    return e;
}

extern "C" {
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "scripted"; }
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) {
    *p = reinterpret_cast<hipMemPool_t>(0x10);
    return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void** p, size_t n, hipMemPool_t, hipStream_t) {
    const hipError_t e = called("alloc");
    *p = e == hipSuccess ? std::malloc(n) : nullptr;
    g_live += *p != nullptr;
    return e;
}
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s) { return hipMallocFromPoolAsync(p, n, nullptr, s); }
hipError_t hipFreeAsync(void* p, hipStream_t) {
    const hipError_t e = called("free");
    if (e == hipSuccess) {
        std::free(p);
        g_live--;
    }
    return e;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { return called("trim"); }
hipError_t hipStreamSynchronize(hipStream_t) { return called("wait"); }
hipError_t hipStreamQuery(hipStream_t) { return called("query"); }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = hipStreamCaptureStatusNone;
    return called("capturing");
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    static hipStreamCaptureMode mine = hipStreamCaptureModeGlobal;
    const hipStreamCaptureMode was = mine;
    mine = *m;
    *m = was;
    g_calls.push_back(mine == hipStreamCaptureModeRelaxed ? "relaxed" : "global");
    return hipSuccess;
}
}

static void report(const char* what, int status) {
    std::printf("%s status=%d kept=%zu live=%d last=%d detail=%d calls=", what, status, mxattn::g_kept[0].bytes, g_live,
                (int)g_last, mxattn::g_last_error[0] != 0);
    for (const std::string& c : g_calls) std::printf("%s,", c.c_str());
    std::printf("\n");
    g_calls.clear();
}

static void take(const char* what, size_t bytes) {
    mxattn::Workspace ws;
    int st = ws.take(bytes, nullptr);
    if (st == MXATTN_OK) {
        std::memset(ws.get(), 0, bytes);
        st = ws.give_back(MXATTN_OK);
    }
    report(what, st);
}

// workspace_host [call=error]...: a call of 3 MiB, then with the named calls
// failing one of 5 MiB (if "grow" is given) and a release; then without.
int main(int argc, char** argv) {
    take("first", (size_t)3 << 20);
    bool grow = false;
    for (int i = 1; i < argc; i++) {
        const char* eq = std::strchr(argv[i], '=');
        if (eq)
            g_result[std::string(argv[i], eq - argv[i])] = (hipError_t)std::atoi(eq + 1);
        else
            grow = true;
    }
    if (grow) take("grow", (size_t)5 << 20);
    report("release", mxattn::release_workspace());
    g_result.clear();
    g_last = hipSuccess;
    mxattn::g_last_error[0] = 0;
    take("again", (size_t)3 << 20);
    report("release", mxattn::release_workspace());
}
