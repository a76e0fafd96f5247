// The HIP runtime calls that libgcoo.so makes, for a process without a GPU: memory is host memory, a kernel launch and every call that
// waits or records is a line in a log, and the answers of calls that can fail are set by the test.  Loaded with global symbols before
// libgcoo.so (tests/host_calls.py), so that the library's host code can be run and its launches read.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <string>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Config { Dim3 grid, block; size_t shared; void* stream; };
thread_local Config t_config;
std::recursive_mutex g_mutex;
std::map<const void*, std::string> g_names;
std::map<const void*, void*> g_vars;
std::map<std::string, long long> g_settings;
std::string g_log;
void* g_told = nullptr;
std::string g_poke_in;                                       // see host_poke()
int32_t* g_poke_at = nullptr;
int32_t g_poke_value = 0;
int32_t g_starts[513];                                       // see host_starts()

long long setting(const char* key)
{
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    auto it = g_settings.find(key);
    return it == g_settings.end() ? 0 : it->second;
}
void say(const std::string& line)
{
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    g_log += line + "\n";
}
void poke(const char* call)
{
    if (g_poke_at && g_poke_in == call) { *g_poke_at = g_poke_value; g_poke_at = nullptr; }
}
}  // namespace

extern "C" {

// For the test: answers by name of the call (0 = success), "answer" = what a counting kernel tells the host, and the log.
void host_set(const char* key, long long value)
{
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    g_settings[key] = value;
}
// The next `call` (hipStreamIsCapturing or hipHostGetDevicePointer) stores `value` at `at`, as another thread of the program might.
void host_poke(const char* call, int32_t* at, int32_t value) { g_poke_in = call; g_poke_at = at; g_poke_value = value; }
const int32_t* host_starts() { return g_starts; }            // what the last order_groups_host was told about the groups
void* host_told() { return g_told; }                         // where the last counting kernel wrote its number
const char* host_log()
{
    static std::string copy;
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    copy.swap(g_log);
    g_log.clear();
    return copy.c_str();
}

void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    g_names[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int)
{
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    g_vars[var] = calloc(1, size);
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) { t_config = {grid, block, shared, stream}; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream)
{
    *grid = t_config.grid; *block = t_config.block; *shared = t_config.shared; *stream = t_config.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t shared, void*)
{
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    const std::string& name = g_names[f];
    say("launch " + name + " " + std::to_string(grid.x) + " " + std::to_string(block.x) + " " + std::to_string(shared));
    if (name.find("order_groups_host") != std::string::npos) memcpy(g_starts, args[1], sizeof g_starts);
    // the kernels that tell the host a number: the place of the pointer among their arguments
    int host = name.find("read_entry_count") != std::string::npos ? 2 : name.find("count_dense_total") != std::string::npos ? 6
             : name.find("count_dense_blocks") != std::string::npos ? 9 : -1;
    if (host >= 0) {
        unsigned long long* to = *static_cast<unsigned long long**>(args[host]);
        if (to) *to = (unsigned long long)setting("answer");
        g_told = to;
    }
    return 0;
}

int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { return (int)setting("hipGetLastError"); }
const char* hipGetErrorString(int) { return "set by the test"; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void* var)
{
    std::lock_guard<std::recursive_mutex> lock(g_mutex);
    *p = g_vars[var];
    return *p ? 0 : 1;
}
int hipHostMalloc(void** p, size_t bytes, unsigned flags) { *p = aligned_alloc(4096, (bytes + 4095) / 4096 * 4096); say("pinned " + std::to_string(flags)); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; poke("hipHostGetDevicePointer"); return 0; }
int hipMemcpyAsync(void* to, const void* from, size_t bytes, int, void*) { memcpy(to, from, bytes); say("copy"); return 0; }
int hipStreamSynchronize(void*) { say("wait stream"); return (int)setting("hipStreamSynchronize"); }
int hipDeviceSynchronize() { say("wait device"); return (int)setting("hipDeviceSynchronize"); }
int hipStreamIsCapturing(void*, int* status) { poke("hipStreamIsCapturing"); *status = (int)setting("capturing"); return (int)setting("hipStreamIsCapturing"); }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { say("record"); return (int)setting("hipEventRecord"); }
int hipEventQuery(void*) { return (int)setting("hipEventQuery"); }
int hipEventSynchronize(void*) { say("wait event"); return (int)setting("hipEventSynchronize"); }

}  // extern "C"
