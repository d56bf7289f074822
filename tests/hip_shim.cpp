// Stands between the library and the HIP runtime in a child process of the allocation tests
// (tests/alloc_child.py): counts the calls that allocate and refuses device blocks above
// limits, as a device without that much free memory does.  Loaded with RTLD_GLOBAL before
// anything that uses the runtime, so that its names are found first.
#include <dlfcn.h>
#include <link.h>

#include <atomic>
#include <cstddef>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

namespace {

std::atomic<long> g_calls[4];  // hipMalloc, hipHostMalloc, hipEventCreateWithFlags, refused
std::atomic<size_t> g_limit{~(size_t)0}, g_total{~(size_t)0};
std::mutex g_mu;
std::map<void *, size_t> g_live;
size_t g_bytes = 0, g_peak = 0;

void *runtime() {
    static void *h = [] {
        std::string path;
        dl_iterate_phdr(
            [](dl_phdr_info *i, size_t, void *out) {
                if (!std::strstr(i->dlpi_name, "libamdhip64")) return 0;
                *static_cast<std::string *>(out) = i->dlpi_name;
                return 1;
            },
            &path);
        return dlopen(path.c_str(), RTLD_LAZY | RTLD_NOLOAD);
    }();
    return h;
}

template <typename F>
F real(const char *name) {
    return reinterpret_cast<F>(dlsym(runtime(), name));
}

}  // namespace

extern "C" {

int hipMalloc(void **p, size_t bytes) {
    static auto f = real<int (*)(void **, size_t)>("hipMalloc");
    g_calls[0]++;
    bool full;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        full = bytes > g_limit || bytes > g_total - (g_bytes < g_total ? g_bytes : g_total.load());
    }
    if (full) {
        g_calls[3]++;
        return 2;  // hipErrorOutOfMemory
    }
    const int e = f(p, bytes);
    if (e == 0) {
        std::lock_guard<std::mutex> lk(g_mu);
        g_live[*p] = bytes;
        g_bytes += bytes;
        g_peak = g_bytes > g_peak ? g_bytes : g_peak;
    }
    return e;
}

int hipFree(void *p) {
    static auto f = real<int (*)(void *)>("hipFree");
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_live.find(p);
        if (it != g_live.end()) {
            g_bytes -= it->second;
            g_live.erase(it);
        }
    }
    return f(p);
}

int hipHostMalloc(void **p, size_t bytes, unsigned flags) {
    static auto f = real<int (*)(void **, size_t, unsigned)>("hipHostMalloc");
    g_calls[1]++;
    return f(p, bytes, flags);
}

int hipEventCreateWithFlags(void **e, unsigned flags) {
    static auto f = real<int (*)(void **, unsigned)>("hipEventCreateWithFlags");
    g_calls[2]++;
    return f(e, flags);
}

void shim_limit(size_t bytes) { g_limit = bytes; }    // of one block
void shim_total(size_t bytes) { g_total = bytes; }    // of all blocks
long shim_calls(int k) { return g_calls[k]; }
size_t shim_live(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_bytes;
}
size_t shim_peak(int reset) {
    std::lock_guard<std::mutex> lk(g_mu);
    const size_t v = g_peak;
    if (reset) g_peak = g_bytes;
    return v;
}
}
