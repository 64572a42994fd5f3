// Host program of test_first_use_threads.py: calls libbimamba.so with the HIP runtime's entry points replaced by the ones
// below (the executable's symbols come first in the lookup order), so no GPU is needed.  They model one rule of the real
// ones: a launch with more than 64 KB of dynamic LDS is refused until the kernel's limit has been raised.
//   race fwd|bwd   a second host thread makes its first call while the first one is inside the raising
//   fail fwd|bwd   the raising fails on the first call only
// Prints the two calls' return codes, the launches and the refused launches.
#include "bimamba.h"

#include <dlfcn.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>

struct dim3 {
    unsigned x, y, z;
};

static std::mutex g_lock;
static std::map<const void*, int> g_limit;
static std::atomic<int> g_raising{0}, g_launches{0}, g_refused{0}, g_failures_left{0};
static bool g_slow = false;
static thread_local struct {
    dim3 grid, block;
    size_t lds;
    void* stream;
} g_config;

extern "C" {
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipPeekAtLastError() { return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void* fn, int, int value)
{
    g_raising++;
    if (g_failures_left.fetch_sub(1) > 0) return 1;
    if (g_slow) std::this_thread::sleep_for(std::chrono::milliseconds(300));
    std::lock_guard<std::mutex> hold(g_lock);
    g_limit[fn] = value;
    return 0;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream)
{
    g_config = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream)
{
    *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void* fn, dim3, dim3, void**, size_t lds, void*)
{
    std::lock_guard<std::mutex> hold(g_lock);
    g_launches++;
    if (lds > 64 * 1024 && (!g_limit.count(fn) || (size_t)g_limit[fn] < lds)) {
        g_refused++;
        return 1;
    }
    return 0;
}
}

int main(int argc, char** argv)
{
    if (argc != 4) return 2;
    void* lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) {
        fprintf(stderr, "%s\n", dlerror());
        return 2;
    }
    auto fwd = (decltype(&bimamba_fwd))dlsym(lib, "bimamba_fwd");
    auto bwd = (decltype(&bimamba_bwd))dlsym(lib, "bimamba_bwd");
    const bool forward = !strcmp(argv[3], "fwd");
    // 256 tokens with activations per direction: 74 KB of B and C rows; the gradient walk takes 80 KB for 16 states
    bimamba_desc d{};
    d.struct_size = sizeof d;
    d.batch = 1; d.seqlen = 256; d.d_inner = 64; d.d_state = 16; d.n_heads = 64; d.n_groups = 1; d.d_conv = 4;
    d.io_dtype = BIMAMBA_BF16;
    uintptr_t next = 1 << 20;      // addresses that nothing reads
    auto place = [&] { return (void*)(next += 1 << 20); };
    auto view = [&](int64_t ch) { return bimamba_tensor{place(), 256 * ch, ch}; };
    auto inputs = [&] { return bimamba_inputs{view(64), view(64), view(64), view(16), view(16)}; };
    const bimamba_inputs f = inputs(), b = inputs();
    const bimamba_tensor out = view(64);
    const float* any = (const float*)place();
    const bimamba_params p{any, any, any, any, nullptr};
    const bimamba_input_grads gf{view(64), view(64), view(64), (float*)place(), (float*)place()};
    const bimamba_input_grads gb{view(64), view(64), view(64), (float*)place(), (float*)place()};
    const bimamba_param_grads qf{(float*)place(), nullptr, (float*)place(), (float*)place(), nullptr}, qb = qf;
    void* ws = place();
    auto call = [&] {
        return forward ? fwd(&d, &p, &p, &f, &b, &out, ws, (size_t)1 << 40, nullptr)
                       : bwd(&d, &p, &p, &f, &b, &out, &gf, &gb, &qf, &qb, ws, (size_t)1 << 40, nullptr);
    };
    int first = 0, second = 0;
    if (!strcmp(argv[2], "race")) {
        g_slow = true;
        std::thread t([&] { first = call(); });
        while (g_raising == 0) std::this_thread::yield();
        second = call();
        t.join();
    } else {
        g_failures_left = 1;
        first = call();
        second = call();
    }
    printf("%d %d %d %d\n", first, second, g_launches.load(), g_refused.load());
    return 0;
}
