// Host program of test_first_use_threads.py: calls libbimamba.so with the HIP runtime's entry points replaced by the ones
// below (the executable's symbols come first in the lookup order), so no GPU is needed.  They model one rule of the real
// ones: a launch with more than 64 KB of dynamic LDS is refused until the kernel's limit has been raised.
//   race CALL     a second host thread makes its first call while the first one is inside the raising
//   fail CALL N   the N-th raising (from 1; 0: none) fails
// CALL: fwd, bwd, block (short calls of lane-per-chain kernels), m2 (chunked Mamba-2, several chunks), m2_block (one chunk), m2_far,
// m2_far_x (time parts, z and out, or x, with rows more than 2^24 elements apart).
// Prints the two calls' return codes, the launches, the refused launches and the launches of the first call ("fail" only).
#include "bimamba.h"

#include <dlfcn.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>

struct dim3 {
    unsigned x, y, z;
};

static std::mutex g_lock;
static std::map<const void*, int> g_limit;
static std::atomic<int> g_raising{0}, g_launches{0}, g_refused{0}, g_fails{0};
static bool g_slow = false;
static thread_local struct {
    dim3 grid, block;
    size_t lds;
    void* stream;
} g_config;

extern "C" {
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipFuncGetAttributes(void*, const void*) { return 1; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 3; return 0; }
int hipPeekAtLastError() { return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void* fn, int, int value)
{
    if (++g_raising == g_fails) return 1;
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
    if (argc < 4) return 2;
    void* lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) {
        fprintf(stderr, "%s\n", dlerror());
        return 2;
    }
    auto fwd = (decltype(&bimamba_fwd))dlsym(lib, "bimamba_fwd");
    auto bwd = (decltype(&bimamba_bwd))dlsym(lib, "bimamba_bwd");
    auto block = (decltype(&bimamba_block_fwd))dlsym(lib, "bimamba_block_fwd");
    auto is = [&](const char* call) { return !strcmp(argv[3], call); };
    // fwd, bwd: 256 tokens with activations per direction: 74 KB of B and C rows; the gradient walk takes 80 KB for 16 states
    bimamba_desc d{};
    d.struct_size = sizeof d;
    d.batch = 1; d.seqlen = 256; d.d_inner = 64; d.d_state = 16; d.n_heads = 64; d.n_groups = 1; d.d_conv = 4;
    d.io_dtype = BIMAMBA_BF16;
    if (is("block")) {   // 65 KB: four sets of B and C rows and what the directions leave for each other
        d.seqlen = 64; d.d_inner = d.n_heads = 128; d.n_groups = 2; d.state_split = 1;
    } else if (!strncmp(argv[3], "m2", 2)) {   // the preparation takes up to 118 KB, the walk of several chunks 115
        d.seqlen = is("m2") ? 128 : is("m2_block") ? 64 : 1030;
        d.d_inner = 128; d.n_heads = 2; d.d_state = 128;
        d.a_kind = BIMAMBA_A_SCALAR_PER_HEAD; d.d_kind = BIMAMBA_D_PER_HEAD; d.dt_softplus = d.conv_bc = 1;
    }
    uintptr_t next = 1 << 20;      // addresses that nothing reads
    auto place = [&] { return (void*)(next += 1 << 20); };
    auto view = [&](int64_t ch) { return bimamba_tensor{place(), d.seqlen * ch, ch}; };
    const int gn = d.n_groups * d.d_state;
    auto inputs = [&] { return bimamba_inputs{view(d.d_inner), view(d.d_inner), view(d.n_heads), view(gn), view(gn)}; };
    bimamba_inputs f = inputs(), b = inputs();
    bimamba_tensor out = view(d.d_inner);
    auto far = [&](bimamba_tensor& t) { t = bimamba_tensor{(void*)(next <<= 1), d.seqlen * ((int64_t)1 << 25), (1 << 24) + 2}; };
    if (is("m2_far")) {
        far(f.z);
        next = (uintptr_t)1 << 42;   // (an output may overlap no input)
        far(out);
    } else if (is("m2_far_x")) {
        far(f.x);
    }
    float* const state = (float*)place();
    void* const tail = place();
    const float* any = (const float*)place();
    const bimamba_params p{any, any, any, any, nullptr};
    const bimamba_input_grads gf{view(64), view(64), view(64), (float*)place(), (float*)place()};
    const bimamba_input_grads gb{view(64), view(64), view(64), (float*)place(), (float*)place()};
    const bimamba_param_grads qf{(float*)place(), nullptr, (float*)place(), (float*)place(), nullptr}, qb = qf;
    void* ws = place();
    auto call = [&] {
        if (is("fwd")) return fwd(&d, &p, &p, &f, &b, &out, ws, (size_t)1 << 40, nullptr);
        if (is("bwd")) return bwd(&d, &p, &p, &f, &b, &out, &gf, &gb, &qf, &qb, ws, (size_t)1 << 40, nullptr);
        return block(&d, &p, &p, &f, &b, state, tail, state, tail, &out, ws, (size_t)1 << 40, nullptr);   // commits in place
    };
    int first = 0, second = 0, of_first = 0;
    if (!strcmp(argv[2], "race")) {
        g_slow = true;
        std::thread t([&] { first = call(); });
        while (g_raising == 0) std::this_thread::yield();
        second = call();
        t.join();
    } else {
        g_fails = atoi(argv[4]);
        first = call();
        of_first = g_launches;
        second = call();
    }
    printf("%d %d %d %d %d\n", first, second, g_launches.load(), g_refused.load(), of_first);
    return 0;
}
