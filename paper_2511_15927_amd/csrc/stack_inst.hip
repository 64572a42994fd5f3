// Choice and launch of the one-launch form of a stack of layers (stack_kernels.h).
#include "stack_kernels.h"
#include "launch.h"

namespace bm {

// How many chains (batch * d_inner) and chain tokens a stack may have: beyond, the walk's vector work, twice the sweep's, costs
// more than the launches and first loads it saves.  A layer and step of 6 layers x 3 steps, us, in one launch / call by call (bf16):
//   16 states  32 tokens: 4096 chains 3.2 / 6.9, 16384 8.2 / 15.6, 32768 15.4 / 18.8, 45056 20.6 / 22.3, 65536 28.9 / 24.8;
//              16 tokens: 49152 15.0 / 17.2; 48: 32768 21.7 / 22.1; 64: 24576 20.6 / 25.0, 32768 26.7 / 25.4;
//              128: 4096 10.9 / 18.1, 12288 26.6 / 28.8, 16384 35.0 / 29.1
//    8 states  32 tokens: 24576 11.7 / 14.2, 32768 14.9 / 14.8; 16: 24576 7.9 / 9.3, 32768 10.3 / 9.6; 64: 24576 20.6 / 23.0
//    4 states  32 tokens: 20480 10.1 / 11.3, 24576 11.7 / 11.5; 16: 24576 7.9 / 8.0; 64: 16384 14.1 / 18.0
constexpr long long kStackMaxChains = 11LL << 12, kStackMaxChains8 = 6LL << 12, kStackMaxChains4 = 5LL << 12;
constexpr long long kStackMaxElements = 3LL << 19, kStackMaxElements4 = 1LL << 20;
constexpr size_t kStackLdsBytes = 160 * 1024;

bool stack_form(int batch, int seqlen, int d_inner, int d_state, RowForm* f)
{
    if (d_state > 16 || seqlen < 1 || seqlen > kRowMaxTokens) return false;
    const long long chains = (long long)batch * d_inner;
    if (chains > (d_state > 8 ? kStackMaxChains : d_state > 4 ? kStackMaxChains8 : kStackMaxChains4)) return false;
    if (chains * seqlen > (d_state > 4 ? kStackMaxElements : kStackMaxElements4)) return false;
    const long long tiles = (long long)batch * ((d_inner + 3) / 4);
    const int groups = (seqlen + kRowTokens - 1) / kRowTokens;
    int nseg = 1;   // segments and tiles as row_form takes them
    while (nseg < kRowMaxWaves / 2 && groups >= 4 * nseg && tiles * 4 * nseg <= 16LL * cu_count()) nseg *= 2;
    f->seg_len = (groups + nseg - 1) / nseg * kRowTokens;
    f->nseg = (seqlen + f->seg_len - 1) / f->seg_len;
    if (seqlen > 32 * kStackOutputs * f->nseg) return false;
    f->tw = 1;
    auto fits = [&](int tw) { return StackLds(seqlen, tw, f->nseg, f->seg_len).total * sizeof(float) <= kStackLdsBytes; };
    while (f->tw < 4 && 2 * f->nseg * f->tw * 2 <= kRowMaxWaves && tiles >= 2LL * f->tw * cu_count() && fits(2 * f->tw)) f->tw *= 2;
    return fits(f->tw);
}

template <typename IO, int OUTPUTS>
static hipError_t launch_outputs(const StackArgs& a, int batch, hipStream_t st)
{
    static LdsLimit limit;
    auto kernel = stack_kernel<IO, OUTPUTS>;
    const size_t lds = (size_t)StackLds(a.L, a.tw, a.nseg, a.seg_len).total * sizeof(float);
    if (lds > 64 * 1024) {
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(kernel), kStackLdsBytes);
        if (err != hipSuccess) return err;
    }
    const dim3 grid((unsigned)((a.Dn + 4 * a.tw - 1) / (4 * a.tw)), 1, (unsigned)batch);
    hipLaunchKernelGGL(kernel, grid, dim3((unsigned)(128 * a.nseg * a.tw)), lds, st, a);
    return hipSuccess;
}

template <typename IO>
static hipError_t launch_io(const StackArgs& a, int batch, hipStream_t st)
{
    const int outputs = (a.L + 32 * a.nseg - 1) / (32 * a.nseg);
    if (outputs <= 1) return launch_outputs<IO, 1>(a, batch, st);
    if (outputs <= 2) return launch_outputs<IO, 2>(a, batch, st);
    return launch_outputs<IO, 4>(a, batch, st);
}

hipError_t launch_stack(int io_bf16, const StackArgs& a, int batch, hipStream_t st)
{
    return io_bf16 ? launch_io<IoBF16>(a, batch, st) : launch_io<IoF32>(a, batch, st);
}

}  // namespace bm
