// Choice and launch of the one-launch form of a stack of layers (stack_kernels.h).
#include "stack_quad.h"
#include "launch.h"

#include <algorithm>
#include <cmath>

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
    // tiles as row_form takes them; segments of two groups or more (of one and a half there, whose segments are held for the second walk)
    int nseg = 1;
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

// Steps side by side in the quad form, 0: the row form is the choice.  Clocks of a layer for all steps of a block, from what a SIMD's
// waves issue: alone on its SIMD a wave issues an instruction every seven clocks, several share the vector pipe at 4.6 a slot.
//   quad   34 / 22 / 16 slots a token and lane (16 / 8 / 4 states); a workgroup to a CU, side / 2 waves a SIMD (the
//          fullest one sets the pace of all at a layer's barriers); 2500 a layer
//   row    14.5 instructions, 11.3 slots; time segments walk their tokens 1.6 times; 1300 a layer, one step after the other
// Measured, us a layer and step, quad / row (bf16; layers feed each other):
//   16 states, 32 tokens, 8 steps   512 chains 1.19/1.92, 4096 1.21/2.34, 8192 2.50/3.35, 16384 5.28/6.92, 32768 10.4/13.2, 45056 15.1/19.4
//   4096 chains x 32, 1 / 2 / 3 / 4 steps   5.63/3.22  2.63/2.56  2.20/2.63  1.58/2.42
//   2 x 16 tokens of 2856, 3 steps 1.84/2.14
//   64 tokens    1640 chains, 3 steps 3.4/3.2, 4096 chains, 8 steps 2.89/5.09, 1024 chains, 4 steps 2.91/3.07, 16384 chains, 8 steps 12.0/12.1
//   128 tokens   1024 chains, 4 steps 8.88/3.88
//   8 states     4096 chains x 32, 8 steps 0.93/2.47, 24576 6.22/10.9, 2616 x 64, 4 steps 2.08/4.80
int stack_side_by_side(const StackArgs& a, int batch)
{
    const size_t bytes = (size_t)QuadLds(a.L, a.N).total * sizeof(float);
    const int most = (int)std::min<size_t>(kQuadMaxSteps, kStackLdsBytes / bytes);
    if (most < 1) return 0;
    const int rounds = (a.n_steps + most - 1) / most, side = (a.n_steps + rounds - 1) / rounds;
    const double cus = cu_count(), slots = a.N == 16 ? 34.0 : a.N == 8 ? 22.0 : 16.0;
    const double quads = std::ceil((double)((a.Dn + kQuadChannels - 1) / kQuadChannels) * batch / cus);
    const double quad = rounds * (a.L * slots * std::max(7.0, 4.6 * std::ceil(quads * side / 2)) + 2500.0);
    const double waves = (double)batch * ((a.Dn + 3) / 4) * 2 * a.nseg / (4 * cus);
    const double tokens = a.nseg > 1 ? 1.6 * a.seg_len : a.L;
    const double row = a.n_steps * (tokens * std::max(7.0 * 14.5, 4.6 * 11.3 * waves) + 1300.0);
    return quad < row ? side : 0;
}

template <typename IO, int N>
static hipError_t launch_quad(const StackArgs& a, int side, int batch, hipStream_t st)
{
    static LdsLimit limit;
    auto kernel = stack_quad_kernel<IO, N>;
    const size_t lds = (size_t)side * QuadLds(a.L, N).total * sizeof(float);
    if (lds > 64 * 1024) {
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(kernel), kStackLdsBytes);
        if (err != hipSuccess) return err;
    }
    const dim3 grid((unsigned)((a.Dn + kQuadChannels - 1) / kQuadChannels), 1, (unsigned)batch);
    hipLaunchKernelGGL(kernel, grid, dim3(128u * (unsigned)side), lds, st, a, side);
    return hipSuccess;
}

template <typename IO>
static hipError_t launch_quad_io(const StackArgs& a, int side, int batch, hipStream_t st)
{
    switch (a.N) {
        case 4: return launch_quad<IO, 4>(a, side, batch, st);
        case 8: return launch_quad<IO, 8>(a, side, batch, st);
        default: return launch_quad<IO, 16>(a, side, batch, st);
    }
}

// (steps side by side store their outputs in no order, and a layer's state and tail are replaced while they may still read those of a
// later layer: what shares memory goes one step after the other, so that the last one's values stay)
hipError_t launch_stack(int io_bf16, const StackArgs& a, int batch, bool apart, hipStream_t st)
{
    if (const int side = apart ? stack_side_by_side(a, batch) : 0; side > 0)
        return io_bf16 ? launch_quad_io<IoBF16>(a, side, batch, st) : launch_quad_io<IoF32>(a, side, batch, st);
    return io_bf16 ? launch_io<IoBF16>(a, batch, st) : launch_io<IoF32>(a, batch, st);
}

}  // namespace bm
