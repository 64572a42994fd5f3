// Host launchers of the gradient kernels (bwd_kernels.h), instantiated for the state counts the selective-scan layout
// uses with one lane per chain.
#include "bwd_kernels.h"
#include "launch.h"

#include <algorithm>

namespace bm {

bool bwd_supported(int d_state) { return d_state == 4 || d_state == 8 || d_state == 16; }

// Time segments of a gradient call and their length: the cheapest by two cost lines.  Workgroups take their segments in rounds of
// what the chip holds (the walk two per CU, the state pass four); a round takes a segment's tokens, plus 15 tokens' time for
// what a segment starts and ends with, and the last one, in which the CUs finish unevenly, a quarter of a round more.  Cutting a
// call at all adds the dh sums to the state pass, 0.3 of the walk's time a token.  Fitted on 44 calls of random size (1 to 32 x 128
// to 8192 tokens of 512 to 4096 channels, 8 and 16 states, bf16 and fp32), each timed with up to 14 numbers of segments: the choice
// costs 0.7 % more than the best one on average, 6 % at worst; a fixed eight waves per SIMD, at 32 tokens or more, 11 %.
// That number of segments is the least there are, though: every token rounds the dh it hands on, so dDelta's error grows over a segment
// (fp32, 4 x 2048 x 1024: 2.5e-7 against 64 bits with 32 tokens, 3.3e-7 with 64), and 3 % of the time, by the cost lines, buy its staying.
void bwd_segments(int d_inner, int batch, int seqlen, int* nseg, int* seg_len, int* seg_chunks)
{
    constexpr double kEnds = 15.0, kLastRound = 0.25, kDhSums = 0.3;
    constexpr int kMaxRounds = 16;                       // (the sums of a segment take workspace)
    constexpr int kLeastWavesPerSimd = 8, kLeastTokens = 32;
    const int all = seqlen > 0 ? (seqlen + kBwdChunk - 1) / kBwdChunk : 1;
    const long long tiles = (long long)((d_inner + 63) / 64), per_segment = (tiles + 1) / 2 * (batch > 0 ? batch : 1);
    const long long waves = 2 * tiles * (batch > 0 ? batch : 1);
    const long long fewest = std::clamp((4LL * cu_count() * kLeastWavesPerSimd + waves / 2) / waves, 1LL, std::max(1LL, (long long)seqlen / kLeastTokens));
    const int longest = (int)((all + fewest - 1) / fewest);   // chunks
    auto rounds = [&](long long workgroups, int per_cu) {
        const long long resident = (long long)per_cu * cu_count();
        return 2 * workgroups <= resident ? 1.0 : (double)((workgroups + resident - 1) / resident) + kLastRound;
    };
    auto cost = [&](long long n, int chunks) {
        const double tokens = chunks * kBwdChunk;
        if (n == 1) return rounds(per_segment, 2) * tokens;
        return rounds(n * per_segment, 2) * (tokens + kEnds) + kDhSums * rounds(n * per_segment, 4) * tokens;
    };
    int best = longest;
    double least = cost((all + longest - 1) / longest, longest);
    for (long long n = fewest + 1; 2 * n <= all && n <= 65535 && n * per_segment <= 2LL * kMaxRounds * cu_count(); n++) {
        const int chunks = (int)((all + n - 1) / n);
        if ((all + chunks - 1) / chunks != n) continue;   // as many segments of this length as a smaller n has
        if (const double c = cost(n, chunks); c < least) {
            least = c;
            best = chunks;
        }
    }
    *seg_chunks = best;
    *seg_len = best * kBwdChunk;
    *nseg = seqlen > 0 ? (seqlen + *seg_len - 1) / *seg_len : 1;
}

template <typename IO>
__global__ __launch_bounds__(256) void bwd_prep_kernel(const BwdPrepArgs a)
{
    using T = typename IO::T;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= a.per_set) return;
    const int set = blockIdx.y;
    const int n = (int)(idx % a.N);
    const int which = (int)(idx / a.N % 2);
    const long long r = idx / (2 * a.N);          // (batch, token, group)
    const int g = (int)(r % a.G), t = (int)(r / a.G % a.L), b = (int)(r / a.G / a.L);
    const TensorArg& src = which ? a.C[set] : a.B[set];
    a.dst[set][idx] = IO::ld((const T*)src.p + (size_t)b * src.sb + (long long)t * src.st + g * a.N + n);
}

void launch_bwd_prep(int io_bf16, const BwdPrepArgs& a, int sets, hipStream_t st)
{
    const dim3 grid((unsigned)((a.per_set + 255) / 256), (unsigned)sets);
    if (io_bf16) hipLaunchKernelGGL(bwd_prep_kernel<IoBF16>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(bwd_prep_kernel<IoF32>, grid, dim3(256), 0, st, a);
}

// src[0], src[step], ... added in order.  The sum is one chain but its addresses are not: sixteen values are requested at a
// time (the addition of one at a time waited out a memory round trip per two or three values).
__device__ __forceinline__ float sum_in_order(const float* src, long long step, int count)
{
    constexpr int kAhead = 16;
    float acc = 0.0f;
    for (int k0 = 0; k0 < count; k0 += kAhead) {
        float v[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; j++) v[j] = src[(long long)min(k0 + j, count - 1) * step];
#pragma unroll
        for (int j = 0; j < kAhead; j++) acc += k0 + j < count ? v[j] : 0.0f;
    }
    return acc;
}

__global__ __launch_bounds__(256) void bwd_sum_kernel(const BwdSumArgs a)
{
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    const int two_n = 2 * a.N;
    const long long per_set = a.rows * two_n;
    if (i < a.sets * per_set) {
        const int set = i >= per_set;
        i -= set * per_set;
        const long long r = i / two_n;
        const int v = (int)(i % two_n);
        const float* src = a.part[set] + r * a.slots * two_n + v;
        const float acc = sum_in_order(src, two_n, a.slots);
        (v % 2 ? a.dC : a.dB)[set][r * a.N + v / 2] = acc;
        return;
    }
    i -= a.sets * per_set;
    const int values = a.N + kBwdParams;
    if (i >= 2LL * values * a.Dn) return;
    const int ch = (int)(i % a.Dn), v = (int)(i / a.Dn % values), s = (int)(i / a.Dn / values);
    const float* src = a.param_part + ((size_t)s * a.segs * values + v) * a.pitch + ch;
    const float acc = sum_in_order(src, values * a.pitch, a.segs);
    if (v < a.N) a.dA[s][(size_t)ch * a.N + v] = acc;
    else if (v == a.N) a.dD[s][ch] = acc;
    else if (v < a.N + 5) {
        const int tap = v - a.N - 1 - (4 - a.K);      // rows are tap positions with w[3] on the current token
        if (tap >= 0) a.dconv_w[s][(size_t)ch * a.K + tap] = acc;
    } else if (v == a.N + 5) {
        if (a.dconv_b[s]) a.dconv_b[s][ch] = acc;
    } else if (a.ddt_bias[s]) a.ddt_bias[s][ch] = acc;
}

void launch_bwd_sum(const BwdSumArgs& a, hipStream_t st)
{
    const long long n = a.sets * a.rows * 2 * a.N + 2LL * (a.N + kBwdParams) * a.Dn;
    hipLaunchKernelGGL(bwd_sum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
}

template <int N, typename IO>
static hipError_t launch_walks(const BwdArgs& a, int batch, hipStream_t st)
{
    auto walk = bwd_kernel<N, IO>;
    if (kBwdLdsBytes<N> > 64 * 1024) {
        static LdsLimit limit;
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(walk), kBwdLdsBytes<N>);
        if (err != hipSuccess) return err;
    }
    const dim3 grid((unsigned)((a.tiles + 1) / 2), (unsigned)a.nseg, (unsigned)batch);
    hipLaunchKernelGGL((bwd_state_kernel<N, IO>), grid, dim3(256), 0, st, a);
    if (a.nseg > 1) {
        const long long threads = 2LL * batch * a.tiles * 64 * N;
        hipLaunchKernelGGL(bwd_carry_kernel<N>, dim3((unsigned)((threads + 255) / 256), 2), dim3(256), 0, st, a, batch);
    }
    hipLaunchKernelGGL(walk, grid, dim3(256), kBwdLdsBytes<N>, st, a);
    return hipSuccess;
}

hipError_t launch_bwd(int d_state, int io_bf16, const BwdArgs& a, int batch, hipStream_t st)
{
#define BM_BWD(n) \
    case n: return io_bf16 ? launch_walks<n, IoBF16>(a, batch, st) : launch_walks<n, IoF32>(a, batch, st);
    switch (d_state) {
        BM_BWD(4)
        BM_BWD(8)
        BM_BWD(16)
        default: return hipErrorInvalidValue;
    }
#undef BM_BWD
}

}  // namespace bm
