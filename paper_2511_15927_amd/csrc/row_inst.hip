// Choice and launch of the one-row-per-chain form (row_kernels.h).
#include "row_kernels.h"
#include "launch.h"

namespace bm {

// The row form spends about twice the vector work of the sweep on a chain and token and wins where the sweep's two to four
// launches and its 100 instructions per dependent token are what a call waits for.  Measured against them (bf16,
// d_inner 4096 unless stated, us, sweep / row): 1 x 32 tokens 14.1 / 6.8, 4 x 32 14.9 / 13.7, 8 x 32 17.7 / 24.1; 2 x 64
// 18.8 / 12.5, 4 x 64 19.6 / 21.2; 1 x 128 26.6 / 16.9, 2 x 128 27.4 / 27.5; 1 x 256 49.6 / 38.2, d_inner 512 48.6 / 11.6.
// Against the sweep as pick_geometry plans it, 1000 calls inside the limits (4, 8 and 16 states, decays per state or per
// head, bf16 and fp32, which differ little), time of the row form over the sweep's, by chains (batch * d_inner):
//   beyond 12288 chains   65 tokens and more: 4 states 1.0 to 1.3, 8 states 0.9 to 1.0, 16 states 0.75 to 1.0: not taken with 4
//   129 to 192 tokens     with 4 / 8 / 16 states up to 4096 chains 0.65 / 0.56 / 0.51, beyond them 1.14 / 0.94 / 0.94: 4 states
//                         stop at 0.75 M channel tokens, the others at 1 M
//   193 to 256 tokens     up to 0.4 M channel tokens 0.56 / 0.48 / 0.50, the worst call 0.81; beyond (bf16, 16 states) 1 x 212
//                         tokens of 2688 channels 28.2 us / 32.6, 1 x 220 of 4112 37.1 / 56.4, 1 x 256 of 4096 34.6 / 37.8
// Up to 64 tokens the other side is short_kernel, one launch too, or two lanes per chain (other / row, us; 4, 16, 32 and 64 tokens, bf16):
//   16 states  12288 chains  8.4/8.7  9.9/9.6 14.1/11.6 22.0/17.3;  16384 chains  8.5/10.4 10.0/12.2 14.4/15.0
//   8 states    8192 chains  8.7/9.2  8.2/8.4 11.2/9.7  16.8/13.5;  12288 chains  9.1/9.6  9.3/10.0 11.3/11.5 16.9/17.3
//   4 states    8192 chains  8.3/8.4  8.4/8.8  9.7/9.4  14.4/13.3;  12288 chains  8.6/8.9  8.6/9.6   9.8/11.5 14.5/17.1
// From 25 tokens on (fewer states: 17) the row form stays ahead for longer where the directions are added up (24, 32, 40 and 48 tokens, per-state decays):
//   16 states, 16384 chains  added 14.9/14.8 17.4/15.4 22.0/18.3 21.5/18.7;  halves 14.7/17.4 17.8/18.6 18.6/23.0 21.3/23.8
//   8 states, 9000 chains    added 12.1/11.1 12.6/11.3 15.6/13.5 16.3/14.5;  halves 11.5/13.0 13.2/13.1 15.3/15.4 17.1/16.2
//   8 states, 12288 chains   added 12.0/11.9 12.3/12.1 15.2/14.5 16.1/14.7;  halves 11.1/13.5 13.1/13.7 15.0/16.3 16.8/17.0
// An arithmetic A is no faster than that on the other side, which takes its exponentials in these sizes too (8, 16, 24 and 32 tokens; halves
// read activations of their own): 16 states, 13312 chains, added 8.4/10.2 9.8/11.0 12.2/13.0, halves 8.3/11.4 10.0/13.0 12.5/15.3 15.3/15.8,
// 40 and 48 tokens 16.6/19.5 18.0/20.7; 8 states, 9216 chains, halves 7.6/8.4 7.6/10.2 9.3/11.6 11.0/11.9, 48 and 64 tokens 14.3/14.3 17.6/21.2.
constexpr long long kRowMaxChainsShort = 3LL << 12, kRowMaxChainsShortFew = 8192;   // up to 64 tokens: 16 states, fewer
constexpr long long kRowMaxChains = 16384, kRowMaxChainsFew = 3LL << 12, kRowMaxElements = 3LL << 18, kRowMaxElementsLong = 1LL << 20;
constexpr long long kRowMaxElementsLongest = 3LL << 17;
constexpr int kRowFewTokens = 24, kRowFewTokensFew = 16,   // 16 states, fewer
              kRowLongTokens = 128, kRowLongestTokens = 192;
constexpr size_t kRowLdsBytes = 160 * 1024;

bool row_reach(int batch, int seqlen, int d_inner)
{
    const long long chains = (long long)batch * d_inner;
    return chains <= kRowMaxChains && chains * seqlen <= kRowMaxElements;
}

bool row_form(int batch, int seqlen, int d_inner, int d_state, bool halves, RowForm* f)
{
    if (d_state > 16 || seqlen < 1 || seqlen > kRowMaxTokens) return false;
    const long long chains = (long long)batch * d_inner;
    const long long most = seqlen > kRowLongestTokens                 ? kRowMaxElementsLongest
                           : seqlen > kRowLongTokens && d_state >= 8 ? kRowMaxElementsLong
                                                                     : kRowMaxElements;
    const bool few = seqlen <= kShortCallTokens && (halves || d_state < 8 || seqlen <= (d_state < 16 ? kRowFewTokensFew : kRowFewTokens));
    const long long most_chains = few                                               ? (d_state < 16 ? kRowMaxChainsShortFew : kRowMaxChainsShort)
                                  : d_state < (seqlen <= kShortCallTokens ? 16 : 8) ? kRowMaxChainsFew
                                                                                    : kRowMaxChains;
    if (chains > most_chains || chains * seqlen > most) return false;
    const long long tiles = (long long)batch * ((d_inner + 3) / 4);
    const int groups = (seqlen + kRowTokens - 1) / kRowTokens;
    // Time segments of one and a half groups or more on average while that leaves the chip at most four waves per SIMD (a segment
    // walked twice costs 1.3 times the work, one of more than kRowHeld groups 1.6); then as many channel tiles beside each other as
    // keep every CU busy.  (Segments of two groups or more: 200 tokens of 512 channels 12.6 us against 10.5, 40 of 1024 6.6 / 5.6, 192 of
    // 256 9.4 / 8.2; of one or more: 32 tokens of 4096 7.1 against 6.1, 128 of 512 7.9 / 6.9.)
    int nseg = 1;
    while (nseg < kRowMaxWaves / 2 && groups >= 3 * nseg && tiles * 4 * nseg <= 16LL * cu_count()) nseg *= 2;
    f->seg_len = (groups + nseg - 1) / nseg * kRowTokens;
    f->nseg = (seqlen + f->seg_len - 1) / f->seg_len;
    f->tw = 1;
    auto fits = [&](int tw) { return RowLds(seqlen, 2, tw, f->nseg, f->seg_len).total * sizeof(float) <= kRowLdsBytes; };
    while (f->tw < 4 && 2 * f->nseg * f->tw * 2 <= kRowMaxWaves && tiles >= 2LL * f->tw * cu_count() && fits(2 * f->tw)) f->tw *= 2;
    return fits(f->tw);
}

// Segments that a wave's registers hold twice over are walked so: 256 tokens of 512 channels 10.7 us (every segment walked anew, fp32)
// -> 9.7, 128 of 2048 10.8 -> 9.7, 64 of 512 6.1 -> 5.75.  A kernel of its own: its 102 registers (against 75) leave a SIMD five waves
// at most, and calls of one segment bring up to eight.
static size_t lds_bytes(const RowArgs& a) { return (size_t)RowLds(a.L, a.same_bc ? 1 : 2, a.tw, a.nseg, a.seg_len).total * sizeof(float); }

template <typename IO, bool HELD>
static hipError_t launch_io(const RowArgs& a, int batch, hipStream_t st)
{
    static LdsLimit limit;
    auto kernel = row_kernel<IO, HELD>;
    const size_t lds = lds_bytes(a);
    if (lds > 64 * 1024) {
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(kernel), kRowLdsBytes);
        if (err != hipSuccess) return err;
    }
    const dim3 grid((unsigned)((a.Dn + 4 * a.tw - 1) / (4 * a.tw)), 1, (unsigned)batch);
    hipLaunchKernelGGL(kernel, grid, dim3((unsigned)(128 * a.nseg * a.tw)), lds, st, a);
    return hipSuccess;
}

hipError_t launch_row(int io_bf16, const RowArgs& a, int batch, hipStream_t st)
{
    if (a.nseg > 1 && a.seg_len <= kRowHeld * kRowTokens) return io_bf16 ? launch_io<IoBF16, true>(a, batch, st) : launch_io<IoF32, true>(a, batch, st);
    return io_bf16 ? launch_io<IoBF16, false>(a, batch, st) : launch_io<IoF32, false>(a, batch, st);
}

}  // namespace bm
