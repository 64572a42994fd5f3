// Short calls with few chains: one row of 16 lanes per chain (up to 16 states), the whole call in one launch.
//
// What bounds such a call (a denoising step of a block at batch 1, a toy model) is not arithmetic but the chain of
// dependent tokens and the launches around it.  With one lane per state a token costs a lane an exponential and four
// operations, and a wave's four chains (a row of 16 lanes each) give a call 16 times the waves of one lane per chain.
// The lanes of a row also deal the tokens among themselves, sixteen at a time: lane n of a chain loads token n of a
// group, evaluates its conv, SiLU and softplus and forms u = Delta xc; the recurrence then takes a token's Delta and u
// out of that lane's registers through the row-broadcast operand, and the products C h of sixteen tokens are summed over the
// row by one reduce-scatter, which leaves token n's output in lane n.  That is about 13 vector instructions per wave and
// token for 4 chains, twice what the sweep spends per chain: the host takes this form while latency is what counts
// (row_form in row_inst.hip).
//
// A workgroup holds both directions of 4 tw adjacent channels over the whole sequence, cut into nseg time segments: waves
// (direction, segment, tile).  With several segments each wave first finds its segment's end state from a zero state,
// leaves it in LDS with the segment's Delta sum, folds those of the segments before it and then walks again from there.  B
// and C rows go to LDS as fp32 once (no preparation launch), the ungated outputs of both directions meet in LDS, and the
// gate, the combine and the rounding are done by the whole workgroup with the channels across the lanes.  The commit of
// the conv tail is part of the launch too.
#pragma once
#include "kernels.h"

namespace bm {

struct RowArgs {
    DirArgs dir[2];
    void* out;
    long long out_sb, out_st;
    const float* h_in;    // [batch][Dn][N] or null
    float* h_out;         // or null
    const void* tail_in;  // io dtype [batch][K-1][Dn] or null
    void* tail_out;       // or null
    int L, Dn, P, HG, G, N, K;
    int dt_softplus, d_per_head, a_scalar, separate;
    int same_z, same_bc;  // both directions gate with the same z; read the same B and C
    int tw, tw_log2, nseg, seg_len;   // channel tiles of 4 (a power of two) and time segments of a workgroup; seg_len a multiple of 16
};

constexpr int kRowTokens = 16;      // tokens of a group: one per lane of a row
constexpr int kRowMaxTokens = 256;  // of a call
constexpr int kRowMaxWaves = 16;

// LDS of a workgroup, in floats: B|C rows, outputs, per-wave (u, Delta, D xc) of its tokens, segment summaries.
struct RowLds {
    int bc, y, ud, sum, total;
    __host__ __device__ RowLds(int L, int sets, int tw, int nseg, int seg_len)
    {
        const int waves = 2 * nseg * tw;
        bc = 0;
        y = bc + sets * (L + 2 * kRowTokens) * 32;      // (a row of spare tokens at either end, see the walk)
        ud = y + 2 * L * tw * 4;
        sum = ud + waves * (seg_len / kRowTokens) * 64 * 3;
        total = sum + waves * 64 * 2;
    }
};

// The value lane I of the caller's row of 16 holds.
template <int I>
__device__ __forceinline__ float row_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + I, 0xF, 0xF, true));
}
// The value k lanes back in the row, or, in the row's first k lanes, that of `before` (the previous group) 16 - k lanes on.
template <int K>
__device__ __forceinline__ float row_back(float v, float before)
{
    const int w = __builtin_amdgcn_update_dpp(0, __float_as_int(before), 0x120 + K, 0xF, 0xF, true);     // row_ror:K
    return __int_as_float(__builtin_amdgcn_update_dpp(w, __float_as_int(v), 0x110 + K, 0xF, 0xF, false));  // row_shr:K
}
template <int CTRL>
__device__ __forceinline__ float row_perm(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_total(float v)
{
    v += row_perm<0xB1>(v);
    v += row_perm<0x4E>(v);
    v += row_perm<0x141>(v);
    v += row_perm<0x128>(v);
    return v;
}
// p[i] summed over the row; lane n returns the total of p[n].  Every step halves the values a lane carries; both partners
// form both sums, and where the lane bit names whole groups of four lanes the second one is written under a bank mask.
__device__ __forceinline__ float row_reduce_scatter(float (&p)[16], int n)
{
#pragma unroll
    for (int i = 0; i < 8; i += 4) {
        asm("s_nop 1\n\t"
            "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %3, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc"
            : "+v"(p[i]), "+v"(p[i + 1]), "+v"(p[i + 2]), "+v"(p[i + 3])
            : "v"(p[i + 8]), "v"(p[i + 9]), "v"(p[i + 10]), "v"(p[i + 11]));
    }
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %2, %6, %6 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %3, %7, %7 row_half_mirror row_mask:0xf bank_mask:0xa"
        : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]) : "v"(p[4]), "v"(p[5]), "v"(p[6]), "v"(p[7]));
    // (every lane forms both sums before it selects: inside a branch a permuted operand would read disabled lanes)
#pragma unroll
    for (int i = 0; i < 4; i++) p[i] += row_perm<0x4E>(p[i]);
    const bool b1 = (n & 2) != 0, b0 = (n & 1) != 0;
    float q0 = b1 ? p[2] : p[0], q1 = b1 ? p[3] : p[1];
    q0 += row_perm<0xB1>(q0);
    q1 += row_perm<0xB1>(q1);
    return b0 ? q1 : q0;
}

// f(integral_constant<int, i>) for the sixteen tokens of a group.
template <typename F>
__device__ __forceinline__ void for_each_row_token(F&& f)
{
    f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{}); f(std::integral_constant<int, 2>{}); f(std::integral_constant<int, 3>{});
    f(std::integral_constant<int, 4>{}); f(std::integral_constant<int, 5>{}); f(std::integral_constant<int, 6>{}); f(std::integral_constant<int, 7>{});
    f(std::integral_constant<int, 8>{}); f(std::integral_constant<int, 9>{}); f(std::integral_constant<int, 10>{}); f(std::integral_constant<int, 11>{});
    f(std::integral_constant<int, 12>{}); f(std::integral_constant<int, 13>{}); f(std::integral_constant<int, 14>{}); f(std::integral_constant<int, 15>{});
}

// The recurrence of a wave's four chains over `groups` groups of sixteen tokens, from state h: (u, Delta, D xc) of the tokens from
// `ud` (STRIDE floats a group), B|C rows of the call from `bc` (in token order: a group's are sixteen constant offsets from its
// lowest-address one).  sink(j, y) takes the output of scan position j + n.
template <bool OUTPUT, int DIR, int STRIDE, typename Sink>
__device__ __forceinline__ void row_walk(float& h, float a2, const float* ud, const float2* bc, int groups, int j0, int last, int lane, int n,
                                         Sink&& sink)
{
    for (int g = 0; g < groups; g++) {
        const float u = ud[g * STRIDE + lane], delta = ud[g * STRIDE + 64 + lane];
        float p[16];
        const int j = j0 + g * kRowTokens;
        const float2* const rows = bc + (DIR > 0 ? j : last - j - (kRowTokens - 1)) * 16;
        auto token = [&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const float2 row = rows[(DIR > 0 ? i : kRowTokens - 1 - i) * 16];
            const float an = fast_exp2(row_lane<i>(delta) * a2);
            h = fmaf(an, h, row_lane<i>(u) * row.x);
            if (OUTPUT) p[i] = row.y * h;
        };
        for_each_row_token(token);
        if constexpr (OUTPUT) sink(j, row_reduce_scatter(p, n) + ud[g * STRIDE + 128 + lane]);
    }
}

// A segment of up to kRowHeld groups walked twice: the first time from a zero state for its end state, keeping every token's decay
// and input, which the second time, from the state entering it, takes an exponential, two products and half of the reads less.
constexpr int kRowHeld = 2;
struct RowSteps {
    float an[kRowHeld][16], ub[kRowHeld][16];
};
template <int DIR>
__device__ __forceinline__ void row_steps(float& h, RowSteps& st, float a2, const float* ud, const float2* bc, int groups, int j0, int last, int lane)
{
#pragma unroll
    for (int g = 0; g < kRowHeld; g++) {
        if (g < groups) {
            const float u = ud[g * 192 + lane], delta = ud[g * 192 + 64 + lane];
            const int j = j0 + g * kRowTokens;
            const float2* const rows = bc + (DIR > 0 ? j : last - j - (kRowTokens - 1)) * 16;
            auto token = [&](auto ic) {
                constexpr int i = decltype(ic)::value;
                st.an[g][i] = fast_exp2(row_lane<i>(delta) * a2);
                st.ub[g][i] = row_lane<i>(u) * rows[(DIR > 0 ? i : kRowTokens - 1 - i) * 16].x;
                h = fmaf(st.an[g][i], h, st.ub[g][i]);
            };
            for_each_row_token(token);
        }
    }
}
template <int DIR, typename Sink>
__device__ __forceinline__ void row_walk_held(float& h, const RowSteps& st, const float* ud, const float2* bc, int groups, int j0, int last, int lane,
                                              int n, Sink&& sink)
{
#pragma unroll
    for (int g = 0; g < kRowHeld; g++) {
        if (g < groups) {
            float p[16];
            const int j = j0 + g * kRowTokens;
            const float2* const rows = bc + (DIR > 0 ? j : last - j - (kRowTokens - 1)) * 16;
#pragma unroll
            for (int i = 0; i < 16; i++) {
                h = fmaf(st.an[g][i], h, st.ub[g][i]);
                p[i] = rows[(DIR > 0 ? i : kRowTokens - 1 - i) * 16].y * h;
            }
            sink(j, row_reduce_scatter(p, n) + ud[g * 192 + 128 + lane]);
        }
    }
}

// grid (ceil(Dn / (4 tw)), 1, batch), block 128 * nseg * tw, dynamic LDS RowLds::total floats.
template <typename IO, bool HELD>
__global__ __launch_bounds__(64 * kRowMaxWaves, 1) void row_kernel(const RowArgs a)
{
    using T = typename IO::T;
    extern __shared__ __attribute__((aligned(16))) float row_lds[];
    const RowLds lds(a.L, a.same_bc ? 1 : 2, a.tw, a.nseg, a.seg_len);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = 2 * a.nseg * a.tw, threads = 64 * waves;
    const int s = wave & 1;
    const int tile = __builtin_amdgcn_readfirstlane((wave >> 1) / a.nseg), seg = (wave >> 1) - tile * a.nseg;   // seg: scan order
    const int b = blockIdx.z, n = lane & 15, shift = a.tw_log2 + 2, width = 1 << shift;   // channels of the workgroup
    const int ch0 = blockIdx.x * width;
    const int ch_of = ch0 + tile * 4 + (lane >> 4);
    const bool valid = ch_of < a.Dn;
    // (integer divisions by run-time values cost some thirty instructions: taken only where there is something to divide)
    const int ch = min(ch_of, a.Dn - 1), head = a.P == 1 ? ch : ch / a.P;
    const int grp = a.G == 1 ? 0 : __builtin_amdgcn_readfirstlane(ch0 / a.P / a.HG);   // a workgroup never straddles two B/C groups
    const int last = a.L - 1;
    const DirArgs& da = a.dir[s];
    auto token_of = [&](int j) { return s == 0 ? j : last - j; };

    // this wave's tokens, requested first: group g, lane n is scan position j0 + 16 g + n
    const int j0 = seg * a.seg_len, j1 = min(a.L, j0 + a.seg_len), groups = max(0, (j1 - j0 + kRowTokens - 1) / kRowTokens);
    const T* xb = (const T*)da.x.p + (size_t)b * da.x.sb + ch;
    const T* db = (const T*)da.dt.p + (size_t)b * da.dt.sb + head;
    auto place = [&](int j) { return (long long)token_of(min(max(j, 0), last)); };
    T x_next = xb[place(j0 + n) * da.x.st], d_next = db[place(j0 + n) * da.dt.st];
    // raw x of the 16 positions before the segment (the last three count): sequence, cached tail or zero
    float before = 0.0f;
    {
        const int j = j0 - kRowTokens + n;
        const T from_seq = xb[place(j) * da.x.st];
        T from_tail = 0;
        const bool tail = s == 0 && a.tail_in != nullptr && a.K > 1 && j0 == 0;
        if (tail) from_tail = ((const T*)a.tail_in)[((size_t)b * (a.K - 1) + max(a.K - 1 + j, 0)) * a.Dn + ch];
        if (j >= 0) before = IO::cvt(from_seq);
        else if (tail && j >= -(a.K - 1)) before = IO::cvt(from_tail);
    }
    float w4[4];
    load_taps(da.conv_w + (size_t)ch * a.K, a.K, w4);
    const float cb = da.conv_b ? da.conv_b[ch] : 0.0f;
    const float dval = da.D[a.d_per_head ? head : ch];
    const float dtb = (a.dt_softplus && da.dt_bias) ? da.dt_bias[head] : 0.0f;
    const bool state = n < a.N;                          // lanes past the last state carry zeros
    const float a2 = state ? da.A[a.a_scalar ? (size_t)head : (size_t)head * a.N + n] * kLog2e : 0.0f;
    float h = 0.0f;
    const bool from_h_in = s == 0 && a.h_in != nullptr;
    const size_t h_at = ((size_t)b * a.Dn + ch) * a.N + n;
    if (from_h_in && state) h = a.h_in[h_at];

    // z of this thread's first outputs (see the end), long before they are needed
    constexpr int kZAhead = 2;
    T z_ahead[2][kZAhead];
    auto z_of = [&](int d, int t, int chan) {
        const TensorArg& z = a.dir[d].z;
        return ((const T*)z.p + (size_t)b * z.sb)[(long long)t * z.st + chan];
    };
#pragma unroll
    for (int k = 0; k < kZAhead; k++) {
        const int i = min(tid + k * threads, a.L * width - 1), t = i >> shift, chan = min(ch0 + (i & (width - 1)), a.Dn - 1);
        z_ahead[0][k] = z_of(0, t, chan);
        if (!a.same_z) z_ahead[1][k] = z_of(1, t, chan);
    }

    // B|C rows as fp32: [set][token][n][2]; a thread keeps its column and has eight tokens in flight at a time.  A group of
    // tokens may reach past either end of the call: sixteen rows of zeros there.
    const int set_rows = a.L + 2 * kRowTokens;
    {
        constexpr int kFlight = 8;
        const int m = tid & 15, which = (tid >> 4) & 1, step = threads >> 5;
        for (int set = 0; set < (a.same_bc ? 1 : 2); set++) {
            const TensorArg& src = which ? a.dir[set].Craw : a.dir[set].Braw;
            const T* const col = (const T*)src.p + (size_t)b * src.sb + grp * a.N + min(m, a.N - 1);
            float* const dst = row_lds + lds.bc + ((set * set_rows + kRowTokens) * 16 + m) * 2 + which;
            for (int t0 = tid >> 5; t0 < a.L; t0 += kFlight * step) {
                T v[kFlight];
#pragma unroll
                for (int k = 0; k < kFlight; k++) v[k] = col[(long long)min(t0 + k * step, last) * src.st];
#pragma unroll
                for (int k = 0; k < kFlight; k++)
                    if (t0 + k * step < a.L) dst[(t0 + k * step) * 32] = m < a.N ? IO::cvt(v[k]) : 0.0f;
            }
            if (a.L % kRowTokens != 0)
                for (int t = tid >> 5; t < kRowTokens; t += step) dst[(t - kRowTokens) * 32] = dst[(a.L + t) * 32] = 0.0f;
        }
    }

    // per-token work of this lane's tokens
    float* const ud = row_lds + lds.ud + wave * (a.seg_len / kRowTokens) * 192;
    float dsum = 0.0f;
    for (int g = 0; g < groups; g++) {
        const int j = j0 + g * kRowTokens + n;
        const bool there = j < j1;
        const float x0 = there ? IO::cvt(x_next) : 0.0f;
        float delta = IO::cvt(d_next);
        x_next = xb[place(j + kRowTokens) * da.x.st];
        d_next = db[place(j + kRowTokens) * da.dt.st];
        float pre = fmaf(w4[3], x0, cb);
        pre = fmaf(w4[2], row_back<1>(x0, before), pre);
        pre = fmaf(w4[1], row_back<2>(x0, before), pre);
        pre = fmaf(w4[0], row_back<3>(x0, before), pre);
        before = x0;
        const float xc = silu(pre);
        if (a.dt_softplus) delta = softplus(delta + dtb);
        if (!there) delta = 0.0f;                        // a token that does not exist leaves the state as it is
        dsum += delta;
        ud[g * 192 + lane] = delta * xc;
        ud[g * 192 + 64 + lane] = delta;
        ud[g * 192 + 128 + lane] = dval * xc;
    }
    asm volatile("" : "+v"(h));                          // (h_in has arrived before any wave can reach its store to an aliased h_out)
    __syncthreads();                                     // B|C rows

    // the recurrence over the segment
    const float2* const bc = reinterpret_cast<const float2*>(row_lds + lds.bc) + ((a.same_bc ? 0 : s) * set_rows + kRowTokens) * 16 + n;
    auto leave = [&](int j, float y) {
        if (j + n < j1) row_lds[lds.y + (s * a.L + token_of(j + n)) * width + tile * 4 + (lane >> 4)] = y;
    };
    auto walk = [&](auto with_output, auto direction) {
        constexpr bool kOutput = decltype(with_output)::value;
        constexpr int kDir = decltype(direction)::value;
        row_walk<kOutput, kDir, 192>(h, a2, ud, bc, groups, j0, last, lane, n, leave);
    };
    using Up = std::integral_constant<int, 1>;
    using Down = std::integral_constant<int, -1>;
    auto fold = [&](float h0) {                          // the state entering the segment, from the end states before it
        row_lds[lds.sum + wave * 128 + lane] = h;
        row_lds[lds.sum + wave * 128 + 64 + lane] = row_total(dsum);
        __syncthreads();
        h = h0;
        for (int e = 0; e < seg; e++) {
            const float* from = row_lds + lds.sum + (((tile * a.nseg + e) << 1) + s) * 128 + lane;
            h = fmaf(fast_exp2(from[64] * a2), h, from[0]);
        }
    };
    const float h0 = h;
    if constexpr (HELD) {
        RowSteps st;
        h = 0.0f;
        if (s == 0) row_steps<1>(h, st, a2, ud, bc, groups, j0, last, lane);
        else row_steps<-1>(h, st, a2, ud, bc, groups, j0, last, lane);
        fold(h0);
        if (s == 0) row_walk_held<1>(h, st, ud, bc, groups, j0, last, lane, n, leave);
        else row_walk_held<-1>(h, st, ud, bc, groups, j0, last, lane, n, leave);
    } else {
        if (a.nseg > 1) {
            h = 0.0f;
            if (seg + 1 < a.nseg) {                      // (nothing starts from the scan-last segment's end)
                if (s == 0) walk(std::false_type{}, Up{});
                else walk(std::false_type{}, Down{});
            }
            fold(h0);
        }
        if (s == 0) walk(std::true_type{}, Up{});
        else walk(std::true_type{}, Down{});
    }
    if (s == 0 && a.h_out && valid && state && j1 == a.L && j1 > j0) a.h_out[h_at] = h;
    __syncthreads();                                     // both directions' outputs

    // gate, combine, round: channels across the lanes
    auto finish = [&](int i, T zf_raw, T zb_raw) {
        const int t = i >> shift, c = i & (width - 1), chan = ch0 + c;
        if (chan >= a.Dn) return;
        const float yf = row_lds[lds.y + t * width + c], yb = row_lds[lds.y + (a.L + t) * width + c];
        T* o = (T*)a.out + (size_t)b * a.out_sb + (long long)t * a.out_st + chan;
        const float gf = silu(IO::cvt(zf_raw)), gb = a.same_z ? gf : silu(IO::cvt(zb_raw));
        if (a.separate) {
            IO::st(o, yf * gf);
            IO::st(o + a.Dn, yb * gb);
        } else {
            IO::st(o, a.same_z ? (yf + yb) * gf : fmaf(yf, gf, yb * gb));
        }
    };
    const int outputs = a.L * width;
#pragma unroll
    for (int k = 0; k < kZAhead; k++)
        if (tid + k * threads < outputs) finish(tid + k * threads, z_ahead[0][k], z_ahead[1][k]);
    for (int i = tid + kZAhead * threads; i < outputs; i += threads) {
        const int t = i >> shift, chan = min(ch0 + (i & (width - 1)), a.Dn - 1);
        finish(i, z_of(0, t, chan), a.same_z ? T(0) : z_of(1, t, chan));
    }
    // the last K - 1 raw tokens of (tail_in || block), by the wave that read tail_in
    if (a.tail_out && s == 0 && seg == 0 && valid && n < a.K - 1) {
        const int pos = a.L + n - (a.K - 1);             // token of the block, or (negative) of the cached tail
        T v = 0;
        if (pos >= 0) v = xb[(long long)pos * da.x.st];
        else if (a.tail_in) v = ((const T*)a.tail_in)[((size_t)b * (a.K - 1) + a.K - 1 + pos) * a.Dn + ch];
        ((T*)a.tail_out)[((size_t)b * (a.K - 1) + n) * a.Dn + ch] = v;
    }
}

}  // namespace bm
