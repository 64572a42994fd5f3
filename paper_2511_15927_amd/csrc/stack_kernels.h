// A block's denoising steps through a stack of layers whose outputs feed each other, in one launch.
//
// Layer l + 1's x is layer l's output, and the mixer (depthwise conv, per-channel scan, gate, combine) mixes channels nowhere: a
// workgroup that holds both directions of a channel tile over the whole block can take it through every layer of every step
// without waiting for any other workgroup.  Launch by launch such a call spends half its time between launches and most of the
// rest on first loads: at batch 1 (d_inner 4096, 16 states) 6.9 us a layer and step of 32 tokens, here 2.4
// (what is left is two walks of dependent tokens at two waves per SIMD, and two barriers).
//
// The walk is that of row_kernels.h: a row of 16 lanes per chain, one state per lane, sixteen tokens dealt to the lanes of a row at
// a time.  x stays in LDS from layer to layer, rounded to the I/O dtype as it would be in memory; B, C (as fp32 rows), Delta
// and the gates of a step, which all layers share, are taken in once per step; the next layer's parameters, state and conv
// tail are requested while the present layer is walked.
#pragma once
#include "row_kernels.h"
#include "bimamba.h"

namespace bm {

struct StackArgs {
    // device copies of the caller's arrays, and [n_steps][n_layers] places of the layers' outputs (null: not stored)
    const bimamba_stack_layer* layers;
    const bimamba_inputs* steps;
    void* const* outs;
    int n_layers, n_steps;
    int L, Dn, P, HG, G, N, K;
    int dt_softplus, d_per_head, a_scalar;
    int tw, tw_log2, nseg, seg_len;   // as in RowArgs
};

// LDS of a workgroup, in floats: B|C rows, x and the outputs by channel, per-wave (u, Delta, D xc, raw Delta), segment summaries.
struct StackLds {
    int bc, x, y, ud, sum, total, pitch;
    __host__ __device__ StackLds(int L, int tw, int nseg, int seg_len)
    {
        const int waves = 2 * nseg * tw, width = 4 * tw;
        pitch = L | 1;                                   // floats of a channel's run of tokens (odd: no bank conflicts across channels)
        bc = 0;
        x = bc + (L + 2 * kRowTokens) * 32;              // (a row of spare tokens at either end, see row_kernels.h)
        y = x + width * pitch;
        ud = (y + 2 * width * pitch + 3) & ~3;
        sum = ud + waves * (seg_len / kRowTokens) * 64 * 4;
        total = sum + waves * 64 * 2;
    }
};

constexpr int kStackOutputs = 4;   // outputs of a thread at most

// grid (ceil(Dn / (4 tw)), 1, batch), block 128 * nseg * tw, dynamic LDS StackLds::total floats.  OUTPUTS: of a thread,
// L / (32 nseg) rounded up to 1, 2 or 4 (more of them cost registers that the walk needs).
template <typename IO, int OUTPUTS>
__global__ __launch_bounds__(64 * kRowMaxWaves, 1) void stack_kernel(const StackArgs a)
{
    using T = typename IO::T;
    extern __shared__ __attribute__((aligned(16))) float row_lds[];
    const StackLds lds(a.L, a.tw, a.nseg, a.seg_len);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = 2 * a.nseg * a.tw, threads = 64 * waves;
    const int s = wave & 1;
    const int tile = __builtin_amdgcn_readfirstlane((wave >> 1) / a.nseg), seg = (wave >> 1) - tile * a.nseg;   // seg: scan order
    const int b = blockIdx.z, n = lane & 15, shift = a.tw_log2 + 2, width = 1 << shift;   // channels of the workgroup
    const int ch0 = blockIdx.x * width, cl = tile * 4 + (lane >> 4);
    const bool valid = ch0 + cl < a.Dn;
    const int ch = min(ch0 + cl, a.Dn - 1), head = a.P == 1 ? ch : ch / a.P;
    const int grp = a.G == 1 ? 0 : __builtin_amdgcn_readfirstlane(ch0 / a.P / a.HG);   // a workgroup never straddles two B/C groups
    const int last = a.L - 1;
    auto token_of = [&](int j) { return s == 0 ? j : last - j; };
    const int j0 = seg * a.seg_len, j1 = min(a.L, j0 + a.seg_len), groups = max(0, (j1 - j0 + kRowTokens - 1) / kRowTokens);
    auto place = [&](int j) { return (long long)token_of(min(max(j, 0), last)); };
    const bool state = n < a.N;                          // lanes past the last state carry zeros
    float* const xs = row_lds + lds.x;
    float* const ud = row_lds + lds.ud + wave * (a.seg_len / kRowTokens) * 256;
    const int outputs = a.L * width;

    // A layer's pointers for this wave's direction: wave-uniform, fetched with scalar loads a layer before they are used, so that
    // the loads through them go out together without waiting.
    struct Places {
        const float *conv_w, *conv_b, *A, *D, *dt_bias;
        const float* h;
        const T* tail;
    };
    // (the tables of layers and steps by scalar loads: pointers read through them are known to be global memory)
    typedef const __attribute__((address_space(4))) bimamba_stack_layer* uniform_layer;
    typedef const __attribute__((address_space(4))) bimamba_inputs* uniform_inputs;
    auto places = [&](int l) {
        const uniform_layer ly = (uniform_layer)(a.layers + l);
        auto p = s == 0 ? &ly->f : &ly->b;
        return Places{p->conv_w, p->conv_b, p->A, p->D, p->dt_bias, s == 0 ? ly->h : nullptr, s == 0 && seg == 0 ? (const T*)ly->tail : nullptr};
    };
    // one layer's parameters, entry state and conv tail, as this lane needs them
    struct Layer {
        float w4[4], cb, dval, dtb, a2, h;
        T tail;                                          // scan position n - 16 of a forward chain's first segment (n > 16 - K)
    };
    const bool reads_tail = s == 0 && seg == 0 && n - kRowTokens >= -(a.K - 1);
    const unsigned tail_at = ((unsigned)b * (a.K - 1) + max(a.K - 1 + n - kRowTokens, 0)) * a.Dn + ch;
    const unsigned conv_at = (unsigned)ch * a.K, skip_at = a.d_per_head ? head : ch;
    const unsigned decay_at = a.a_scalar ? (unsigned)head : (unsigned)head * a.N + min(n, a.N - 1);
    const unsigned state_at = ((unsigned)b * a.Dn + ch) * a.N + min(n, a.N - 1);
    auto request = [&](const Places& p) {
        Layer v;
        load_taps(p.conv_w + conv_at, a.K, v.w4);
        v.cb = v.dtb = v.h = 0.0f;
        v.tail = 0;
        v.dval = p.D[skip_at];
        v.a2 = p.A[decay_at];
        if (p.conv_b) v.cb = p.conv_b[ch];
        if (a.dt_softplus && p.dt_bias) v.dtb = p.dt_bias[head];
        if (p.h) v.h = p.h[state_at];
        if (p.tail && a.K > 1) v.tail = p.tail[tail_at];
        return v;
    };
    Layer next = request(places(0));
    Places ahead = places(a.n_layers > 1 ? 1 : 0);

    for (int step = 0; step < a.n_steps; step++) {
        // ---- what the layers of a step share: x of the first one, B|C rows as fp32, Delta, the gates
        const uniform_inputs in = (uniform_inputs)(a.steps + step);
        const T* const zb = (const T*)in->z.ptr + (size_t)b * in->z.stride_batch;
        const T* const xb = (const T*)in->x.ptr + (size_t)b * in->x.stride_batch;
        const T* const db = (const T*)in->dt.ptr + (size_t)b * in->dt.stride_batch + head;
        T xr[OUTPUTS], zr[OUTPUTS];
#pragma unroll
        for (int k = 0; k < OUTPUTS; k++) {
            if (k * threads < outputs) {
                const int i = min(tid + k * threads, outputs - 1), t = i >> shift, chan = min(ch0 + (i & (width - 1)), a.Dn - 1);
                xr[k] = xb[(long long)t * in->x.stride_token + chan];
                zr[k] = zb[(long long)t * in->z.stride_token + chan];
            }
        }
        for (int g = 0; g < groups; g++) ud[g * 256 + 192 + lane] = IO::cvt(db[place(j0 + g * kRowTokens + n) * in->dt.stride_token]);
        {
            constexpr int kFlight = 8;
            const int m = tid & 15, which = (tid >> 4) & 1, rows = threads >> 5;
            const long long col_token = which ? in->C.stride_token : in->B.stride_token;
            const T* const col = (which ? (const T*)in->C.ptr : (const T*)in->B.ptr) + (size_t)b * (which ? in->C.stride_batch : in->B.stride_batch) + grp * a.N + min(m, a.N - 1);
            float* const dst = row_lds + lds.bc + (kRowTokens * 16 + m) * 2 + which;
            for (int t0 = tid >> 5; t0 < a.L; t0 += kFlight * rows) {
                T v[kFlight];
#pragma unroll
                for (int k = 0; k < kFlight; k++) v[k] = col[(long long)min(t0 + k * rows, last) * col_token];
#pragma unroll
                for (int k = 0; k < kFlight; k++)
                    if (t0 + k * rows < a.L) dst[(t0 + k * rows) * 32] = m < a.N ? IO::cvt(v[k]) : 0.0f;
            }
            if (a.L % kRowTokens != 0)
                for (int t = tid >> 5; t < kRowTokens; t += rows) dst[(t - kRowTokens) * 32] = dst[(a.L + t) * 32] = 0.0f;
        }
        float gate[OUTPUTS];
#pragma unroll
        for (int k = 0; k < OUTPUTS; k++) {
            if (k * threads < outputs) {
                const int i = tid + k * threads;
                gate[k] = silu(IO::cvt(zr[k]));
                if (i < outputs) xs[(i & (width - 1)) * lds.pitch + (i >> shift)] = IO::cvt(xr[k]);
            }
        }
        __syncthreads();

        const bool commit = step + 1 == a.n_steps;
        for (int l = 0; l < a.n_layers; l++) {
            Layer p = next;
            p.a2 = state ? p.a2 * kLog2e : 0.0f;
            if (!state) p.h = 0.0f;
            // (the state and tail of the next layer are not touched before it: one layer of a stack of one is committed last)
            if (l + 1 < a.n_layers || !commit) {
                next = request(ahead);
                ahead = places((l + 2) % a.n_layers);
            }
            typedef void* const __attribute__((address_space(4)))* uniform_place;
            T* const out = (T*)((uniform_place)a.outs)[step * a.n_layers + l];   // (fetched here, used at the layer's end)
            // ---- per-token work of this lane's tokens: group g, lane n is scan position j0 + 16 g + n
            const float* const xc_row = xs + cl * lds.pitch;
            float before = 0.0f;
            {
                const int j = j0 - kRowTokens + n;
                if (j >= 0) before = xc_row[token_of(j)];
                else if (reads_tail) before = IO::cvt(p.tail);
            }
            float dsum = 0.0f;
            for (int g = 0; g < groups; g++) {
                const int j = j0 + g * kRowTokens + n;
                const bool there = j < j1;
                const float x0 = there ? xc_row[token_of(min(j, last))] : 0.0f;
                float delta = ud[g * 256 + 192 + lane];
                float pre = fmaf(p.w4[3], x0, p.cb);
                pre = fmaf(p.w4[2], row_back<1>(x0, before), pre);
                pre = fmaf(p.w4[1], row_back<2>(x0, before), pre);
                pre = fmaf(p.w4[0], row_back<3>(x0, before), pre);
                before = x0;
                const float xc = silu(pre);
                if (a.dt_softplus) delta = softplus(delta + p.dtb);
                if (!there) delta = 0.0f;                // a token that does not exist leaves the state as it is
                dsum += delta;
                ud[g * 256 + lane] = delta * xc;
                ud[g * 256 + 64 + lane] = delta;
                ud[g * 256 + 128 + lane] = p.dval * xc;
            }
            // the committed tail: the last K - 1 raw tokens of (tail || block), by the wave that holds the old one
            if (commit && a.K > 1 && s == 0 && seg == 0 && ((uniform_layer)(a.layers + l))->tail) {
                const int pos = a.L + n - (a.K - 1);     // token of the block, or (negative) of the cached tail: lane pos + 16 holds that
                const float old = __shfl(IO::cvt(p.tail), (lane & 48) | ((pos + kRowTokens) & 15));
                if (n < a.K - 1 && valid)
                    ((T*)((uniform_layer)(a.layers + l))->tail)[((size_t)b * (a.K - 1) + n) * a.Dn + ch] = io_value<IO>(pos >= 0 ? xc_row[pos] : old);
            }
            // ---- the recurrence over the segment
            float h = p.h;
            const float2* const bc = reinterpret_cast<const float2*>(row_lds + lds.bc) + kRowTokens * 16 + n;
            auto walk = [&](auto with_output, auto direction) {
                constexpr bool kOutput = decltype(with_output)::value;
                constexpr int kDir = decltype(direction)::value;
                row_walk<kOutput, kDir, 256>(h, p.a2, ud, bc, groups, j0, last, lane, n, [&](int j, float y) {
                    if (j + n < j1) row_lds[lds.y + (s * width + cl) * lds.pitch + token_of(j + n)] = y;
                });
            };
            using Up = std::integral_constant<int, 1>;
            using Down = std::integral_constant<int, -1>;
            if (a.nseg > 1) {
                h = 0.0f;
                if (seg + 1 < a.nseg) {                  // (nothing starts from the scan-last segment's end)
                    if (s == 0) walk(std::false_type{}, Up{});
                    else walk(std::false_type{}, Down{});
                }
                row_lds[lds.sum + wave * 128 + lane] = h;
                row_lds[lds.sum + wave * 128 + 64 + lane] = row_total(dsum);
                __syncthreads();
                h = p.h;
                for (int e = 0; e < seg; e++) {
                    const float* from = row_lds + lds.sum + (((tile * a.nseg + e) << 1) + s) * 128 + lane;
                    h = fmaf(fast_exp2(from[64] * p.a2), h, from[0]);
                }
            }
            if (s == 0) walk(std::true_type{}, Up{});
            else walk(std::true_type{}, Down{});
            float* const h_out = ((uniform_layer)(a.layers + l))->h;
            if (commit && s == 0 && h_out && valid && state && j1 == a.L && j1 > j0) h_out[state_at] = h;
            __syncthreads();                             // both directions' outputs
            // ---- gate, combine, round: channels across the lanes; the result is the next layer's x
#pragma unroll
            for (int k = 0; k < OUTPUTS; k++) {
                if (k * threads < outputs) {
                    const int i = tid + k * threads, t = i >> shift, c = i & (width - 1);
                    if (i < outputs) {
                        const float yf = row_lds[lds.y + c * lds.pitch + t], yb = row_lds[lds.y + (width + c) * lds.pitch + t];
                        const T v = io_value<IO>((yf + yb) * gate[k]);
                        xs[c * lds.pitch + t] = IO::cvt(v);
                        if (out && ch0 + c < a.Dn) out[((size_t)b * a.L + t) * a.Dn + ch0 + c] = v;
                    }
                }
            }
            __syncthreads();                             // the next layer's x
        }
    }
}

}  // namespace bm
