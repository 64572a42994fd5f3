// The stack of layers of stack_kernels.h with four lanes to a chain and the steps of a block side by side.
//
// A block's steps do not depend on each other: each has inputs of its own and starts from the same cached state, which only the
// last one replaces.  A workgroup holds 16 channels and takes up to eight steps through the layers at once, a wave for each (step,
// direction), so that a SIMD has four waves to issue from where a row of lanes per chain, one step after the other, has two.
//
// The four lanes of a chain hold a quarter of its states each and deal its tokens among themselves, four at a time, as in kernels.h:
// the token's owner evaluates conv, SiLU and softplus, the others read Delta and u out of its registers through quad-permute operands.
// That is 33 vector instructions a lane and token at 16 states, 132 a chain's token; one lane per state takes 180.  24 layers x 8 steps
// of 32 tokens at batch 1, d_inner 4096, 16 states: 450 -> 221 us.  The directions meet in
// the middle: in the first half of its walk a wave leaves its outputs in LDS, in the second it adds what the other one left, gates,
// rounds and puts the result where the next layer reads its x.  Two barriers a layer.
#pragma once
#include "stack_kernels.h"

namespace bm {

constexpr int kQuadChannels = 16;   // of a workgroup
constexpr int kQuadMaxSteps = 8;    // side by side

// LDS of a step, in floats: B|C rows as [token][quarter of the states][B, C], then x, the outputs left for the other direction, the gates
// and Delta by channel.  pitch / 4 is odd: a wave's accesses (16 channels x 4 tokens) hit every bank once.  Nothing is read of the row in
// front of B|C; it moves the steps of a workgroup against each other by half the banks (24 layers x 8 steps of 32 tokens 239.0 us, 241.8
// without it).
struct QuadLds {
    int tokens, pitch, bc, x, y, gate, delta, total;   // tokens: of the block, rounded up to whole groups of either half
    __host__ __device__ QuadLds(int L, int N)
    {
        tokens = (L + 7) & ~7;
        pitch = tokens + 4;
        bc = 2 * N;
        x = bc + tokens * 2 * N;
        y = x + kQuadChannels * pitch;
        gate = y + kQuadChannels * pitch;
        delta = gate + kQuadChannels * pitch;
        total = delta + kQuadChannels * pitch;
    }
};

__device__ __forceinline__ float quad_other_pair(float v)   // quad_perm [2,3,0,1]
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));
}

// grid (ceil(Dn / 16), 1, batch), block 128 * side, dynamic LDS side * QuadLds::total floats; side: steps side by side.
template <typename IO, int N>
__global__ __launch_bounds__(64 * 2 * kQuadMaxSteps, 1) void stack_quad_kernel(const StackArgs a, const int side)
{
    static_assert(N == 4 || N == 8 || N == 16, "a quad holds 4, 8 or 16 states");
    using T = typename IO::T;
    constexpr int NS = N / 4;
    typedef __attribute__((__vector_size__(NS * sizeof(float)), __aligned__(4))) float Slice;
    extern __shared__ __attribute__((aligned(16))) float quad_lds[];
    const QuadLds lds(a.L, N);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), s = wave & 1, slot = wave >> 1;
    const int b = blockIdx.z, sub = lane & 3, cl = lane >> 2;
    const int ch0 = blockIdx.x * kQuadChannels;
    const bool valid = ch0 + cl < a.Dn;
    const int ch = min(ch0 + cl, a.Dn - 1), head = a.P == 1 ? ch : ch / a.P;
    const int grp = a.G == 1 ? 0 : __builtin_amdgcn_readfirstlane(ch0 / a.P / a.HG);   // a workgroup never straddles two B/C groups
    float* const mine = quad_lds + slot * lds.total;
    const int groups = lds.tokens / 4;

    // A layer's pointers for this wave's direction and what this lane needs of it, both a layer ahead (as in stack_kernel).
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
        return Places{p->conv_w, p->conv_b, p->A, p->D, p->dt_bias, s == 0 ? ly->h : nullptr, s == 0 ? (const T*)ly->tail : nullptr};
    };
    struct Layer {
        float w4[4], cb, dval, dtb;
        Slice a2, h;
        T tail;                                          // token sub - 4 (sub > 4 - K)
    };
    const bool reads_tail = s == 0 && sub - 4 >= -(a.K - 1);
    const unsigned tail_at = ((unsigned)b * (a.K - 1) + max(a.K - 1 + sub - 4, 0)) * a.Dn + ch;
    const unsigned conv_at = (unsigned)ch * a.K, skip_at = a.d_per_head ? head : ch;
    const unsigned state_at = ((unsigned)b * a.Dn + ch) * N + sub * NS;
    auto request = [&](const Places& p) {
        Layer v;
        load_taps(p.conv_w + conv_at, a.K, v.w4);
        v.cb = v.dtb = 0.0f;
        v.tail = 0;
        v.dval = p.D[skip_at];
        if (a.a_scalar) {
            const float v0 = p.A[head];
#pragma unroll
            for (int n = 0; n < NS; n++) v.a2[n] = v0;
        } else {
            v.a2 = *(const Slice*)(p.A + (unsigned)head * N + sub * NS);
        }
#pragma unroll
        for (int n = 0; n < NS; n++) v.h[n] = 0.0f;
        if (p.conv_b) v.cb = p.conv_b[ch];
        if (a.dt_softplus && p.dt_bias) v.dtb = p.dt_bias[head];
        if (p.h) v.h = *(const Slice*)(p.h + state_at);
        if (p.tail && a.K > 1) v.tail = p.tail[tail_at];
        return v;
    };
    Layer next = request(places(0));
    Places ahead = places(a.n_layers > 1 ? 1 : 0);

    for (int first = 0; first < a.n_steps; first += side) {
        const int step = first + slot;
        const bool active = step < a.n_steps, last_round = first + side >= a.n_steps;
        // ---- what the layers of a step share: x of the first one, the gates, Delta, B|C rows; tokens past the block's end are zeros
        if (active) {
            const uniform_inputs in = (uniform_inputs)(a.steps + step);
            const int t2 = tid & 127, c = t2 & 15, chan = min(ch0 + c, a.Dn - 1), hd = a.P == 1 ? chan : chan / a.P;
            const T* const xb = (const T*)in->x.ptr + (size_t)b * in->x.stride_batch + chan;
            const T* const zb = (const T*)in->z.ptr + (size_t)b * in->z.stride_batch + chan;
            const T* const db = (const T*)in->dt.ptr + (size_t)b * in->dt.stride_batch + hd;
            constexpr int kCols = 2 * N, kRows = 128 / kCols;
            const int col = t2 % kCols, which = col / NS % 2, n = col / (2 * NS) * NS + col % NS;   // [quarter][B, C][state]
            const T* const from = (which ? (const T*)in->C.ptr : (const T*)in->B.ptr) + (size_t)b * (which ? in->C.stride_batch : in->B.stride_batch) + grp * N + n;
            const long long from_token = which ? in->C.stride_token : in->B.stride_token;
            constexpr int kFlight = 4, kTokens = 8 * kFlight, kBcFlight = kTokens / kRows;
            // (tokens at a time with all of their loads in flight, x, z and Delta's with the rows': 6 layers x 4 steps of 64 tokens at
            // batch 2 143.8 -> 139.7 us, 8 layers x 2 steps of 32, fp32, 48.8 -> 47.8)
            for (int base = 0; base < lds.tokens; base += kTokens) {
                const int t0 = base + (t2 >> 4), r0 = base + t2 / kCols;
                T xr[kFlight], zr[kFlight], dr[kFlight], bc[kBcFlight];
#pragma unroll
                for (int k = 0; k < kFlight; k++) {
                    const long long t = min(t0 + 8 * k, a.L - 1);
                    xr[k] = xb[t * in->x.stride_token];
                    zr[k] = zb[t * in->z.stride_token];
                    dr[k] = db[t * in->dt.stride_token];
                }
#pragma unroll
                for (int k = 0; k < kBcFlight; k++) bc[k] = from[(long long)min(r0 + kRows * k, a.L - 1) * from_token];
#pragma unroll
                for (int k = 0; k < kFlight; k++) {
                    const int t = t0 + 8 * k, at = c * lds.pitch + t;
                    const bool there = t < a.L;
                    if (t < lds.tokens) {
                        mine[lds.x + at] = there ? IO::cvt(xr[k]) : 0.0f;
                        mine[lds.gate + at] = there ? silu(IO::cvt(zr[k])) : 0.0f;
                        mine[lds.delta + at] = there ? IO::cvt(dr[k]) : 0.0f;
                    }
                }
#pragma unroll
                for (int k = 0; k < kBcFlight; k++) {
                    const int t = r0 + kRows * k;
                    if (t < lds.tokens) mine[lds.bc + t * kCols + col] = t < a.L ? IO::cvt(bc[k]) : 0.0f;
                }
            }
        }
        __syncthreads();

        const bool commits = active && step + 1 == a.n_steps && s == 0;
        for (int l = 0; l < a.n_layers; l++) {
            Layer p = next;
            // (in the last round no layer is requested after the last one: its state may have been committed by then)
            if (l + 1 < a.n_layers || !last_round) {
                next = request(ahead);
                ahead = places((l + 2) % a.n_layers);
            }
            float a2[NS], h[NS];
#pragma unroll
            for (int n = 0; n < NS; n++) {
                a2[n] = p.a2[n] * kLog2e;
                h[n] = p.h[n];
            }
            float before = reads_tail ? IO::cvt(p.tail) : 0.0f;   // raw x of the group before
            // the committed tail: the last K - 1 raw tokens of (tail || block), stored once every step has read the old one
            float tail_new = 0.0f;
            if (commits && a.K > 1) {
                const int pos = a.L + sub - (a.K - 1);   // token of the block, or (negative) of the cached tail: lane pos + 4 holds that
                const float old = __shfl(before, (lane & ~3) | ((pos + 4) & 3));
                tail_new = pos >= 0 ? mine[lds.x + cl * lds.pitch + min(pos, a.L - 1)] : old;
            }
            typedef void* const __attribute__((address_space(4)))* uniform_place;
            T* const out = active ? (T*)((uniform_place)a.outs)[step * a.n_layers + l] : nullptr;

            auto half = [&](auto dir_c, auto final_c, int g0, int g1) {
                constexpr bool kUp = decltype(dir_c)::value > 0, kFinal = decltype(final_c)::value;
                const int own = kUp ? sub : 3 - sub;     // the lane's token above the group's lowest one
                float* const x_l = mine + lds.x + cl * lds.pitch + own;
                const float* const bc_l = mine + lds.bc + sub * 2 * NS;
                const int to_y = lds.y - lds.x, to_gate = lds.gate - lds.x, to_delta = lds.delta - lds.x;
#pragma unroll 1
                for (int g = g0; g < g1; g++) {
                    const int t0 = kUp ? 4 * g : lds.tokens - 4 - 4 * g, t = t0 + own;
                    float* const at = x_l + t0;
                    const float x0 = at[0];
                    float delta = at[to_delta];
                    float pre = fmaf(p.w4[3], x0, p.cb);
#pragma unroll
                    for (int k = 1; k <= 3; k++)         // (the lanes that wrap round hand on the group before)
                        pre = fmaf(chain_lane_back<4>(sub >= 4 - k ? before : x0, k), p.w4[3 - k], pre);
                    before = x0;
                    float xc = silu(pre);
                    if (a.dt_softplus) delta = softplus(delta + p.dtb);
                    if (t >= a.L) delta = xc = 0.0f;     // a token that does not exist leaves the state as it is
                    const float u = delta * xc;
                    float ys[4];
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        const float* const row = bc_l + (t0 + (kUp ? j : 3 - j)) * (2 * N);
                        float bv[NS], cv[NS];
#pragma unroll
                        for (int n = 0; n < NS; n++) {
                            bv[n] = row[n];
                            cv[n] = row[NS + n];
                        }
                        float dj = chain_lane_pick<4>(delta, j), uj = chain_lane_pick<4>(u, j);
                        // (values of their own, not permuted operands, which halve an instruction's rate: four of them cost what two
                        // moves and eight products do not; 24 layers x 8 steps of 32 tokens 225.5 -> 220.8 us)
                        if constexpr (NS > 1) asm volatile("" : "+v"(dj), "+v"(uj));
                        float yj = 0.0f;
#pragma unroll
                        for (int n = 0; n < NS; n++) {
                            h[n] = fmaf(fast_exp2(dj * a2[n]), h[n], uj * bv[n]);
                            yj = n == 0 ? cv[n] * h[n] : fmaf(cv[n], h[n], yj);
                        }
                        ys[j] = sum_over_chain_lanes<2>(yj);
                    }
                    // each lane its own token's sum over the quad: pairs, then what the other pair has of the tokens alike (six permuted
                    // additions and three selects where a sum in every lane takes eight and four: 232.8 -> 225.5 us, the same bits)
                    const float even = (sub & 1) ? ys[1] : ys[0], odd = (sub & 1) ? ys[3] : ys[2];
                    const float y01 = even + quad_other_pair(even), y23 = odd + quad_other_pair(odd);
                    const float y = fmaf(p.dval, xc, (sub & 2) ? y23 : y01);
                    if constexpr (!kFinal) {
                        at[to_y] = y;
                    } else {
                        const T v = io_value<IO>((y + at[to_y]) * at[to_gate]);
                        at[0] = t < a.L ? IO::cvt(v) : 0.0f;
                        if (out && valid && t < a.L) out[((size_t)b * a.L + t) * a.Dn + ch] = v;
                    }
                }
            };
            using Up = std::integral_constant<int, 1>;
            using Down = std::integral_constant<int, -1>;
            if (active) {
                if (s == 0) half(Up{}, std::false_type{}, 0, groups / 2);
                else half(Down{}, std::false_type{}, 0, groups / 2);
            }
            __syncthreads();                             // what the other direction left is there
            if (active) {
                if (s == 0) half(Up{}, std::true_type{}, groups / 2, groups);
                else half(Down{}, std::true_type{}, groups / 2, groups);
            }
            __syncthreads();                             // the next layer's x; every step has read the layer's state and tail
            if (commits) {
                float* const h_out = ((uniform_layer)(a.layers + l))->h;
                T* const t_out = (T*)((uniform_layer)(a.layers + l))->tail;
                if (h_out && valid) {
                    Slice v;
#pragma unroll
                    for (int n = 0; n < NS; n++) v[n] = h[n];
                    *(Slice*)(h_out + state_at) = v;
                }
                if (t_out && valid && sub < a.K - 1) t_out[((size_t)b * (a.K - 1) + sub) * a.Dn + ch] = io_value<IO>(tail_new);
            }
        }
    }
}

}  // namespace bm
