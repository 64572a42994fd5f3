// Gradients of the bidirectional mixer path in the selective-scan layout (one head per channel: Delta, A and D per
// channel; B and C shared by the channels of a group; no conv on B and C), for gfx950.
//
// The paper trains these models (App. A.2) but gives no backward algorithm; what is computed here is the chain rule of
// the forward definition (Sec. 3.2 eqs. 4-6 in the concrete selective form), evaluated in the reverse of each
// direction's scan order.  With t+ the token after t in scan order, t- the one before, and dg_t the gradient of the
// gated output of the direction:
//   dz_t = dg_t y_t silu'(z_t)                       dy_t = dg_t silu(z_t)
//   dh_t[n] = C_t[n] dy_t + a_{t+}[n] dh_{t+}[n]
//   dC_t[n] += sum_channels dy_t h_t[n]              dB_t[n] += sum_channels dh_t[n] Delta_t xc_t
//   dA[n] += dh_t[n] h_{t-}[n] a_t[n] Delta_t        dD += dy_t xc_t
//   dDelta_t = sum_n dh_t[n] (h_{t-}[n] a_t[n] A[n] + B_t[n] xc_t)
//   dxc_t = D dy_t + sum_n dh_t[n] Delta_t B_t[n]    dpre_t = dxc_t silu'(pre_t)
//   dx_t = sum_j w[K-1-j] dpre_{t + j steps}         dw[k] += dpre_t x_{t - (K-1-k) steps},  dcb += dpre_t
//
// Mapping: a lane is one (direction, batch, channel) chain, as in the forward sweep with one lane per chain, and the
// sequence is cut into segments that all walk at once, so that a call of any size brings the two waves per SIMD which
// the walk's register budget allows (bwd_segments in bwd_inst.hip).  The backward recurrence needs the states in the
// reverse of the order the forward recurrence makes them, so
//   bwd_state_kernel  walks each segment forward from a zero state and stores the state entering every chunk of
//                     kBwdChunk tokens, the Delta summed up to there, and the segment's end state.  On the way it also
//                     sums what the segment's tokens contribute to the dh of the tokens before it:
//                     sum_t exp(A W_t) C_t dy_t, W_t the Delta from the segment's start to t;
//   bwd_carry_kernel  folds both across the segments (h in scan order, dh against it);
//   bwd_kernel        takes a segment's chunks last to first, starting from the folded dh: it recomputes a chunk's
//                     states from the stored one (plus the decayed state entering the segment) and then walks the chunk
//                     backwards.  A token's dx takes dpre of the three tokens after it, which the next segment owns:
//                     the walk starts with those three, for their dpre only.  For the same reason the dh sums run over
//                     windows that start three tokens into their segment.
// dB_t and dC_t are sums over the channels of a group: each wave adds its 64 channels with a reduce-scatter over its
// lanes and stores the sums into its own slot of a partial buffer.  Parameter gradients are kept per lane and stored
// once per segment.  bwd_sum_kernel adds the slots of both in a fixed order (no atomics: the result does not depend on
// timing).  When both directions read the same activations their gradients of x, z and Delta have to be added: the two
// waves of a channel tile walk a segment's tokens in opposite orders and meet in its middle, as in the forward sweep;
// each parks its fp32 values for the half it reaches first and, past one workgroup barrier, adds what the other parked
// to its own values for the other half and rounds once to the I/O dtype.
#pragma once
#include "kernels.h"

namespace bm {

// The fp32 gradients of x, z and Delta of one (token, channel) as one direction leaves them for the other to add.
struct Parked {
    float dx, dz, ddt;
};

struct BwdArgs {
    DirArgs dir[2];          // x, z, dt views, prepared fp32 B|C rows and parameters of each direction
    TensorArg dout;          // [batch][L][Dn] (ADD) or [batch][L][2 Dn] (SEPARATE), I/O dtype
    // Workspace blocks of one wave: [..][tile][N / 4][64 lanes][4] floats for states, [..][tile][64 lanes] for sums.
    float* state;            // [2][batch][nseg][seg_chunks] blocks: the state entering each chunk (scan order), from a zero
                             // state at the segment's start
    float* state_w;          // [2][batch][nseg][seg_chunks]: Delta summed from the segment's start to the chunk
    float* seg_h;            // [2][batch][nseg] blocks: the segment's end state, then the state entering it
    float* seg_d;            // [2][batch][nseg] blocks: the segment's dh sum, then the dh of the tokens after its window
    float* seg_w;            // [2][2][batch][nseg]: Delta summed over the segment, over its dh window
    float* param_part;       // [2][batch][nseg][N + 7][tiles * 64]: dA, dD, dconv_w, dconv_b, ddt_bias of a segment
    Parked* parked;          // [batch][L][Dn]: values of the direction that reaches a token first (park only)
    TensorArg gdx[2], gdz[2], gddt[2];   // the caller's gradient views per direction (equal when park)
    int park;                // both directions read the same activations: their gradients are added (see above)
    float* bc_part[2];       // per direction: [batch][L][G][slots][N][2] fp32 partial sums of dB and dC, one slot per wave
    int bc_slots;            // slots per group: channel tiles of a group (x 2 when both directions feed one buffer)
    int bc_slot_of_rev;      // slot offset of the reverse direction's waves (0 when it has a buffer of its own)
    int L, Dn, G, K, dt_softplus, separate;
    int nseg, seg_len, seg_chunks, tiles;
};

// Tokens per chunk: what bwd_kernel keeps of one chunk is a state per token, half of them in registers and, for 16
// states, the other half in LDS, so that a wave fits 256 registers and a SIMD holds two.
constexpr int kBwdChunk = 8;
template <int N>
constexpr int kBwdLdsTokens = N >= 16 ? 5 : 0;
template <int N>
constexpr size_t kBwdLdsBytes = (size_t)4 * kBwdLdsTokens<N> * 64 * N * sizeof(float);   // of a workgroup: two fit a CU
constexpr int kBwdParams = 7;   // parameter gradients of a chain besides dA: dD, four taps, conv bias, Delta bias

__device__ __forceinline__ float dsilu(float v)
{
    const float s = __builtin_amdgcn_rcpf(1.0f + fast_exp2(-kLog2e * v));
    return s * fmaf(v, 1.0f - s, 1.0f);
}
__device__ __forceinline__ float sigmoidf(float v) { return __builtin_amdgcn_rcpf(1.0f + fast_exp2(-kLog2e * v)); }

// Sums scale * v[j], NV values per lane, over the 64 lanes of the wave and leaves the total of value j in the lanes
// j * (64 / NV) ... (j + 1) * (64 / NV) - 1 (returned by every lane: the total of value lane / (64 / NV)).
// A reduce-scatter: each step halves the values a lane still carries.  The lane whose bit is clear keeps the first half
// and receives its partner's first half, the other lane the second half, so about 2 NV instructions do the work of
// 6 * NV adds.  Partners: the other 32-lane half and the other row of 16 by the swap instructions of gfx950, then inside a
// row by lane-permute operands.  There both partners can form both sums, each an add with a permuted operand, and the
// second one is written only where it is kept (bank masks pick lane groups of four): two instructions for a pair of
// values where selecting first takes three.  The products are formed after the first exchange, with both partners' scales at
// hand: a multiplication and a multiply-add for a pair of values, not two multiplications and an add.  (Inline assembly: the compiler does not form an add that keeps its old
// result in some banks.  s_nop 1: a permuted operand must not have been written by the two instructions before.)
template <int CTRL>
__device__ __forceinline__ float from_partner(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int NV>
__device__ __forceinline__ float wave_reduce_scatter(float (&v)[NV], float scale)
{
    static_assert(NV == 4 || NV == 8 || NV == 16, "4, 8 or 16 values per lane");
    // lane bit 5: the other half of the wave
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(scale), __float_as_uint(scale), false, false);
#pragma unroll
    for (int i = 0; i < NV / 2; i++) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[NV / 2 + i]), false, false);
        v[i] = fmaf(__uint_as_float(r[1]), __uint_as_float(s[1]), __uint_as_float(r[0]) * __uint_as_float(s[0]));
    }
    // lane bit 4: the neighbouring row of 16
#pragma unroll
    for (int i = 0; i < NV / 4; i++) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[NV / 4 + i]), false, false);
        v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    float t = v[0];
    if constexpr (NV == 16) {
        // lane bit 3: banks 2 and 3 of a row keep the second half; the partner is 8 lanes away.  Lane bit 2: banks 1 and 3; the
        // partner is the mirror lane of the other bank of the half row.
        float a, b;
        asm("s_nop 1\n\t"
            "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
            "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
            "s_nop 0\n\t"
            "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
            "s_nop 0\n\t"
            "v_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa"
            : "=&v"(a), "=&v"(b) : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
        t = a;
    } else if constexpr (NV == 8) {
        asm("s_nop 1\n\t"
            "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc"
            : "=&v"(t) : "v"(v[0]), "v"(v[1]));
    }
    // what is left of the lane index carries the same value: plain sums, quads first (the mirror needs equal quads)
    t += from_partner<0xB1>(t);                             // quad_perm [1,0,3,2]
    t += from_partner<0x4E>(t);                             // quad_perm [2,3,0,1]
    if constexpr (NV <= 8) t += from_partner<0x141>(t);     // row_half_mirror
    if constexpr (NV <= 4) t += from_partner<0x128>(t);     // row_ror:8
    return t;
}

// The per-wave view of a (segment, direction, channel tile): places, constants and the scan-order token walk.
template <int N, typename IO>
struct BwdWave {
    using T = typename IO::T;
    int s, b, seg, tile, lane, ch, grp;
    bool exists, valid;          // the wave has a tile of its own; the lane has a channel of its own
    int j0, j1;                  // the segment's scan positions [j0, j1); those outside [0, L) do not exist
    int k0, k1;                  // its chunks [k0, k1) that hold tokens
    int L, dir;
    float a2[N];                 // A * log2(e)
    float w4[4], cb, dval, dtb;  // conv taps (w4[3] on the current token), conv bias, D, Delta bias

    // A tensor walked token by token: a wave-uniform byte pointer; the lane's place in a row is a byte offset of its own.
    struct Walked {
        const char* base;    // token 0 of this batch element (and direction, where the tensor has one half per direction)
        int stride;          // bytes per token (the host bounds token strides at 2^26 elements, channels included)
    };
    Walked x, z, dt, g, row;

    __device__ __forceinline__ int token(int j) const { return dir > 0 ? j : L - 1 - j; }
    __device__ __forceinline__ const char* at(const Walked& t, int j) const { return t.base + (long long)token(j) * t.stride; }
    __device__ __forceinline__ int step(const Walked& t) const { return dir * t.stride; }   // bytes from one scan position to the next
    // block `i` of a [2][batch][nseg]... workspace array, in waves
    __device__ __forceinline__ size_t place(const BwdArgs& a, int per_seg, int i) const
    {
        return ((((size_t)s * gridDim.z + b) * a.nseg + seg) * per_seg + i) * a.tiles + tile;
    }
};

template <int N, typename IO>
__device__ __forceinline__ void bwd_wave_setup(const BwdArgs& a, BwdWave<N, IO>& w)
{
    using T = typename IO::T;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    w.s = wave & 1;
    w.b = blockIdx.z;
    w.seg = blockIdx.y;
    w.lane = threadIdx.x & 63;
    w.tile = (int)blockIdx.x * 2 + (wave >> 1);
    w.exists = w.tile < a.tiles;                         // the second tile of the last workgroup may not exist:
    if (!w.exists) w.tile -= 1;                          // its waves shadow the first (they compute and store nothing)
    w.valid = w.exists && w.tile * 64 + w.lane < a.Dn;
    w.ch = min(w.tile * 64 + w.lane, a.Dn - 1);          // lanes past the last channel shadow it and contribute nothing
    // uniform: a tile never straddles two B/C groups (divisions run on the vector ALU: back to a scalar register at once,
    // or everything addressed through the quotient stays there)
    w.grp = __builtin_amdgcn_readfirstlane(w.tile * 64 / (a.Dn / a.G));
    w.L = a.L;
    w.dir = w.s == 0 ? 1 : -1;
    // every segment is seg_chunks whole chunks, so that the chunks of both directions hold the same tokens: the last one
    // may reach past the sequence (scan positions from L on in the forward direction, below 0 in the reverse one)
    const int t0 = w.seg * a.seg_len;
    w.j0 = w.s == 0 ? t0 : a.L - t0 - a.seg_len;
    w.j1 = w.j0 + a.seg_len;
    w.k0 = w.j0 < 0 ? -w.j0 / kBwdChunk : 0;
    w.k1 = min(a.seg_chunks, (a.L - w.j0 + kBwdChunk - 1) / kBwdChunk);
    const DirArgs& da = a.dir[w.s];
#pragma unroll
    for (int n = 0; n < N; n++) w.a2[n] = da.A[(size_t)w.ch * N + n] * kLog2e;
    load_taps(da.conv_w + (size_t)w.ch * a.K, a.K, w.w4);
    w.cb = da.conv_b ? da.conv_b[w.ch] : 0.0f;
    w.dval = da.D[w.ch];
    w.dtb = (a.dt_softplus && da.dt_bias) ? da.dt_bias[w.ch] : 0.0f;
    auto walked = [&](const TensorArg& t, int off) {
        return typename BwdWave<N, IO>::Walked{(const char*)t.p + ((size_t)w.b * t.sb + off) * sizeof(T), (int)(t.st * (long long)sizeof(T))};
    };
    w.x = walked(da.x, 0);
    w.z = walked(da.z, 0);
    w.dt = walked(da.dt, 0);
    w.g = walked(a.dout, a.separate ? w.s * a.Dn : 0);
    w.row = {(const char*)(da.bc + ((size_t)w.b * a.L * a.G + w.grp) * (2 * N)), a.G * 2 * N * (int)sizeof(float)};
}

// f(n, exp(v A[n])) for all n.  One exponential each, whatever A: forming the factors of an arithmetic A by repeated
// products, as the forward sweep does for bf16 I/O, puts up to N - 1 more roundings into the fp32 gradients: error of dB
// against 64 bits 2.3e-7 with exponentials, 3.8e-7 with products (8 x 8192 tokens of 4096 channels; 11.3 against 10.1 ms).
template <int N, typename IO, typename F>
__device__ __forceinline__ void for_each_decay(const BwdWave<N, IO>& w, float v, F f)
{
#pragma unroll
    for (int n = 0; n < N; n++) f(n, fast_exp2(v * w.a2[n]));
}

// Two raw values of a token, kept in one register where the I/O dtype allows it.
template <typename IO>
struct RawPair {
    float a, b;
    __device__ __forceinline__ void set(float va, float vb) { a = va; b = vb; }
    __device__ __forceinline__ float first() const { return a; }
    __device__ __forceinline__ float second() const { return b; }
    __device__ __forceinline__ void clear_first() { a = 0.0f; }
    __device__ __forceinline__ void clear_second() { b = 0.0f; }
    __device__ __forceinline__ void opaque() {}
};
template <>
struct RawPair<IoBF16> {
    unsigned v;
    __device__ __forceinline__ void set(unsigned short va, unsigned short vb) { v = (unsigned)va | ((unsigned)vb << 16); opaque(); }
    __device__ __forceinline__ float first() const { return __uint_as_float(v << 16); }
    __device__ __forceinline__ float second() const { return __uint_as_float(v & 0xffff0000u); }
    __device__ __forceinline__ void clear_first() { v &= 0xffff0000u; }
    __device__ __forceinline__ void clear_second() { v &= 0xffffu; }
    __device__ __forceinline__ void opaque() { asm volatile("" : "+v"(v)); }   // unpacked where used, not kept unpacked
};

// Has a value computed where it stands.  Left alone the compiler moves sums that are used much later (and what only a
// conditional store needs) down the token's blocks and keeps their operands alive instead: more registers than there are.
__device__ __forceinline__ void settle(float& v) { asm volatile("" : "+v"(v)); }

template <int N>
__device__ __forceinline__ void store_block(float* dst, const float (&v)[N], int lane)
{
#pragma unroll
    for (int q = 0; q < N / 4; q++)
        *reinterpret_cast<float4*>(dst + (q * 64 + lane) * 4) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}
template <int N>
__device__ __forceinline__ void load_block(const float* src, float (&v)[N], int lane)
{
#pragma unroll
    for (int q = 0; q < N / 4; q++) {
        const float4 t = *reinterpret_cast<const float4*>(src + (q * 64 + lane) * 4);
        v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
    }
}

// The walk of bwd_state_kernel.  WITH_D: the dh sum is wanted (some segment precedes this one in scan order).
template <int N, typename IO, bool WITH_D>
__device__ __forceinline__ void bwd_state_walk(const BwdArgs& a, const BwdWave<N, IO>& w, float4* ds)
{
    using T = typename IO::T;
    constexpr int CT = kBwdChunk / 2, kSteps = kBwdChunk / CT;   // half a chunk at a time: what is requested ahead fits beside the sums
    const bool sp = a.dt_softplus != 0;
    const bool end_wanted = w.j1 < a.L;                   // some segment follows in scan order
    unsigned lo = (unsigned)(w.ch * sizeof(T));
    float h[N];
    // The dh sum by chunks: exp(A W) at the chunk's start, an exponential, times what its tokens add up to with the decays counted
    // from there, products of those that the states take anyway: a multiplication where an exponential of its own takes a
    // multiplication and two issue slots more (state pass of 8 x 8192 tokens, 4096 channels: 3.19 -> 2.4 ms with the rest of its
    // steps).  The sum then rounds once a chunk, which is more than the products' roundings cost: relative error against 64 bits of dB just
    // before a segment's 29 tokens 1.45e-7 term by term with an exponential each, 1.52e-7 with products and one sum, 1.21e-7 so.
    float pd[WITH_D ? N : 1], part[WITH_D ? N : 1];       // ds: the sum, in LDS (N / 4 places, 64 lanes apart), which 128 registers do not hold too
#pragma unroll
    for (int n = 0; n < N; n++) h[n] = 0.0f;
    if constexpr (WITH_D) {
#pragma unroll
        for (int n = 0; n < N; n++) {
            part[n] = 0.0f;
            pd[n] = 1.0f;
        }
#pragma unroll
        for (int q = 0; q < N / 4; q++) ds[q * 64] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    float wsum = 0.0f, dsum = 0.0f, d0 = 0.0f;            // Delta so far: the segment's, the window's, the window's up to the chunk
    float xh[3];                                          // raw x one, two, three tokens back in scan order
#pragma unroll
    for (int e = 0; e < 3; e++) xh[e] = w.j0 - 1 - e >= 0 ? IO::cvt(*(const T*)(w.at(w.x, max(w.j0 - 1 - e, 0)) + lo)) : 0.0f;
    // The next step's activations are requested before the current step is worked through (positions outside the sequence
    // repeat its nearest token).
    auto inside = [&](int j) { return min(max(j, 0), a.L - 1); };
    T xn[CT], dn[CT], zn[WITH_D ? CT : 1], gn[WITH_D ? CT : 1];
    const int sx = w.step(w.x), sd = w.step(w.dt), sz = w.step(w.z), sg = w.step(w.g);
    auto request = [&](int k) {
        const int first = w.j0 + k * CT;
        keep_narrow(lo);
        const char *px = w.at(w.x, inside(first)), *pd = w.at(w.dt, inside(first)), *pz = w.at(w.z, inside(first)), *pg = w.at(w.g, inside(first));
#pragma unroll
        for (int i = 0; i < CT; i++) {
            xn[i] = *(const T*)(px + lo);
            dn[i] = *(const T*)(pd + lo);
            const bool m = first + i >= 0 && first + i + 1 < a.L;
            px += m ? sx : 0; pd += m ? sd : 0;
            if constexpr (WITH_D) {
                zn[i] = *(const T*)(pz + lo);
                gn[i] = *(const T*)(pg + lo);
                pz += m ? sz : 0; pg += m ? sg : 0;
            }
        }
    };
    auto add_to_d = [&](int n, float an, float dy, float c) {
        const int i = WITH_D ? n : 0;
        pd[i] *= an;
        part[i] = fmaf(pd[i], dy * c, part[i]);
    };
    auto fold_part = [&]() {
        float sum[N];
#pragma unroll
        for (int q = 0; q < N / 4; q++) {
            const float4 v = ds[q * 64];
            sum[4 * q] = v.x; sum[4 * q + 1] = v.y; sum[4 * q + 2] = v.z; sum[4 * q + 3] = v.w;
        }
        for_each_decay<N>(w, d0, [&](int n, float p) {
            const int i = WITH_D ? n : 0;
            sum[n] = fmaf(p, part[i], sum[n]);
            part[i] = 0.0f;
            pd[i] = 1.0f;
        });
#pragma unroll
        for (int q = 0; q < N / 4; q++) ds[q * 64] = make_float4(sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]);
        d0 = dsum;
    };
    // a token's B and C, requested as soon as the values of the token before have had their last use
    // (8 x 8192 tokens of 4096 channels, the whole call 9.70 -> 9.50 ms, 4 x 771 x 1536 261 -> 257 us)
    float row[WITH_D ? 2 * N : N];
    auto request_row = [&](int j) {
        uniform_ro_ptr from = (uniform_ro_ptr)w.at(w.row, inside(j));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < (WITH_D ? 2 * N : N); n++) row[n] = from[n];
        __builtin_amdgcn_sched_barrier(0);
    };
    request(w.k0 * kSteps);
    request_row(w.j0 + w.k0 * kBwdChunk);
    float* dst = a.state + w.place(a, a.seg_chunks, w.k0) * (64 * N);
    float* dst_w = a.state_w + w.place(a, a.seg_chunks, w.k0) * 64 + w.lane;
    for (int k = w.k0 * kSteps; k < w.k1 * kSteps; k++) {
        const int first = w.j0 + k * CT;
        if (k % kSteps == 0) {
            if (w.exists) {
                store_block<N>(dst, h, w.lane);
                *dst_w = wsum;
            }
            dst += (size_t)a.tiles * 64 * N;
            dst_w += (size_t)a.tiles * 64;
            if (k == (w.k1 - 1) * kSteps && !end_wanted && !WITH_D) return;    // what is left feeds nothing
        }
        float x[CT], delta[CT];
        RawPair<IO> zg[WITH_D ? CT : 1];
#pragma unroll
        for (int i = 0; i < CT; i++) {
            x[i] = IO::cvt(xn[i]);
            delta[i] = IO::cvt(dn[i]);
            if constexpr (WITH_D) zg[i].set(zn[i], w.valid ? gn[i] : T(0));
        }
        request(min(k + 1, w.k1 * kSteps - 1));
        if (sp) {
#pragma unroll
            for (int i = 0; i < CT; i++) delta[i] = softplus(delta[i] + w.dtb);
        }
        if (first < 0 || first + CT > a.L) {              // tokens that do not exist change nothing
#pragma unroll
            for (int i = 0; i < CT; i++) {
                if (first + i < 0 || first + i >= a.L) {
                    x[i] = delta[i] = 0.0f;
                    if constexpr (WITH_D) zg[i].clear_second();
                }
            }
        }
#pragma unroll
        for (int i = 0; i < CT; i++) {
            const float pre = fmaf(w.w4[0], xh[2], fmaf(w.w4[1], xh[1], fmaf(w.w4[2], xh[0], fmaf(w.w4[3], x[i], w.cb))));
            xh[2] = xh[1]; xh[1] = xh[0]; xh[0] = x[i];
            wsum += delta[i];
            const float u = delta[i] * silu(pre);
            // (a segment that something precedes starts inside the sequence, k0 = 0, and its first three tokens are not in its window)
            const bool in_window = i >= 3 || k > 0;
            const float dy = WITH_D && in_window ? zg[WITH_D ? i : 0].second() * silu(zg[WITH_D ? i : 0].first()) : 0.0f;
            for_each_decay<N>(w, delta[i], [&](int n, float an) {
                h[n] = fmaf(an, h[n], u * row[n]);
                if constexpr (WITH_D) add_to_d(n, an, dy, row[WITH_D ? N + n : 0]);
            });
            if constexpr (!WITH_D) {
#pragma unroll
                for (int n = 0; n < N; n++) settle(h[n]);
            }
            if constexpr (WITH_D) {
#pragma unroll
                for (int n = 0; n < N; n++) {   // (a token at a time: more at once than the registers hold)
                    settle(h[n]);
                    settle(part[n]);
                    settle(pd[n]);
                }
                dsum += in_window ? delta[i] : 0.0f;
                if (i == 2 && k == 0) {
#pragma unroll
                    for (int n = 0; n < N; n++) pd[n] = 1.0f;
                }
            }
            if (WITH_D && i == CT - 1 && k % kSteps == kSteps - 1) fold_part();   // (waiting for LDS would wait for a row requested before)
            request_row(first + i + 1);
        }
    }
    if constexpr (WITH_D) {
        // the window reaches three tokens into the segments that follow
        for (int j = max(w.j1, w.j0 + 3); j < min(w.j1 + 3, a.L); j++) {
            float delta = IO::cvt(*(const T*)(w.at(w.dt, j) + lo));
            if (sp) delta = softplus(delta + w.dtb);
            const float dg = w.valid ? IO::cvt(*(const T*)(w.at(w.g, j) + lo)) : 0.0f;
            const float dy = dg * silu(IO::cvt(*(const T*)(w.at(w.z, j) + lo)));
            uniform_ro_ptr c = (uniform_ro_ptr)w.at(w.row, j) + N;
            dsum += delta;
            for_each_decay<N>(w, delta, [&](int n, float an) { add_to_d(n, an, dy, c[n]); });
        }
        fold_part();
    }
    if (w.exists) {
        store_block<N>(a.seg_h + w.place(a, 1, 0) * (64 * N), h, w.lane);
        a.seg_w[w.place(a, 1, 0) * 64 + w.lane] = wsum;
        if constexpr (WITH_D) {
            const size_t half = (size_t)2 * gridDim.z * a.nseg * a.tiles * 64;
            float* const to = a.seg_d + w.place(a, 1, 0) * (64 * N);
#pragma unroll
            for (int q = 0; q < N / 4; q++) *reinterpret_cast<float4*>(to + (q * 64 + w.lane) * 4) = ds[q * 64];
            a.seg_w[half + w.place(a, 1, 0) * 64 + w.lane] = dsum;
        }
    }
}

// grid (ceil(tiles / 2), nseg, batch), block 256: waves 0 / 1 the forward / reverse chains of one channel tile, waves
// 2 / 3 those of the next.
template <int N, typename IO>
__global__ __launch_bounds__(256, 4) void bwd_state_kernel(const BwdArgs a)
{
    __shared__ float4 sums[4][N / 4][64];   // (a lane reads what it wrote itself: no barrier)
    BwdWave<N, IO> w;
    bwd_wave_setup<N, IO>(a, w);
    if (!w.exists) return;
    float4* const ds = &sums[threadIdx.x >> 6][0][w.lane];
    const bool with_d = w.j0 > 0;   // some segment precedes this one in scan order
    if (with_d) bwd_state_walk<N, IO, true>(a, w, ds);
    else bwd_state_walk<N, IO, false>(a, w, ds);
}

// One thread per (direction, batch, tile, N / 4, lane, 4): the state entering each segment in scan order, and against
// it the dh of the tokens after each segment's window:
//   h_next = exp(A sum Delta) h + S,   D_before = exp(A sum Delta over the window) D + S_d.
// blockIdx.y: the h fold, the dh fold.  Either waits for its rounds of loads more than it computes, so they run beside each other.
template <int N>
__global__ __launch_bounds__(256) void bwd_carry_kernel(const BwdArgs a, int batch)
{
    constexpr int kAhead = 8;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long per_seg = (long long)a.tiles * 64 * N;
    if (idx >= 2 * batch * per_seg) return;
    const long long e = idx % per_seg;                    // element of one segment's blocks
    const int b = (int)(idx / per_seg % batch), s = (int)(idx / per_seg / batch);
    const int lane = (int)(e / 4 % 64), tile = (int)(e / (64 * N));
    const int n = (int)(e / 256 % (N / 4)) * 4 + (int)(e % 4);
    const float a2 = a.dir[s].A[(size_t)min(tile * 64 + lane, a.Dn - 1) * N + n] * kLog2e;
    const size_t seg0 = ((size_t)s * batch + b) * a.nseg;
    const size_t half = (size_t)2 * batch * a.nseg * a.tiles * 64;
    auto seg_of = [&](int i) { return s == 0 ? i : a.nseg - 1 - i; };   // i: scan order
    if (blockIdx.y == 0) {
        float h = 0.0f;
        for (int i0 = 0; i0 < a.nseg; i0 += kAhead) {
            float end[kAhead], sw[kAhead];
#pragma unroll
            for (int j = 0; j < kAhead; j++) {
                const size_t at = seg0 + seg_of(min(i0 + j, max(a.nseg - 2, 0)));      // nothing needs the last segment's end
                end[j] = a.seg_h[at * per_seg + e];
                sw[j] = a.seg_w[(at * a.tiles + tile) * 64 + lane];
            }
#pragma unroll
            for (int j = 0; j < kAhead; j++) {
                if (i0 + j < a.nseg) {
                    a.seg_h[(seg0 + seg_of(i0 + j)) * per_seg + e] = h;
                    h = fmaf(fast_exp2(sw[j] * a2), h, end[j]);
                }
            }
        }
        return;
    }
    float d = 0.0f;
    for (int i0 = a.nseg - 1; i0 >= 0; i0 -= kAhead) {
        float sum[kAhead], sw[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; j++) {
            const size_t at = seg0 + seg_of(max(i0 - j, min(1, a.nseg - 1)));      // nothing needs the first segment's sum
            sum[j] = a.seg_d[at * per_seg + e];
            sw[j] = a.seg_w[half + (at * a.tiles + tile) * 64 + lane];
        }
#pragma unroll
        for (int j = 0; j < kAhead; j++) {
            if (i0 - j >= 0) {
                a.seg_d[(seg0 + seg_of(i0 - j)) * per_seg + e] = d;
                d = fmaf(fast_exp2(sw[j] * a2), d, sum[j]);
            }
        }
    }
}

// What becomes of a chunk's dx, dz and dDelta: parked for the other direction, added to what it parked, or stored alone.
enum { kBwdPark = 0, kBwdAdd = 1, kBwdAlone = 2 };

// One wave's walk over its segment.  Every chunk has kBwdChunk tokens: where the sequence ends inside the last segment's
// tokens, the missing ones are walked as tokens with Delta = 0 and dout = 0, which change nothing and are not stored.
template <int N, typename IO>
struct BwdWalk {
    using T = typename IO::T;
    using Wave = BwdWave<N, IO>;
    using Walked = typename Wave::Walked;
    static constexpr int CT = kBwdChunk, LT = kBwdLdsTokens<N>;
    static constexpr int kLanesPerState = 64 / N;

    const BwdArgs& a;
    const Wave& w;
    float* const lds;
    bool sp;
    unsigned lo_t;                                       // the lane's byte offset into a row of the I/O dtype
    // What the walk writes (and fetches) token by token.  A pointer of each lane's own, moved by a row a token, is one vector
    // instruction where the row's address from its number is six scalar ones and the reading of spilled scalars: 8 x 8192 tokens
    // of 4096 channels, bf16 9531 -> 9302 us, 4 x 4096 with activations of their own for each direction 2447 -> 2372, 8 x 2048
    // with 8 states 1651 -> 1572, 2 x 500 x 700 85.9 -> 83.5.  fp32 I/O with 16 states lacks the registers (4 x 4096: 2570 ->
    // 2615, 13 spilled): from the number.
    static constexpr bool kLanePointers = N < 16 || sizeof(T) == 2;
    struct Running {
        // (a pointer to global memory by its type: past the asm below the compiler could not tell, and would use flat instructions)
        __attribute__((address_space(1))) char* at;   // the lane's place, or (wave-uniform) token 0
        int stride, step;    // bytes from a token to the next, and to the one before it in scan order
        unsigned lo;         // the lane's byte offset into a row
        __device__ __forceinline__ void start(const Wave& w, const void* base, int stride_, unsigned lo_, int j)
        {
            at = (__attribute__((address_space(1))) char*)const_cast<void*>(base);
            stride = stride_;
            step = -w.dir * stride_;
            lo = lo_;
            if constexpr (kLanePointers) {
                at += (long long)w.token(j) * stride + lo;
                opaque();
            }
        }
        __device__ __forceinline__ void opaque() { asm volatile("" : "+v"(at)); }
        __device__ __forceinline__ char* place(const Wave& w, int j)   // j: the scan position it stands at
        {
            if constexpr (kLanePointers) return (char*)at;
            keep_narrow(lo);
            return (char*)(at + (long long)w.token(j) * stride + lo);
        }
        __device__ __forceinline__ void next()
        {
            if constexpr (kLanePointers) {
                at += step;
                opaque();
            }
        }
    };
    Running odx, odz, oddt, pk, part;
    float dh[N], gA[N];
    float gD, gcb, gbias, gw[4];
    float dp1, dp2, dp3;                                 // dpre of the tokens one, two, three steps later in scan order
    float q[2][3];                                       // what the other direction parked for the next two tokens
    // the next chunk to be walked, requested half a chunk early
    T xnext[CT], dnext[CT], znext[CT], gnext[CT];
    T xbefore[3];                                        // raw x of the three tokens before it
    float hseg[N];                                       // the state entering the segment, for the next chunk
    float hnext[N], wnext;                               // the state entering it (from zero at the segment's start), and the Delta up to there

    __device__ __forceinline__ BwdWalk(const BwdArgs& a_, const Wave& w_, float* lds_) : a(a_), w(w_), lds(lds_) {}

    __device__ __forceinline__ bool carried() const { return w.j0 > 0; }   // the segment starts from a state of its own
    __device__ __forceinline__ float delta_of(float raw) const { return sp ? softplus(raw + w.dtb) : raw; }
    __device__ __forceinline__ int inside(int j) const { return min(max(j, 0), a.L - 1); }
    __device__ __forceinline__ bool exists(int j) const { return j >= 0 && j < a.L; }

    __device__ __forceinline__ void request(int k)
    {
        // (positions outside the sequence repeat its nearest token; rows as offsets from the chunk's lowest one, which the load
        // instruction adds: a scalar multiplication a row.  Seven rows of the widest token stride stay below 2^31 bytes.)
        const int first = w.j0 + k * CT;
        keep_narrow(lo_t);
#pragma unroll
        for (int e = 0; e < 3; e++) xbefore[e] = *(const T*)(w.at(w.x, inside(first - 3 + e)) + lo_t);
        const int ja = inside(first), jb = inside(first + CT - 1), low = w.dir > 0 ? ja : a.L - 1 - jb;
        auto range_of = [&](const Walked& t) { return raw_range(t.base + (long long)low * t.stride); };
        const Rsrc rx = range_of(w.x), rd = range_of(w.dt), rz = range_of(w.z), rg = range_of(w.g);
        static_assert(CT <= 8, "row offsets");
#pragma unroll
        for (int i = 0; i < CT; i++) {
            const int j = inside(first + i), row = w.dir > 0 ? j - ja : jb - j;
            xnext[i] = IO::ld_raw(rx, lo_t, row * w.x.stride);
            dnext[i] = IO::ld_raw(rd, lo_t, row * w.dt.stride);
            znext[i] = IO::ld_raw(rz, lo_t, row * w.z.stride);
            gnext[i] = IO::ld_raw(rg, lo_t, row * w.g.stride);
        }
        load_block<N>(a.state + w.place(a, a.seg_chunks, k) * (64 * N), hnext, w.lane);
        wnext = a.state_w[w.place(a, a.seg_chunks, k) * 64 + w.lane];
        __builtin_amdgcn_sched_barrier(0);                       // (not moved into the tokens that follow)
    }

    __device__ __forceinline__ void fetch_parked(float (&v)[3], const char* row)
    {
        const Parked r = *(const Parked*)row;
        v[0] = r.dx; v[1] = r.dz; v[2] = r.ddt;
    }

    // dh of the tokens after the segment's window, then the (up to) three tokens between the segment's end and there, for
    // their dpre
    __device__ __forceinline__ void start_from_next_segment()
    {
        load_block<N>(a.seg_d + w.place(a, 1, 0) * (64 * N), dh, w.lane);
        T xe[6], de[3], ze[3], ge[3];
#pragma unroll
        for (int e = 0; e < 6; e++) xe[e] = *(const T*)(w.at(w.x, inside(w.j1 - 3 + e)) + lo_t);
#pragma unroll
        for (int e = 0; e < 3; e++) {
            const int j = inside(w.j1 + e);
            de[e] = *(const T*)(w.at(w.dt, j) + lo_t);
            ze[e] = *(const T*)(w.at(w.z, j) + lo_t);
            ge[e] = *(const T*)(w.at(w.g, j) + lo_t);
        }
#pragma unroll
        for (int e = 2; e >= 0; e--) {
            if (w.j1 + e < a.L) {
                uniform_ro_ptr row = (uniform_ro_ptr)w.at(w.row, w.j1 + e);
                float pre = w.cb;
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (w.j1 + e - 3 + i >= 0) pre = fmaf(w.w4[i], IO::cvt(xe[e + i]), pre);
                const float delta = delta_of(IO::cvt(de[e]));
                const float dy = (w.valid ? IO::cvt(ge[e]) : 0.0f) * silu(IO::cvt(ze[e]));
                float dh_dot_b = 0.0f;
                for_each_decay<N>(w, delta, [&](int n, float an) {
                    dh[n] = fmaf(row[N + n], dy, dh[n]);
                    dh_dot_b = fmaf(dh[n], row[n], dh_dot_b);
                    dh[n] *= an;
                });
                dp3 = dp2; dp2 = dp1;
                dp1 = fmaf(w.dval, dy, dh_dot_b * delta) * dsilu(pre);
            }
        }
    }

    template <int MODE>
    __device__ __forceinline__ void chunk(int k)
    {
        const int first = w.j0 + k * CT;                            // scan position of the chunk's first token
        // B and C rows are requested ahead into scalar registers, where the values they replace have had their last use: a
        // token's B while the token before is worked through, then, going back, B and C of the next token once this one's dh and
        // their products stand.  (Where a token asked for its own rows it waited: 8 x 8192 tokens of 4096 channels 10.44 ->
        // 9.70 ms, 4 x 771 x 1536 281 -> 261 us.)
        float rows[2][N];                                           // forwards: B of this token and the next; backwards: B, C
        auto request_row = [&](float (&to)[N], int j, int half) {
            uniform_ro_ptr from = (uniform_ro_ptr)w.at(w.row, inside(j)) + half * N;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < N; n++) to[n] = from[n];
            __builtin_amdgcn_sched_barrier(0);
        };
        request_row(rows[0], first, 0);
        // x and Delta, z and dout of the chunk's tokens; xd[0 .. 2]: x of the three tokens before it
        RawPair<IO> xd[CT + 3], zg[CT];
#pragma unroll
        for (int e = 0; e < 3; e++) xd[e].set(xbefore[e], T(0));
#pragma unroll
        for (int i = 0; i < CT; i++) {
            xd[i + 3].set(xnext[i], dnext[i]);
            zg[i].set(znext[i], w.valid ? gnext[i] : T(0));         // (shadow lanes add nothing to the sums below)
        }
        const bool at_an_end = first < 3 || first + CT > a.L;
        if (at_an_end) {
#pragma unroll
            for (int e = 0; e < CT + 3; e++)
                if (!exists(first - 3 + e)) {
                    xd[e].clear_first();
                    if (e >= 3) zg[e >= 3 ? e - 3 : 0].clear_second();
                }
        }
        // the state entering the chunk: the stored one plus what is left of the state entering the segment
        float h[N];
#pragma unroll
        for (int n = 0; n < N; n++) h[n] = hnext[n];
        if (carried()) {
            for_each_decay<N>(w, wnext, [&](int n, float c) { h[n] = fmaf(c, hseg[n], h[n]); });
        }
        float delta[CT], xc[CT], sig[CT];   // Delta, conv + SiLU output, sigmoid of the conv output
#pragma unroll
        for (int i = 0; i < CT; i++) delta[i] = xd[i + 3].second();
        if (sp) {
#pragma unroll
            for (int i = 0; i < CT; i++) delta[i] = softplus(delta[i] + w.dtb);
        }
        if (at_an_end) {
#pragma unroll
            for (int i = 0; i < CT; i++) delta[i] = exists(first + i) ? delta[i] : 0.0f;
        }
        // forward over the chunk, keeping every state: hs[i] enters token i; those of the first LT tokens wait in LDS
        float hs[CT + 1][N];
        {
            float x1 = xd[2].first(), x2 = xd[1].first(), x3 = xd[0].first();
#pragma unroll
            for (int i = 0; i < CT; i++) {
                if (i < LT) store_block<N>(lds + i * 64 * N, h, w.lane);
                else {
#pragma unroll
                    for (int n = 0; n < N; n++) hs[i][n] = h[n];
                }
                const float x0 = xd[i + 3].first();
                const float pre = fmaf(w.w4[0], x3, fmaf(w.w4[1], x2, fmaf(w.w4[2], x1, fmaf(w.w4[3], x0, w.cb))));
                x3 = x2; x2 = x1; x1 = x0;
                sig[i] = sigmoidf(pre);
                xc[i] = pre * sig[i];
                const float u = delta[i] * xc[i];
                // (scalar loads return in any order, so waiting for one waits for all: this token's row first, then the next request.
                // Of an even number of tokens the last one's B is in rows[1], its C goes to rows[0].)
                asm volatile("" ::"s"(rows[i & 1][0]), "s"(rows[i & 1][N - 1]));
                request_row(rows[(i + 1) & 1], first + min(i + 1, CT - 1), i + 1 < CT ? 0 : 1);
                for_each_decay<N>(w, delta[i], [&](int n, float an) { h[n] = fmaf(an, h[n], u * rows[i & 1][n]); });
            }
        }
        static_assert(CT % 2 == 0, "the chunk's last B row is expected in rows[1]");
        float (&row_b)[N] = rows[1], (&row_c)[N] = rows[0];
#pragma unroll
        for (int n = 0; n < N; n++) hs[CT][n] = h[n];
        // backward over the chunk, last token first; xw: x of the token at hand and the three before it
        float xw[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            xd[CT - 1 + e].opaque();
            xw[e] = xd[CT - 1 + e].first();
        }
#pragma unroll
        for (int i = CT - 1; i >= 0; i--) {
            const int j = first + i;
            const bool there = exists(j);
            // Half way through the walk the states of the chunk's later tokens are dead: their registers take the
            // next chunk, its entering state and the three x before it.  (Also after the last chunk, when nothing uses it:
            // under a condition the old values would stay live beside the states.)
            if (i == CT / 2 - 1) request(max(k - 1, w.k0));
            // (asked for here: where the chunk that uses it asked, it waited; its registers are free only now.  Unused where nothing
            // precedes the segment.)
            if (i == 0) load_block<N>(a.seg_h + w.place(a, 1, 0) * (64 * N), hseg, w.lane);
            if (i < LT) load_block<N>(lds + i * 64 * N, hs[i], w.lane);
            float y = w.dval * xc[i];
#pragma unroll
            for (int n = 0; n < N; n++) y = fmaf(row_c[n], hs[i + 1][n], y);
            const float zv = zg[i].first(), dg = zg[i].second();
            const float z_sig = sigmoidf(zv), z_silu = zv * z_sig;
            float dzv = dg * y * fmaf(z_silu, 1.0f - z_sig, z_sig);
            settle(dzv);
            const float dy = dg * z_silu;
            gD = fmaf(dy, xc[i], gD);
            const float u = delta[i] * xc[i];
            // this channel's terms of dC_t, summed over the wave's channels: value n in lanes n * kLanesPerState ...
            float terms[N];
#pragma unroll
            for (int n = 0; n < N; n++) terms[n] = hs[i + 1][n];
            float dc_total = wave_reduce_scatter<N>(terms, dy);
            settle(dc_total);
            // (formed again: kept from the forward half, a chunk's decays would take as many registers as its states)
            float dlt = delta[i];
            asm volatile("" : "+v"(dlt));
            // sum_n dh[n] B[n] serves both dDelta (times xc) and dxc (times Delta); sum_n (dh h_prev a)[n] a2[n] is
            // dDelta's decay part up to the factor ln 2 (A = a2 ln 2)
            // (both in two halves: shorter chains, fewer roundings on the way)
            float dot[2] = {0.0f, 0.0f}, decay[2] = {0.0f, 0.0f};
#pragma unroll
            for (int n = 0; n < N; n++) {
                dh[n] = fmaf(row_c[n], dy, dh[n]);
                dot[n & 1] = fmaf(dh[n], row_b[n], dot[n & 1]);
            }
            if (i > 0) {
                request_row(row_c, j - 1, 1);
                request_row(row_b, j - 1, 0);
            }
            for_each_decay<N>(w, dlt, [&](int n, float an) {
                terms[n] = dh[n];                                    // of dB_t, times u
                dh[n] *= an;
                const float da = dh[n] * hs[i][n];                   // dh * a * h_prev
                gA[n] = fmaf(da, dlt, gA[n]);
                decay[n & 1] = fmaf(da, w.a2[n], decay[n & 1]);
            });
            const float dh_dot_b = dot[0] + dot[1], decay_part = decay[0] + decay[1];
#pragma unroll
            for (int n = 0; n < N; n++) {
                settle(gA[n]);
                settle(dh[n]);
            }
            float ddt = fmaf(decay_part, kLn2, dh_dot_b * xc[i]);
            float dxc = fmaf(w.dval, dy, dh_dot_b * dlt);
            settle(ddt);
            settle(dxc);
            settle(gD);
            {
                // the two totals of a state side by side: the first half of its lanes has dB_t[n], the second dC_t[n]
                const float db_total = wave_reduce_scatter<N>(terms, u);
                const bool second = (w.lane & (kLanesPerState / 2)) != 0;
                if (there && w.exists && w.lane % (kLanesPerState / 2) == 0) *(float*)part.place(w, j) = second ? dc_total : db_total;
                part.next();
            }
            if (sp) {
                ddt *= sigmoidf(xd[i + 3].second() + w.dtb);
                gbias += there ? ddt : 0.0f;
            }
            const float dpre = dxc * fmaf(xc[i], 1.0f - sig[i], sig[i]);
            gcb += dpre;
#pragma unroll
            for (int e = 0; e < 4; e++) gw[e] = fmaf(dpre, xw[e], gw[e]);
            float dxv = fmaf(w.w4[3], dpre, fmaf(w.w4[2], dp1, fmaf(w.w4[1], dp2, w.w4[0] * dp3)));
            settle(dxv);
            settle(gcb);
#pragma unroll
            for (int e = 0; e < 4; e++) settle(gw[e]);
            dp3 = dp2; dp2 = dp1; dp1 = dpre;
            xw[3] = xw[2]; xw[2] = xw[1]; xw[1] = xw[0];
            if (i > 0) {
                xd[i - 1].opaque();
                xw[0] = xd[i - 1].first();
            }
            if constexpr (MODE == kBwdAdd) {
                dxv += q[i & 1][0]; dzv += q[i & 1][1]; ddt += q[i & 1][2];
                fetch_parked(q[i & 1], pk.place(w, j - 2));   // (the buffer has rows to spare on both sides)
            }
            if (there && w.valid) {
                if constexpr (MODE == kBwdPark) {
                    *(Parked*)pk.place(w, j) = Parked{dxv, dzv, ddt};
                } else {
                    IO::st((T*)odx.place(w, j), dxv);
                    IO::st((T*)odz.place(w, j), dzv);
                    IO::st((T*)oddt.place(w, j), ddt);
                }
            }
            if constexpr (MODE != kBwdAlone) pk.next();
            if constexpr (MODE != kBwdPark) { odx.next(); odz.next(); oddt.next(); }
            // (convergent: keeps the compiler from copying the loop's exit test into both sides of the branch above, which
            // would make the loop counter, and with it every row address, a per-lane value)
            __builtin_amdgcn_wave_barrier();
        }
    }

    template <int MODE>
    __device__ __forceinline__ void chunks(int from, int to)   // from, from - 1 ... to
    {
        for (int k = from; k >= to; k--) chunk<MODE>(k);
    }

    __device__ __forceinline__ void run()
    {
        sp = a.dt_softplus != 0;
        lo_t = (unsigned)(w.ch * sizeof(T));
        auto park_from = [&](int j) { pk.start(w, a.parked + (size_t)w.b * a.L * a.Dn, a.Dn * (int)sizeof(Parked), (unsigned)(w.ch * sizeof(Parked)), j); };
        auto store_from = [&](int j) {
            auto view = [&](Running& r, const TensorArg& t) { r.start(w, (const char*)t.p + (size_t)w.b * t.sb * sizeof(T), (int)(t.st * (long long)sizeof(T)), lo_t, j); };
            view(odx, a.gdx[w.s]);
            view(odz, a.gdz[w.s]);
            view(oddt, a.gddt[w.s]);
        };
        const int last = w.j0 + w.k1 * CT - 1;          // the walk's first token, which the sequence may not reach
        // this wave's slot of the dB and dC partial sums: [batch][L][G][slots][N][2]
        const int tiles_per_group = (a.Dn / a.G + 63) / 64;
        const int slot = __builtin_amdgcn_readfirstlane(w.tile % tiles_per_group) + (w.s == 1 ? a.bc_slot_of_rev : 0);
        part.start(w, (a.bc_part[w.s] + (((size_t)w.b * a.L * a.G + w.grp) * a.bc_slots + slot) * (2 * N)),
                   a.G * a.bc_slots * 2 * N * (int)sizeof(float), (unsigned)(w.lane / (kLanesPerState / 2) * sizeof(float)), last);
#pragma unroll
        for (int n = 0; n < N; n++) dh[n] = gA[n] = 0.0f;
        gD = gcb = gbias = dp1 = dp2 = dp3 = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; e++) gw[e] = 0.0f;
        if (w.j1 < a.L) start_from_next_segment();
        if (!a.park) {
            store_from(last);
            request(w.k1 - 1);
            load_block<N>(a.seg_h + w.place(a, 1, 0) * (64 * N), hseg, w.lane);
            chunks<kBwdAlone>(w.k1 - 1, w.k0);
        } else {
            // The two waves of a tile walk the segment's tokens in opposite orders.  The forward direction's wave parks the
            // later half, the reverse one's the earlier half; the barrier is a workgroup-scope release / acquire: past it,
            // what the other wave parked is visible.  It is fetched two tokens ahead.
            const int to = w.s == 0 ? a.seg_chunks / 2 : a.seg_chunks - a.seg_chunks / 2;
            park_from(last);
            request(w.k1 - 1);
            load_block<N>(a.seg_h + w.place(a, 1, 0) * (64 * N), hseg, w.lane);
            chunks<kBwdPark>(w.k1 - 1, max(to, w.k0));
            __syncthreads();
            const int from = min(to, w.k1) - 1, j = w.j0 + from * CT + CT - 1;
            if (from >= w.k0) {
                park_from(j);
                fetch_parked(q[1], pk.place(w, j));
                pk.next();
                fetch_parked(q[0], pk.place(w, j - 1));
                pk.next();
                store_from(j);
            }
            chunks<kBwdAdd>(from, w.k0);
        }
        if (w.exists) {
            // this segment's share of the parameter gradients: rows dA[0..N), dD, dconv_w[4] (w[3] on the current token), dconv_b, ddt_bias
            const size_t pitch = (size_t)a.tiles * 64;
            float* dst = a.param_part + ((((size_t)w.s * gridDim.z + w.b) * a.nseg + w.seg) * (N + kBwdParams)) * pitch + w.tile * 64 + w.lane;
#pragma unroll
            for (int n = 0; n < N; n++) dst[n * pitch] = gA[n];
            dst[N * pitch] = gD;
#pragma unroll
            for (int i = 0; i < 4; i++) dst[(N + 1 + i) * pitch] = gw[i];
            dst[(N + 5) * pitch] = gcb;
            dst[(N + 6) * pitch] = gbias;
        }
    }
};

template <int N, typename IO>
__global__ __launch_bounds__(256, 2) void bwd_kernel(const BwdArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds_all[];   // kBwdLdsBytes<N>
    BwdWave<N, IO> w;
    bwd_wave_setup<N, IO>(a, w);
    // (a wave without a tile of its own still runs, as a shadow of its neighbour: the meeting barrier counts four waves)
    float* lds = lds_all + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * (kBwdLdsTokens<N> * 64 * N);
    BwdWalk<N, IO>(a, w, lds).run();
}

// Prepared fp32 B | C rows of one or two sets of activations (prep_bc_kernel without the conv), both in one launch.
struct BwdPrepArgs {
    TensorArg B[2], C[2];
    float* dst[2];       // [batch][L][G][2N]
    int L, G, N;
    long long per_set;   // batch * L * G * 2N
};

// What the walk left in slots, added in a fixed order: dB and dC from the per-wave partial sums (one thread per (batch,
// token, group, value)), then the parameter gradients from the per-segment ones.
struct BwdSumArgs {
    const float* part[2];   // per set of activations: [batch][L][G][slots][N][2]
    float* dB[2];           // [batch][L][G][N]
    float* dC[2];
    int sets, slots, N;
    long long rows;         // batch * L * G
    const float* param_part;   // [2][segs][N + 7][pitch]
    long long pitch;
    int segs;               // batch * nseg (0: the gradients are zero)
    float* dA[2];
    float* dD[2];
    float* dconv_w[2];
    float* dconv_b[2];      // or null
    float* ddt_bias[2];     // or null
    int Dn, K;
};

}  // namespace bm
