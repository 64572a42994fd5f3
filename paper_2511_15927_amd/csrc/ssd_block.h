// Mamba-2 calls of up to 64 tokens (block-diffusion steps), both directions, without a barrier between the phases of a wave.
//
// Such a call is 1500 vector instructions and 46 KB of memory traffic an item (batch, head) at 32 tokens of 64 channels: what it
// costs is the length of its chains of loads and phases.  Here a wave owns 16 channels over the whole block and does all phases
// for them: it requests everything it reads at its start, scans Delta (both directions in one pass over the two halves of the wave at
// 32 tokens), forms the masked, decayed score operands, the conv + SiLU of its channels right in operand layout and the bf16 operand
// of its entry state, and multiplies.  Four waves share x, z and the output, which cross global memory in whole rows of 64 channels
// through LDS, and the score operands of a head, made by its waves in shares (with 2-byte accesses and operands of each wave's own
// a call of 16 x 32 tokens, 64 heads x 64, 128 states took 26.2 us, most of it address and tag cycles; 18.8 then, the bytes alone
// 9).  (Before: a workgroup an item with producer and consumer waves, one direction after the other, 39.9.)
//
// The operands that all heads of a group share (scores, C, B^T) are 4350 vector instructions a batch element at 32 tokens.  Where
// the chip holds the call at once, workgroups of sixteen waves make them for themselves (WHOLE), while the state and x that the
// waves have requested are on their way: a launch of one workgroup per (direction, group, batch element) before the walk
// (ssd_block_prep_kernel) costs 5 us whatever it does.  16 x 32 tokens of 64 heads x 64 18.7 -> 16.2 us, 1 x 32 10.8 -> 8.0, with
// state and tail committed to places of their own 23.7 -> 20.4 and 13.9 -> 9.2.  (Committed in place, as a decode loop does, the tail of
// B and C takes a launch of its own behind, 11.4 for the second call; calls with four tiles a workgroup, the first one, keep to two
// launches then, 23.4.)  So do longer blocks and calls of more workgroups.
//
// The barriers of the walk are those of the sharing: the first before the convs, which read x and the score operands that all four
// waves have put into LDS; the last before the output's rows are read back from the y columns that the waves have left there.  With
// more than 32 tokens y lies over x and the operands, and one more orders their last reads before it.
//
// Both directions work in token order: the reverse direction's operands hold j >= i.  MFMA 16x16x32: operand A lane l holds row
// l%16, B column l%16, eight contraction slots of group g = l/16; accumulator register r of lane l is row 4g + r, column l%16.
// Positions fill the slots of a 32-token block in order (slot e of group g is token 8g + e: a lane convolves a run of eight);
// states as 4t + e of group g = state 16t + 4g + e, the accumulator's own order, so that the state loaded once (16-byte
// pieces) is both operand and accumulator of the update.  The skip term's xc in accumulator layout is a product with the
// identity, which is exact.
#pragma once
#include "ssd_kernels.h"

namespace bm {

struct SsdBlockDir {
    TensorArg x, z, dt, B, C;
    const float *conv_w, *conv_b, *A, *D, *dt_bias;
};

struct SsdBlockArgs {
    SsdBlockDir dir[2];   // forward, reverse
    // operands shared by the heads of a group, per (batch, group): C of the forward direction [32 states][16 rows][lane][8], its
    // B^T [16 states][32 tokens][lane][8], both directions' scores [32 x 32 block][16 rows][lane][8]
    __bf16 *c_op, *b_op;
    float* score[2];
    void* out;
    long long out_sb, out_st;
    const float* h_in;    // [batch][Dn][N] or null
    float* h_out;         // or null; may alias h_in
    const void* tail_in;  // bf16 [batch][K-1][tail_ch] or null
    void* tail_out;       // or null; may alias tail_in: x's part is written by whoever reads it there, B's and C's by the preparation, or, in
                          // one launch that commits the state, by a group's first workgroup (there not aliasing, since every workgroup of the
                          // group reads it; a launch that does not commit the state writes no part of B and C)
    int batch, L, Dn, H, P, HG, G, K, tail_ch;
    int dt_softplus, d_per_head, conv_bc, separate;
    int shared;           // both directions read the same x and the same z
    int tiles;            // one launch: 64-channel tiles of a workgroup
};

// Eight channels of one token.
typedef unsigned __attribute__((ext_vector_type(4), aligned(2))) Piece;

// 32 x 32 score blocks of a call: the causal (forward) or anti-causal (reverse) ones of BLOCKS x BLOCKS.
template <int BLOCKS>
constexpr int ssd_block_scores() { return BLOCKS == 1 ? 1 : 3; }

template <int N, int BLOCKS>
constexpr size_t ssd_block_prep_lds() { return 2 * (size_t)(32 * BLOCKS) * (N + 1) * sizeof(float) + 12 * 64 * 4 * sizeof(float); }

// grid (G, 2, batch), block 1024, dynamic LDS ssd_block_prep_lds<N, BLOCKS>().  B and C of one direction after conv + SiLU as fp32
// in LDS, then the operands.  Scores are formed as in ssd_prep_kernel: operands split into a bf16 head and remainder, three products.
template <int N, int BLOCKS>
__global__ __launch_bounds__(1024) void ssd_block_prep_kernel(const SsdBlockArgs a)
{
    using T = unsigned short;
    constexpr int kTok = 32 * BLOCKS;
    extern __shared__ __attribute__((aligned(16))) unsigned char ssd_block_lds[];
    float(*sB)[N + 1] = reinterpret_cast<float(*)[N + 1]>(ssd_block_lds);
    float(*sC)[N + 1] = sB + kTok;
    float* const sums = reinterpret_cast<float*>(sC + kTok);   // [12][64][4]
    const int g = blockIdx.x, s = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, last = a.L - 1;
    const SsdBlockDir& d = a.dir[s];
    {
        constexpr int kCols = 2 * N, kParts = 1024 / kCols, kLen = kTok / kParts;
        const int col = tid % kCols, part = tid / kCols;   // one column of B|C, tokens part*kLen ..
        const int which = col / N, n = col % N;
        const TensorArg& src = which ? d.C : d.B;
        const T* base = (const T*)src.p + (size_t)b * src.sb + g * N + n;
        const int row = a.Dn + which * a.G * N + g * N + n;   // this column's conv channel
        const int t0 = part * kLen - (s == 0 ? 3 : 0);        // first token of the run and its halo (behind it in scan order)
        T raw[kLen + 3];
#pragma unroll
        for (int q = 0; q < kLen + 3; q++) raw[q] = base[(long long)min(max(t0 + q, 0), last) * src.st];
        float w4[4] = {0.0f, 0.0f, 0.0f, 0.0f}, bias = 0.0f;   // w4[3] on the current position
        if (a.conv_bc) {
            load_taps(d.conv_w + (size_t)row * a.K, a.K, w4);
            bias = d.conv_b ? d.conv_b[row] : 0.0f;
        }
        float xr[kLen + 3];
#pragma unroll
        for (int q = 0; q < kLen + 3; q++) xr[q] = (t0 + q >= 0 && t0 + q <= last) ? IoBF16::cvt(raw[q]) : 0.0f;
        if (s == 0 && part == 0 && a.tail_in && a.conv_bc && a.K > 1) {
            T cached[3];
#pragma unroll
            for (int q = 0; q < 3; q++)   // 3 - q tokens before the block, from clamped rows (a tap beyond the conv width has a zero weight)
                cached[q] = ((const T*)a.tail_in)[((size_t)b * (a.K - 1) + max(a.K - 1 - (3 - q), 0)) * a.tail_ch + row];
#pragma unroll
            for (int q = 0; q < 3; q++)
                if (3 - q <= a.K - 1) xr[q] = IoBF16::cvt(cached[q]);
        }
        if (s == 0 && part == 0 && a.tail_out && a.conv_bc) {   // the last K - 1 raw tokens of (tail_in || block)
            T last_raw[3];
#pragma unroll
            for (int q = 0; q < 3; q++) last_raw[q] = base[(long long)max(a.L - 3 + q, 0) * src.st];
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const int n_out = q - 3 + (a.K - 1), pos = a.L - 3 + q;   // row of the tail, token of the block (negative: of tail_in)
                T v = last_raw[q];
                if (pos < 0) {   // (xr[0 .. 2] hold the tokens before the block)
                    v = 0;
#pragma unroll
                    for (int e = 0; e < 3; e++)
                        if (pos + 3 == e) v = io_bits<IoBF16>(xr[e]);
                }
                if (n_out >= 0) ((T*)a.tail_out)[((size_t)b * (a.K - 1) + n_out) * a.tail_ch + row] = v;
            }
        }
        float(*dst)[N + 1] = which ? sC : sB;
#pragma unroll
        for (int i = 0; i < kLen; i++) {
            const int t = part * kLen + i;
            float v = xr[s == 0 ? i + 3 : i];
            if (a.conv_bc) {
                float pre = bias;
#pragma unroll
                for (int k = 0; k < 4; k++) pre = fmaf(w4[k], xr[s == 0 ? i + k : i + 3 - k], pre);
                v = silu(pre);
            }
            dst[t][n] = t > last ? 0.0f : v;
        }
    }
    __syncthreads();
    const size_t item = (size_t)b * a.G + g;
    if (s == 0 && a.h_in) {
        for (int idx = tid; idx < kTok * N / 8; idx += 1024) {
            const int ln = idx % 64, f = idx / 64, i = (f % (2 * BLOCKS)) * 16 + ln % 16, n0 = (f / (2 * BLOCKS)) * 32 + 4 * (ln / 16);
            bf16x8 v;
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = (__bf16)sC[i][n0 + 16 * (e / 4) + e % 4];
            *reinterpret_cast<bf16x8*>(&a.c_op[(item * (kTok * N / 8) + idx) * 8]) = v;
        }
    }
    if (s == 0 && a.h_out) {
        for (int idx = tid; idx < kTok * N / 8; idx += 1024) {
            const int ln = idx % 64, f = idx / 64, n = (f / BLOCKS) * 16 + ln % 16, j0 = (f % BLOCKS) * 32 + 8 * (ln / 16);
            bf16x8 v;
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = (__bf16)sB[j0 + e][n];
            *reinterpret_cast<bf16x8*>(&a.b_op[(item * (kTok * N / 8) + idx) * 8]) = v;
        }
    }
    // 16 x 16 tiles (rows j, columns i): at 32 tokens four waves share a tile's contraction and add up through LDS
    const int wave = tid / 64, lane = tid % 64, g4 = lane / 16, c16 = lane % 16;
    constexpr int kSplit = BLOCKS == 1 ? 4 : 1, kSteps = N / 32 / kSplit > 0 ? N / 32 / kSplit : 1;
    const int tile = wave / kSplit, kpart = wave % kSplit;
    const int it = tile / (2 * BLOCKS), jt = tile % (2 * BLOCKS);
    const bool wanted = s == 0 ? jt / 2 <= it / 2 : jt / 2 >= it / 2;   // of a 32 x 32 block that is kept
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    if (wanted && kpart * kSteps < N / 32) {
#pragma unroll
        for (int ks = 0; ks < kSteps; ks++) {
            const int k0 = (kpart * kSteps + ks) * 32 + 8 * g4;
            bf16x8 ah, al, bh, bl;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const float bv = sB[jt * 16 + c16][k0 + e], cv = sC[it * 16 + c16][k0 + e];
                ah[e] = (__bf16)bv;
                al[e] = (__bf16)(bv - (float)ah[e]);
                bh[e] = (__bf16)cv;
                bl[e] = (__bf16)(cv - (float)bh[e]);
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
        }
    }
    if constexpr (kSplit > 1) {
        const int slot = tile * 3 + kpart - 1;
        if (kpart > 0) *reinterpret_cast<f32x4*>(&sums[(slot * 64 + lane) * 4]) = acc;
        __syncthreads();
        if (kpart > 0) return;
#pragma unroll
        for (int o = 0; o < 3; o++) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(&sums[((tile * 3 + o) * 64 + lane) * 4]);
#pragma unroll
            for (int r = 0; r < 4; r++) acc[r] += v[r];
        }
    }
    if (!wanted) return;
    const int i = it * 16 + c16, j0 = jt * 16 + 4 * g4;
#pragma unroll
    for (int r = 0; r < 4; r++)
        if (s == 0 ? j0 + r > i : j0 + r < i) acc[r] = 0.0f;
    // block (i, j) of the kept ones: forward (0,0), (1,0), (1,1); reverse (0,0), (0,1), (1,1)
    const int block = it / 2 + jt / 2;
    float* const dst = a.score[s] + item * (ssd_block_scores<BLOCKS>() * 1024) +
                       ((block * 2 + it % 2) * 64 + (2 * (jt % 2) + g4 / 2) * 16 + c16) * 8 + 4 * (g4 % 2);
    *reinterpret_cast<f32x4*>(dst) = acc;
}

// Prefix sums inside the two halves of a wave.
__device__ __forceinline__ float half_wave_inclusive_sum(float v)
{
#define BM_DPP_ADD(ctrl, rows) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xF, false))
    BM_DPP_ADD(0x111, 0xF);
    BM_DPP_ADD(0x112, 0xF);
    BM_DPP_ADD(0x114, 0xF);
    BM_DPP_ADD(0x118, 0xF);
    BM_DPP_ADD(0x142, 0xA);
#undef BM_DPP_ADD
    return v;
}
__device__ __forceinline__ float lane_value(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }

// One launch (up to 32 tokens): LDS of ssd_block_kernel<.., WHOLE>.  B and C rows of both directions as bf16 head and rest, over
// which the outputs lie once the operands have been made; scores; B^T of the forward direction; then the tiles' own parts.
template <int N, bool COMMIT, bool SHARED>
struct SsdBlockLds {
    static constexpr int kRow = N + kPrepPad;
    static constexpr size_t kSplit = 2 * 4 * 32 * (size_t)kRow * sizeof(__bf16), kY = 2 * 32 * 68 * sizeof(float);
    static constexpr size_t kScore = 2 * 1024 * sizeof(float), kBt = COMMIT ? 32 * (size_t)N * sizeof(__bf16) : 0;
    static constexpr size_t kTab = 4 * 6 * 32 * sizeof(float), kX = (SHARED ? 1 : 2) * 38 * 68 * sizeof(unsigned short), kM = 2 * 4 * 64 * 16;
    static constexpr size_t kTile = kTab + kX + kM;
    static constexpr size_t front(int tiles) { return kSplit > tiles * kY ? kSplit : tiles * kY; }
    static constexpr size_t bytes(int tiles) { return front(tiles) + kScore + kBt + tiles * kTile; }
};

// B and C of one (group, batch element) after conv + SiLU, both directions, from the first 8 N threads of the workgroup: two columns
// and eight tokens a thread, as in ssd_prep_kernel but in token order.  split[direction][B head, B rest, C head, C rest][token].
template <int N, bool COMMIT>
struct SsdBlockRows {
    using T = unsigned short;
    int s, part, n, which, row, last, t0;   // direction, run of eight tokens, first column of B or C, its conv channel
    bf16_pair raw[11];
    float w4[2][4], bias[2];                // w4[.][3] on the current position
    bool from_tail, writes_tail;

    __device__ __forceinline__ void request(const SsdBlockArgs& a, int g, int b, int tid, bool tail_writer)
    {
        s = __builtin_amdgcn_readfirstlane(tid / (4 * N));
        part = __builtin_amdgcn_readfirstlane(tid / N % 4);
        n = 2 * (tid % (N / 2));
        last = a.L - 1;
        which = tid % N / (N / 2);
        if constexpr (N == 128) which = __builtin_amdgcn_readfirstlane(which);
        const SsdBlockDir& d = a.dir[s];
        const TensorArg& src = which ? d.C : d.B;
        const T* const base = (const T*)src.p + (size_t)b * src.sb + g * N + n;
        row = a.Dn + which * a.G * N + g * N + n;
        t0 = part * 8 - (s == 0 ? 3 : 0);   // first token of the run and its halo (behind it in scan order)
#pragma unroll
        for (int q = 0; q < 11; q++) raw[q] = *(const bf16_pair*)(base + (long long)min(max(t0 + q, 0), last) * src.st);
        const bool before = s == 0 && part == 0 && a.conv_bc && a.K > 1;
        from_tail = before && a.tail_in;
        if (from_tail) {
#pragma unroll
            for (int q = 0; q < 3; q++)   // 3 - q tokens before the block, from clamped rows (a tap beyond the conv width has a zero weight)
                raw[q] = *(const bf16_pair*)((const T*)a.tail_in + ((size_t)b * (a.K - 1) + max(a.K - 1 - (3 - q), 0)) * a.tail_ch + row);
        }
        writes_tail = COMMIT && before && tail_writer && a.tail_out;
        if (a.conv_bc) {
#pragma unroll
            for (int k = 0; k < 2; k++) {
                load_taps(d.conv_w + (size_t)(row + k) * a.K, a.K, w4[k]);
                bias[k] = d.conv_b ? d.conv_b[row + k] : 0.0f;
            }
        }
    }

    __device__ __forceinline__ float column(int q, int k) const { return __uint_as_float(k ? raw[q] & 0xffff0000u : raw[q] << 16); }

    template <bool CONV, bool REVERSE>
    __device__ __forceinline__ void rows(__bf16 (*const split)[4][32][N + kPrepPad], bf16x8* const bt)
    {
        bf16x8 piece[2];
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int t = part * 8 + i;
            __bf16 head[2], rest[2];
#pragma unroll
            for (int k = 0; k < 2; k++) {
                float v = column(REVERSE ? i : i + 3, k);
                if constexpr (CONV) {
                    float pre = bias[k];
#pragma unroll
                    for (int w = 0; w < 4; w++) pre = fmaf(w4[k][w], column(REVERSE ? i + 3 - w : i + w, k), pre);
                    v = silu(pre);
                }
                v = t <= last ? v : 0.0f;
                head[k] = (__bf16)v;
                rest[k] = (__bf16)(v - (float)head[k]);
                piece[k][i] = head[k];
            }
            *reinterpret_cast<bf16x2*>(&split[s][2 * which][t][n]) = bf16x2{head[0], head[1]};
            *reinterpret_cast<bf16x2*>(&split[s][2 * which + 1][t][n]) = bf16x2{rest[0], rest[1]};
        }
        if constexpr (COMMIT && !REVERSE) {   // B^T as the state update takes it: [16 states][lane][8]
            if (which == 0)
#pragma unroll
                for (int k = 0; k < 2; k++) bt[(n / 16) * 64 + part * 16 + n % 16 + k] = piece[k];
        }
    }

    __device__ __forceinline__ void finish(const SsdBlockArgs& a, int b, __bf16 (*const split)[4][32][N + kPrepPad], bf16x8* const bt)
    {
#pragma unroll
        for (int q = 0; q < 11; q++) {
            const bool there = (t0 + q >= 0 || (from_tail && 3 - q <= a.K - 1)) && t0 + q <= last;
            raw[q] = there ? raw[q] : 0u;
        }
        if (writes_tail) {   // the last K - 1 raw tokens of (tail_in || block)
            const SsdBlockDir& d = a.dir[0];
            const TensorArg& src = which ? d.C : d.B;
            const T* const base = (const T*)src.p + (size_t)b * src.sb + (row - a.Dn - which * a.G * N);
            bf16_pair end_raw[3];
#pragma unroll
            for (int q = 0; q < 3; q++) end_raw[q] = *(const bf16_pair*)(base + (long long)max(a.L - 3 + q, 0) * src.st);
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const int n_out = q - 3 + (a.K - 1), pos = a.L - 3 + q;   // row of the tail, token of the block (negative: before it)
                bf16_pair v = end_raw[q];
#pragma unroll
                for (int e = 0; e < 3; e++)
                    if (pos + 3 == e) v = raw[e];
                if (n_out >= 0) *(bf16_pair*)((T*)a.tail_out + ((size_t)b * (a.K - 1) + n_out) * a.tail_ch + row) = v;
            }
        }
        if (s == 0) a.conv_bc ? rows<true, false>(split, bt) : rows<false, false>(split, bt);
        else a.conv_bc ? rows<true, true>(split, bt) : rows<false, true>(split, bt);
    }
};

// Scores of both directions, a 16 x 16 tile a wave (eight waves): [direction][16 rows i][lane][8], zero where they are masked.
template <int N>
__device__ __forceinline__ void ssd_block_scores_of(int wave, int lane, const __bf16 (*const split)[4][32][N + kPrepPad], float* score)
{
    const int s = wave / 4, it = wave % 4 / 2, jt = wave % 2, g4 = lane / 16, c16 = lane % 16;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    if (s == 0 ? jt <= it : jt >= it) {
#pragma unroll
        for (int ks = 0; ks < N / 32; ks++) {
            const int k0 = ks * 32 + 8 * g4;
            const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&split[s][0][jt * 16 + c16][k0]), al = *reinterpret_cast<const bf16x8*>(&split[s][1][jt * 16 + c16][k0]);
            const bf16x8 bh = *reinterpret_cast<const bf16x8*>(&split[s][2][it * 16 + c16][k0]), bl = *reinterpret_cast<const bf16x8*>(&split[s][3][it * 16 + c16][k0]);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
        }
    }
    const int i = it * 16 + c16, j0 = jt * 16 + 4 * g4;
#pragma unroll
    for (int r = 0; r < 4; r++)
        if (s == 0 ? j0 + r > i : j0 + r < i) acc[r] = 0.0f;
    *reinterpret_cast<f32x4*>(&score[s * 1024 + ((it * 64 + (2 * jt + g4 / 2) * 16 + c16) * 8 + 4 * (g4 % 2))]) = acc;
}

// What the walk's two forms do in different places, as functions of values.  A closure that holds the kernel's arguments by reference, anywhere
// in its body, changes how the compiler orders their loads in all of it: calls in two launches whose directions have x and z of their own
// lose by it (16 x 64 tokens of 64 heads x 64, state committed, 49.4 us without and 50.5 with), those that share them gain (state not
// committed 28.9 and 28.4; 9 x 64 of 640 channels 22.6 and 22.2), so there the last of these takes one.
template <int BLOCKS>
__device__ __forceinline__ void ssd_block_rows(Piece (&to)[BLOCKS], const unsigned short* from, long long stride, int t, int last)
{
#pragma unroll
    for (int k = 0; k < BLOCKS; k++) to[k] = *reinterpret_cast<const Piece*>(from + (long long)min(t + 32 * k, last) * stride);
}
// A wave's share of the score units of its head: first, first + step, ..
template <int SCORES, int SHARES>
__device__ __forceinline__ void ssd_block_score_units(f32x4 (&sc)[SHARES][2], const float* fwd, const float* rev, size_t at, int first, int step, int lane)
{
#pragma unroll
    for (int k = 0; k < SHARES; k++) {
        const int u = first + k * step, us = u / (2 * SCORES), v = u - us * (2 * SCORES);
        if (u < 2 * SHARES) {
            const float* const src = (us == 0 ? fwd : rev) + at + (v * 64 + lane) * 8;
            sc[k][0] = *reinterpret_cast<const f32x4*>(src);
            sc[k][1] = *reinterpret_cast<const f32x4*>(src + 4);
        }
    }
}
// Inter-block term of the forward direction: exp(l_i) C_i H.
template <int NB, int RT, typename COp>
__device__ __forceinline__ void ssd_block_inter(f32x4 (&y)[RT], const f32x4 (&h)[NB][2], const float* exp_l, int g4, COp c_op)
{
#pragma unroll
    for (int nb = 0; nb < NB; nb++) {
        bf16x8 hb;
#pragma unroll
        for (int e = 0; e < 8; e++) hb[e] = (__bf16)h[nb][e / 4][e % 4];
#pragma unroll
        for (int rt = 0; rt < RT; rt++) y[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c_op(nb, rt), hb, y[rt], 0, 0, 0);
    }
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
        const float4 e4 = *reinterpret_cast<const float4*>(&exp_l[16 * rt + 4 * g4]);
        y[rt][0] *= e4.x; y[rt][1] *= e4.y; y[rt][2] *= e4.z; y[rt][3] *= e4.w;
    }
}

// grid (ceil(Dn / 64), 1, batch), block 256: wave w owns channels 16 (4 blockIdx.x + w) .. of one batch element.  COMMIT: h_out is
// written; SHARED: both directions read the same x and the same z (the registers of the other cases are not held here).
// WHOLE: grid (ceil(Dn / 64 / tiles), 1, batch), block 1024, dynamic LDS SsdBlockLds::bytes(tiles): the workgroup makes the operands
// for itself, and its waves own up to four such tiles of one group.
template <int N, int BLOCKS, bool COMMIT, bool SHARED, bool WHOLE = false>
__global__ __launch_bounds__(WHOLE ? 1024 : 256, WHOLE ? 4 : BLOCKS == 1 ? 4 : COMMIT ? 2 : 3) void ssd_block_kernel(const SsdBlockArgs a)
{
    static_assert(!WHOLE || BLOCKS == 1, "one launch: up to 32 tokens");
    using T = unsigned short;
    constexpr int kTok = 32 * BLOCKS, kRT = 2 * BLOCKS, kNB = N / 32, kScores = ssd_block_scores<BLOCKS>();
    // wave-private tables by token: forward e_i, f_j Delta_j, exp(l_i), end weight; reverse e_i, f_j Delta_j
    constexpr int kTabBytes = 4 * 6 * kTok * (int)sizeof(float);
    // raw x by row (row r: token r - 3; zeros outside the block and its cached tail), and the outputs before the gate
    constexpr int kRows = kTok + 6, kXPitch = 68, kYPitch = 68;
    // and the score operands, made once per head: [head of the tile][direction, block, 16 rows][lane].  With 64 tokens the
    // outputs lie over x and the operands, in one launch over the rows of B and C.
    constexpr int kXBytes = (SHARED ? 1 : 2) * kRows * kXPitch * (int)sizeof(T), kUnits = 2 * kScores * 2;
    constexpr int kMAt = (kXBytes + 15) / 16 * 16, kMBytes = 2 * kUnits * 64 * 16, kYBytes = 2 * kTok * kYPitch * 4;
    constexpr int kYAt = BLOCKS == 1 ? kMAt + kMBytes : 0, kAll = BLOCKS == 1 ? kYAt + kYBytes : kMAt + kMBytes > kYBytes ? kMAt + kMBytes : kYBytes;
    const int tid = WHOLE ? threadIdx.x & 255 : threadIdx.x, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = WHOLE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0, tiles = WHOLE ? a.tiles : 1;
    unsigned char *s_all, *s_yall;
    float(*tab)[kTok];
    using Lds = SsdBlockLds<N, COMMIT, SHARED>;
    __bf16(*split)[4][32][N + kPrepPad] = nullptr;
    float* s_score = nullptr;
    bf16x8* s_bt = nullptr;
    if constexpr (WHOLE) {
        static_assert(Lds::kY == kYBytes && Lds::kTab == kTabBytes && Lds::kX == kMAt && Lds::kM == kMBytes, "the parts of a tile");
        extern __shared__ __attribute__((aligned(16))) unsigned char ssd_block_lds[];
        unsigned char* const after = ssd_block_lds + Lds::front(tiles);
        unsigned char* const own = after + Lds::kScore + Lds::kBt + tile * Lds::kTile;
        split = reinterpret_cast<__bf16(*)[4][32][N + kPrepPad]>(ssd_block_lds);
        s_score = reinterpret_cast<float*>(after);
        s_bt = reinterpret_cast<bf16x8*>(after + Lds::kScore);
        tab = reinterpret_cast<float(*)[kTok]>(own) + wave * 6;
        s_all = own + kTabBytes;
        s_yall = ssd_block_lds + tile * kYBytes;
    } else {
        __shared__ __attribute__((aligned(16))) unsigned char s_tab[kTabBytes];
        __shared__ __attribute__((aligned(16))) unsigned char s_own[kAll];
        tab = reinterpret_cast<float(*)[kTok]>(s_tab) + wave * 6;
        s_all = s_own;
        s_yall = s_own + kYAt;
    }
    auto* const s_x = reinterpret_cast<T(*)[kRows][kXPitch]>(s_all);
    auto* const s_m = reinterpret_cast<bf16x8*>(s_all + kMAt);
    auto* const s_y = reinterpret_cast<float(*)[kTok][kYPitch]>(s_yall);
    // workgroups dealt to the XCDs batch-major: the heads of a batch element share its operands
    int wg = blockIdx.x, b = blockIdx.z;
    {
        const unsigned total = gridDim.x * gridDim.z, id = blockIdx.x + gridDim.x * blockIdx.z;
        if (total % 8 == 0) {
            const unsigned item = (id % 8) * (total / 8) + id / 8;
            wg = (int)(item % gridDim.x);
            b = (int)(item / gridDim.x);
        }
    }
    const int wg_ch0 = (wg * tiles + tile) * 64;
    // (one launch) the rows of B and C are requested first and worked on when everything else has been requested
    SsdBlockRows<N, COMMIT> bc;
    const bool has_rows = threadIdx.x < 8 * N;
    if constexpr (WHOLE) {
        const int g = wg * tiles * 64 / (a.HG * a.P);
        if (has_rows) bc.request(a, g, b, threadIdx.x, wg * tiles * 64 == g * a.HG * a.P);
        if (tile >= tiles || wg_ch0 >= a.Dn) {   // waves without channels: rows, the scores of the first eight waves, the barriers
            if (has_rows) bc.finish(a, b, split, s_bt);
            __syncthreads();
            const int w = tile * 4 + wave;
            if (w < 8) ssd_block_scores_of<N>(w, lane, split, s_score);
            __syncthreads();
            __syncthreads();
            __syncthreads();
            return;
        }
    }
    // (waves past the last channel shadow the last tile: they join the barriers and store nothing)
    const bool active = wg_ch0 + wave * 16 < a.Dn;
    const int ch0 = active ? wg_ch0 + wave * 16 : a.Dn - 16;
    const int head = ch0 / a.P, grp = head / a.HG, ch = ch0 + c16, last = a.L - 1;
    const size_t item = (size_t)b * a.G + grp;

    // ---- everything the wave reads
    T dtraw[BLOCKS];
    float a2, dtb = 0.0f;
    {
        // 32 tokens: the lower half of the wave scans the forward direction, the upper half the reverse one, each in its order
        const int s = BLOCKS == 1 ? lane >> 5 : 0;
        const SsdBlockDir& df = a.dir[0];
        const SsdBlockDir& db = a.dir[1];
        if constexpr (BLOCKS == 1) {
            const T* const dp = s == 0 ? (const T*)df.dt.p + (size_t)b * df.dt.sb : (const T*)db.dt.p + (size_t)b * db.dt.sb;
            const int t = s == 0 ? lane : kTok - 1 - (lane - 32);
            dtraw[0] = dp[min(t, last) * (s == 0 ? df.dt.st : db.dt.st) + head];
            a2 = (s == 0 ? df.A : db.A)[head] * kLog2e;
            const float* const bias = s == 0 ? df.dt_bias : db.dt_bias;
            if (a.dt_softplus && bias) dtb = bias[head];
        } else {
            dtraw[0] = ((const T*)df.dt.p + (size_t)b * df.dt.sb)[min(lane, last) * df.dt.st + head];
            dtraw[BLOCKS - 1] = ((const T*)db.dt.p + (size_t)b * db.dt.sb)[min(kTok - 1 - lane, last) * db.dt.st + head];
            a2 = 0.0f;
        }
    }
    // x and z in pieces of eight channels (any alignment: global accesses need no more than the elements')
    constexpr int kXPieces = (kRows * 8 + 255) / 256;
    constexpr bool kTwoX = !SHARED;
    Piece xraw[kTwoX ? 2 : 1][kXPieces], zraw[kTwoX ? 2 : 1][BLOCKS];
    const int pc = 8 * (tid & 7);                          // this thread's channels within the workgroup's 64
    const bool piece_there = wg_ch0 + pc < a.Dn;
    const int piece_ch = piece_there ? wg_ch0 + pc : a.Dn - 8;
#pragma unroll
    for (int s = 0; s < (kTwoX ? 2 : 1); s++)
#pragma unroll
        for (int k = 0; k < kXPieces; k++) {
            const int t = (tid >> 3) + 32 * k - 3;
            const bool tail = s == 0 && t < 0 && a.tail_in && -t <= a.K - 1;
            const T* const src = tail ? (const T*)a.tail_in + ((size_t)b * (a.K - 1) + (a.K - 1 + t)) * a.tail_ch
                                      : (const T*)a.dir[s].x.p + (size_t)b * a.dir[s].x.sb + (long long)min(max(t, 0), last) * a.dir[s].x.st;
            xraw[s][k] = *reinterpret_cast<const Piece*>(src + piece_ch);
            if ((t < 0 && !tail) || t > last) xraw[s][k] = Piece{0, 0, 0, 0};
        }
    float w4[2][4], cb[2], dval[2];
#pragma unroll
    for (int s = 0; s < 2; s++) {
        const SsdBlockDir& d = a.dir[s];
        load_taps(d.conv_w + (size_t)ch * a.K, a.K, w4[s]);
        cb[s] = d.conv_b ? d.conv_b[ch] : 0.0f;
        dval[s] = d.D[a.d_per_head ? head : ch];
    }
    f32x4 h[kNB][2];   // states 32 nb + 16 t + 4 g4 + r of channel ch
    const size_t h_at = ((size_t)b * a.Dn + ch) * N + 4 * g4;
#pragma unroll
    for (int nb = 0; nb < kNB; nb++)
#pragma unroll
        for (int t = 0; t < 2; t++) {
            h[nb][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (a.h_in) h[nb][t] = *reinterpret_cast<const f32x4*>(a.h_in + h_at + 32 * nb + 16 * t);
        }
    // scores: the waves of a head deal its units (direction, block, 16 rows) among themselves
    const int head_waves = a.P / 16, hw = wave % head_waves;
    bf16x8* const m_ops = s_m + (wave / head_waves) * (kUnits * 64) + lane;
    f32x4 sc[kUnits / 2][2];
    if constexpr (!WHOLE) ssd_block_score_units<kScores>(sc, a.score[0], a.score[1], item * (kScores * 1024), hw, head_waves, lane);
    constexpr bool kLateZ = WHOLE && COMMIT && !SHARED && N == 128;   // (for which there are no registers beside the rows')
    if constexpr (!kLateZ) {
#pragma unroll
        for (int s = 0; s < (kTwoX ? 2 : 1); s++)
            ssd_block_rows(zraw[s], (const T*)a.dir[s].z.p + (size_t)b * a.dir[s].z.sb + piece_ch, a.dir[s].z.st, tid >> 3, last);
    }
    if constexpr (WHOLE) {
        __builtin_amdgcn_sched_barrier(0);
        if (has_rows) bc.finish(a, b, split, s_bt);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kLateZ) {
#pragma unroll
        for (int s = 0; s < (kTwoX ? 2 : 1); s++)
            ssd_block_rows(zraw[s], (const T*)a.dir[s].z.p + (size_t)b * a.dir[s].z.sb + piece_ch, a.dir[s].z.st, tid >> 3, last);
    }
#pragma unroll
    for (int s = 0; s < (kTwoX ? 2 : 1); s++)
#pragma unroll
        for (int k = 0; k < kXPieces; k++) {
            const int r = (tid >> 3) + 32 * k;
            uint2* const dst = reinterpret_cast<uint2*>(&s_x[s][r < kRows ? r : 0][pc]);
            if (r < kRows) {
                dst[0] = make_uint2(xraw[s][k][0], xraw[s][k][1]);
                dst[1] = make_uint2(xraw[s][k][2], xraw[s][k][3]);
            }
        }

    // ---- Delta, the cumulative decays and the tables
    bool separable[2];
    float decay_q = 1.0f;
    {
        // separable decay exp(l_i - l_j) = e_i f_j around the block's middle unless it decays too fast (as in ssd_wide.h)
        if constexpr (BLOCKS == 1) {
            const int s = lane >> 5, t = s == 0 ? lane : kTok - 1 - (lane - 32);
            float dl = IoBF16::cvt(dtraw[0]);
            if (a.dt_softplus) dl = softplus(dl + dtb);
            if (t > last) dl = 0.0f;
            const float l2 = half_wave_inclusive_sum(dl * a2);
            const float endf = lane_value(l2, 31), endr = lane_value(l2, 63);
            separable[0] = lane_value(l2, 0) - endf <= 100.0f;
            separable[1] = lane_value(l2, 32) - endr <= 100.0f;
            const float mid = s == 0 ? lane_value(l2, 15) : lane_value(l2, 47), end = s == 0 ? endf : endr;
            const bool sep = s == 0 ? separable[0] : separable[1];
            float* const row = tab[s == 0 ? 0 : 4] + t;
            row[0] = sep ? fast_exp2(l2 - mid) : l2;
            row[kTok] = sep ? fast_exp2(mid - l2) * dl : dl;
            if (s == 0) {
                row[2 * kTok] = fast_exp2(l2);
                row[3 * kTok] = fast_exp2(end - l2) * dl;
            }
            decay_q = fast_exp2(endf);
        } else {
#pragma unroll
            for (int s = 0; s < 2; s++) {
                const int t = s == 0 ? lane : kTok - 1 - lane;
                float dl = IoBF16::cvt(dtraw[s == 0 ? 0 : BLOCKS - 1]);
                if (a.dt_softplus) dl = softplus(dl + (a.dir[s].dt_bias ? a.dir[s].dt_bias[head] : 0.0f));
                if (t > last) dl = 0.0f;
                const float l2 = wave_inclusive_sum(dl * (a.dir[s].A[head] * kLog2e));
                const float mid = lane_value(l2, 31), end = lane_value(l2, 63);
                separable[s] = lane_value(l2, 0) - end <= 100.0f;
                float* const row = tab[s == 0 ? 0 : 4] + t;
                row[0] = separable[s] ? fast_exp2(l2 - mid) : l2;
                row[kTok] = separable[s] ? fast_exp2(mid - l2) * dl : dl;
                if (s == 0) {
                    row[2 * kTok] = fast_exp2(l2);
                    row[3 * kTok] = fast_exp2(end - l2) * dl;
                    decay_q = fast_exp2(end);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }

    if constexpr (WHOLE) {
        __syncthreads();                                   // the rows of B and C
        const int w = tile * 4 + wave;
        if (w < 8) ssd_block_scores_of<N>(w, lane, split, s_score);
    }
    // ---- inter-block term of the forward direction, exp(l_i) C_i H: in one launch while the scores are made, else once the registers of
    // the scores are free (with them held, 15 layers x 4 steps of 9 x 64 tokens of 640 channels took 1338 us; 1237)
    f32x4 y[2][kRT];
#pragma unroll
    for (int rt = 0; rt < kRT; rt++) y[0][rt] = y[1][rt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (WHOLE) {
        if (a.h_in)
            ssd_block_inter(y[0], h, tab[2], g4, [=](int nb, int rt) -> bf16x8 {
                const __bf16* const row = &split[0][2][16 * rt + c16][32 * nb + 4 * g4];
                const bf16x4 lo = *reinterpret_cast<const bf16x4*>(row), hi = *reinterpret_cast<const bf16x4*>(row + 16);
                return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            });
        __syncthreads();                                   // the scores
        ssd_block_score_units<kScores>(sc, s_score, s_score + 1024, 0, hw, head_waves, lane);
    }
    // ---- the head's masked, decayed score operands
#pragma unroll
    for (int k = 0; k < kUnits / 2; k++) {
        const int u = hw + k * head_waves, us = u / (2 * kScores), v = u - us * (2 * kScores), m = v / 2;
        if (u < kUnits) {
            // block (i, j) of the kept ones: forward (0,0), (1,0), (1,1); reverse (0,0), (0,1), (1,1)
            const int ib = us == 0 ? (m > 0) : (m > 1), jb = m - ib, i = ib * 32 + 16 * (v % 2) + c16, j0 = jb * 32 + 8 * g4;
            const float* const te = tab[us == 0 ? 0 : 4];
            const float* const tf = te + kTok;
            const float ei = te[i];
            bf16x8 op;
#pragma unroll
            for (int h2 = 0; h2 < 2; h2++) {
                const f32x4 sv = sc[k][h2];
                const float4 f4 = *reinterpret_cast<const float4*>(&tf[j0 + 4 * h2]);
                const float fj[4] = {f4.x, f4.y, f4.z, f4.w};
                if (us == 0 ? separable[0] : separable[1]) {
#pragma unroll
                    for (int e = 0; e < 4; e++) op[4 * h2 + e] = (__bf16)(sv[e] * ei * fj[e]);
                } else {
                    const float4 l4 = *reinterpret_cast<const float4*>(&te[j0 + 4 * h2]);
                    const float lj[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const int j = j0 + 4 * h2 + e;
                        const float val = sv[e] * fast_exp2(ei - lj[e]) * fj[e];
                        op[4 * h2 + e] = (__bf16)((us == 0 ? j > i : j < i) ? 0.0f : val);
                    }
                }
            }
            m_ops[u * 64] = op;
        }
    }

    if constexpr (!WHOLE) {
        if constexpr (SHARED) {   // (by reference: see ssd_block_rows)
            if (a.h_in)
                ssd_block_inter(y[0], h, tab[2], g4, [&](int nb, int rt) {
                    return reinterpret_cast<const bf16x8*>(a.c_op)[item * (kTok * N / 8) + (nb * kRT + rt) * 64 + lane];
                });
        } else if (a.h_in) {
            const bf16x8* const c_op = reinterpret_cast<const bf16x8*>(a.c_op) + item * (kTok * N / 8) + lane;
            ssd_block_inter(y[0], h, tab[2], g4, [=](int nb, int rt) { return c_op[(nb * kRT + rt) * 64]; });
        }
    }

    __syncthreads();                                       // x and the score operands
    // ---- conv + SiLU of the lane's runs, as contraction operands, and (forward) weighted to the block's end
    bf16x8 xc[2][BLOCKS], xw[BLOCKS];
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
        for (int blk = 0; blk < BLOCKS; blk++) {
            const int t0 = blk * 32 + 8 * g4;
            float xr[11];   // forward: tokens t0 - 3 ..; reverse: tokens t0 ..
#pragma unroll
            for (int q = 0; q < 11; q++) xr[q] = IoBF16::cvt(s_x[kTwoX ? s : 0][t0 + q + 3 * s][wave * 16 + c16]);
            const float4 wa = *reinterpret_cast<const float4*>(&tab[3][t0]), wb = *reinterpret_cast<const float4*>(&tab[3][t0 + 4]);
            const float wq[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
            for (int e = 0; e < 8; e++) {
                float pre = cb[s];
#pragma unroll
                for (int k = 0; k < 4; k++) pre = fmaf(w4[s][k], xr[s == 0 ? e + k : e + 3 - k], pre);
                const float v = silu(pre);
                xc[s][blk][e] = (__bf16)v;
                if (COMMIT && s == 0) xw[blk][e] = (__bf16)(v * wq[e]);
            }
        }

    // ---- x's part of the committed tail: the last K - 1 raw tokens of (tail_in || block)
    if (a.tail_out && (tid >> 3) < a.K - 1 && piece_there) {
        const int n = tid >> 3;
        const uint2* const src = reinterpret_cast<const uint2*>(&s_x[0][a.L - (a.K - 1) + n + 3][pc]);
        const uint2 lo = src[0], hi = src[1];
        *reinterpret_cast<Piece*>((T*)a.tail_out + ((size_t)b * (a.K - 1) + n) * a.tail_ch + piece_ch) = Piece{lo.x, lo.y, hi.x, hi.y};
    }

    // ---- intra-block products with the scores, and the skip term
#pragma unroll
    for (int s = 0; s < 2; s++) {
#pragma unroll
        for (int rt = 0; rt < kRT; rt++) {
            const int ib = rt / 2;
#pragma unroll
            for (int jb = s == 0 ? 0 : ib; jb < (s == 0 ? ib + 1 : BLOCKS); jb++)
                y[s][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m_ops[((s * kScores + ib + jb) * 2 + rt % 2) * 64], xc[s][jb], y[s][rt], 0, 0, 0);
            bf16x8 one;    // rows of the identity
#pragma unroll
            for (int e = 0; e < 8; e++) one[e] = (__bf16)(8 * g4 + e == 16 * (rt % 2) + c16 ? 1.0f : 0.0f);
            const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
            const f32x4 xa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(one, xc[s][ib], zero, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; r++) y[s][rt][r] += dval[s] * xa[r];
        }
    }

    // ---- the committed state
    if constexpr (COMMIT) {
        const bf16x8* const b_op = (WHOLE ? s_bt : reinterpret_cast<const bf16x8*>(a.b_op) + item * (kTok * N / 8)) + lane;
#pragma unroll
        for (int nb = 0; nb < kNB; nb++)
#pragma unroll
            for (int t = 0; t < 2; t++) {
                f32x4 v = h[nb][t];
#pragma unroll
                for (int r = 0; r < 4; r++) v[r] *= decay_q;
#pragma unroll
                for (int blk = 0; blk < BLOCKS; blk++)
                    v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b_op[((2 * nb + t) * BLOCKS + blk) * 64], xw[blk], v, 0, 0, 0);
                if (active) *reinterpret_cast<f32x4*>(a.h_out + h_at + 32 * nb + 16 * t) = v;
            }
    }

    // ---- gate, combine, round: a token's eight channels per thread
    const bool one_y = SHARED && !a.separate;
    if constexpr (BLOCKS > 1) __syncthreads();             // (x and the operands have been read)
#pragma unroll
    for (int rt = 0; rt < kRT; rt++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int t = 16 * rt + 4 * g4 + r, c = wave * 16 + c16;
            if (one_y) s_y[0][t][c] = y[0][rt][r] + y[1][rt][r];
            else {
                s_y[0][t][c] = y[0][rt][r];
                s_y[1][t][c] = y[1][rt][r];
            }
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BLOCKS; k++) {
        const int t = (tid >> 3) + 32 * k;
        if (t > last || !piece_there) continue;
        T* const o = (T*)a.out + (size_t)b * a.out_sb + (long long)t * a.out_st + piece_ch;
        Piece res[2];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            float v[2][2];
#pragma unroll
            for (int e = 0; e < 2; e++) {
                auto part = [e](unsigned p) { return __uint_as_float(e == 0 ? p << 16 : p & 0xffff0000u); };
                const float zf = silu(part(zraw[0][k][i])), yf = s_y[0][t][pc + 2 * i + e];
                if (one_y) v[0][e] = yf * zf;
                else {
                    const float zb = SHARED ? zf : silu(part(zraw[kTwoX ? 1 : 0][k][i])), yb = s_y[1][t][pc + 2 * i + e];
                    v[0][e] = a.separate ? yf * zf : fmaf(yf, zf, yb * zb);
                    v[1][e] = yb * zb;
                }
            }
            typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
#pragma unroll
            for (int h2 = 0; h2 < 2; h2++) res[h2][i] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)v[h2][0], (__bf16)v[h2][1]});
        }
        *reinterpret_cast<Piece*>(o) = res[0];
        if (a.separate) *reinterpret_cast<Piece*>(o + a.Dn) = res[1];
    }
}

}  // namespace bm
