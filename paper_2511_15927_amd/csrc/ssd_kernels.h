// Chunked state-space-duality kernels for the Mamba-2 parameterisation (one decay rate per head) on gfx950.
//
// With a scalar decay per head the recurrence over a chunk of Q = 64 tokens is a set of dense contractions
// (j, i: positions in the chunk in scan order; l_i = sum_{r<=i} Delta_r A; H: state entering the chunk, [N, P]):
//   y_i   = sum_{j<=i} (C_i . B_j) exp(l_i - l_j) Delta_j xc_j  +  exp(l_i) C_i H  +  D xc_i
//   H_out = exp(l_Q) H + sum_j exp(l_Q - l_j) Delta_j B_j^T xc_j
// which run on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate).  One workgroup owns one
// (direction, batch, head) and walks the chunks in scan order with H in accumulator registers (fp32 for the whole
// sequence).  Decay factors are formed in fp32; only MFMA operands (xc, B, C, the masked score tile, a copy of H) are
// rounded to bf16.  ssd_prep_kernel builds, once per (direction, batch, chunk, group) and shared by all heads, the
// score tile C B^T, C and the transposed B in bf16, all in the order in which the walk's matrix products take them.
//
// Kernels in this file: ssd_prep_kernel (above); ssd_state_kernel and ssd_carry_kernel, which find the state entering each time part
// when a call has too few (batch, head) items to fill the chip.  The chunk walk is in ssd_wide.h, calls of one chunk in ssd_block.h.
//
// Lane layouts of the 32x32x16 MFMA (checked on hardware): operand A lane l holds row l%32, k = 8*(l/32)..+7;
// operand B lane l holds column l%32, same k; accumulator register r of lane l is row 8*(r/4) + 4*(l/32) + r%4,
// column l%32.  A contraction index may be enumerated in any order as long as both operands agree, which lets an
// accumulator tile be fed back as an operand without a transpose: registers 8*kb..8*kb+7 of a lane are the 8
// k-slots of k-block kb, i.e. k = 16*kb + 8*jj + 4*(l/32) + e for slot 4*jj + e.
#pragma once
#include "kernels.h"
#include <type_traits>

namespace bm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// A channel pair at any 2-byte aligned place (global accesses need no more than that here).
typedef unsigned __attribute__((aligned(2))) bf16_pair;

constexpr int kQ = 64;     // chunk length
constexpr int kPadK = 8;   // bf16 elements of row padding in LDS tiles (keeps 16-byte alignment, spreads banks)
constexpr int kScoreOp = 3 * 2 * 64 * 8;   // floats of one chunk's score tile: 3 lower-triangular 32x32 blocks

struct SsdPrepArgs {
    TensorArg B, C;       // bf16 [batch][L][G*N]
    const float* conv_w;  // full [conv_ch][K] table of this direction (rows Dn.. are B|C) when conv_bc
    const float* conv_b;  // or null
    const void* tail_in;  // bf16 [batch][K-1][tail_ch] or null (causal direction of the block variant)
    __bf16* c_rows;    // [batch][nchunk][G][64 x N], MFMA operand order (see the kernel)
    __bf16* b_t;       // the same
    float* score_op;   // [batch][nchunk][G][kScoreOp]: B_j . C_i for j, i in the chunk, MFMA operand order (see the kernel)
    int L, G, K, Dn, tail_ch, conv_bc;
    int dir;           // +1: scan position tau is token tau; -1: token L-1-tau
    int lead;          // positions before the sequence that the first chunk starts with (kSsdMeet)
};

struct SsdPrepPair {
    SsdPrepArgs dir[2];   // forward, reverse: one launch prepares both
};

// LDS of ssd_prep_kernel: the chunk's B and C rows after the conv, each value as a bf16 head and the bf16 rest of it.  (The form
// of sixteen waves adds the partial score accumulators of the waves that share a block: [12][64][16] floats.)
constexpr int kPrepPad = 8;
template <int N, int THREADS>
constexpr size_t ssd_prep_lds_bytes()
{
    return 4 * (size_t)kQ * (N + kPrepPad) * sizeof(__bf16) + (THREADS > 256 ? 12 * 64 * 16 * sizeof(float) : 0);
}

// grid (nchunk, G, 2 * batch), block THREADS (256 or 1024), dynamic LDS ssd_prep_lds_bytes<N, THREADS>();
// blockIdx.z / batch selects the direction.  Reads the raw B and C rows of one chunk (plus the conv halo), two columns a
// thread, applies the short conv + SiLU along the scan direction when they pass through it, and leaves the result in LDS split the
// way the score product takes it, so that every operand below is read in pieces of eight or sixteen bytes (fp32 columns, read
// one by one and split by every wave that needs them: 61.4 us for 8 x 8192 tokens, N 128; this: 41.5; 1 x 1024 tokens, sixteen waves,
// 9.3 -> 7.5).  B^T pieces are a column's consecutive positions: they go out from registers.  The form
// of sixteen waves is for launches of few workgroups (short sequences), whose duration is one workgroup's chain of phases.
template <int N, int THREADS = 256>
__global__ __launch_bounds__(THREADS) void ssd_prep_kernel(const SsdPrepPair both)
{
    static_assert(THREADS == 256 || THREADS == 1024, "four or sixteen waves");
    using T = unsigned short;
    constexpr int kRow = N + kPrepPad;
    const int batch = gridDim.z / 2;
    const SsdPrepArgs& a = both.dir[blockIdx.z / batch];
    extern __shared__ __attribute__((aligned(16))) unsigned char ssd_prep_lds[];
    __bf16(*const split)[kQ][kRow] = reinterpret_cast<__bf16(*)[kQ][kRow]>(ssd_prep_lds);   // B head, B rest, C head, C rest
    const int c = blockIdx.x, g = blockIdx.y, b = blockIdx.z % batch, tid = threadIdx.x;
    const int nchunk = gridDim.x;
    const size_t tile = ((size_t)b * nchunk + c) * a.G + g;
    constexpr int kParts = THREADS / N, kLen = kQ / kParts;   // positions of a thread
    constexpr bool kFromRegisters = kLen >= 8;
    {
        const int seg = __builtin_amdgcn_readfirstlane(tid / N), n = 2 * (tid % (N / 2));   // columns n, n + 1 of B or C
        int which = tid % N / (N / 2);
        if constexpr (N == 128) which = __builtin_amdgcn_readfirstlane(which);   // rows at wave-uniform addresses
        const TensorArg& src = which ? a.C : a.B;
        const T* const base = (const T*)src.p + (size_t)b * src.sb + g * N;
        const int last = a.L - 1;
        const int row = a.Dn + which * a.G * N + g * N + n;   // the first column's conv channel
        const int tau0 = c * kQ + seg * kLen - 3 - a.lead;
        bf16_pair raw[kLen + 3];
        {   // (positions outside the sequence repeat its nearest row)
            const int first = min(max(tau0, 0), last);
            const T* at = base + (long long)(a.dir > 0 ? first : last - first) * src.st;
            const long long step = a.dir > 0 ? src.st : -src.st;
#pragma unroll
            for (int q = 0; q < kLen + 3; q++) {
                raw[q] = *(const bf16_pair*)(at + n);
                at += ((tau0 + q >= 0) & (tau0 + q < last)) ? step : 0;
            }
        }
        const bool from_tail = c == 0 && seg == 0 && a.dir > 0 && a.tail_in && a.conv_bc && a.K > 1;
        if (from_tail) {
            // requested together from clamped rows (a tap beyond the conv width has a zero weight)
#pragma unroll
            for (int q = 0; q < 3; q++)   // 3 - q tokens before the block
                raw[q] = *(const bf16_pair*)((const T*)a.tail_in + ((size_t)b * (a.K - 1) + max(a.K - 1 - (3 - q), 0)) * a.tail_ch + row);
        }
        float w4[2][4], bias[2] = {0.0f, 0.0f};   // w4[.][3] on the current position
#pragma unroll
        for (int q = 0; q < 2; q++)
#pragma unroll
            for (int i = 0; i < 4; i++) w4[q][i] = 0.0f;
        if (a.conv_bc) {
#pragma unroll
            for (int q = 0; q < 2; q++) load_taps(a.conv_w + (size_t)(row + q) * a.K, a.K, w4[q]);
            if (a.conv_b) {
                bias[0] = a.conv_b[row];
                bias[1] = a.conv_b[row + 1];
            }
        }
        // positions before the sequence (or the cached tail) and past its end are zeros
        const int front = from_tail ? 4 - a.K : max(-tau0, 0), end = last - tau0;
#pragma unroll
        for (int q = 0; q < kLen + 3; q++) raw[q] = ((q >= front) & (q <= end)) ? raw[q] : 0u;
        auto column = [&](int q, int k) -> float { return __uint_as_float(k ? raw[q] & 0xffff0000u : raw[q] << 16); };
        bf16x8 piece[2];
        auto rows = [&](auto conv) {
#pragma unroll
            for (int i = 0; i < kLen; i++) {
                __bf16 head[2], rest[2];
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    float v = column(i + 3, k);
                    if constexpr (decltype(conv)::value) {
                        float pre = bias[k];
                        pre = fmaf(w4[k][0], column(i, k), pre);
                        pre = fmaf(w4[k][1], column(i + 1, k), pre);
                        pre = fmaf(w4[k][2], column(i + 2, k), pre);
                        pre = fmaf(w4[k][3], column(i + 3, k), pre);
                        v = silu(pre);
                    }
                    v = ((i + 3 >= front) & (i + 3 <= end)) ? v : 0.0f;
                    head[k] = (__bf16)v;
                    rest[k] = (__bf16)(v - (float)head[k]);
                    if constexpr (kFromRegisters) piece[k][i % 8] = head[k];
                }
                const int r = seg * kLen + i;
                *reinterpret_cast<bf16x2*>(&split[2 * which][r][n]) = bf16x2{head[0], head[1]};
                *reinterpret_cast<bf16x2*>(&split[2 * which + 1][r][n]) = bf16x2{rest[0], rest[1]};
                if constexpr (kFromRegisters) {
                    if (i % 8 == 7 && which == 0) {
                        // B^T as [32 states][16 positions][lane]: lane l holds state l%32, positions 8 (l/32) .. + 7
                        const int j0 = r - 7;
#pragma unroll
                        for (int k = 0; k < 2; k++) {
                            const int idx = ((n / 32) * 4 + j0 / 16) * 64 + (j0 / 8) % 2 * 32 + n % 32 + k;
                            *reinterpret_cast<bf16x8*>(&a.b_t[(tile * kQ * N / 8 + idx) * 8]) = piece[k];
                        }
                    }
                }
            }
        };
        if (a.conv_bc) rows(std::true_type{});
        else rows(std::false_type{});
    }
    __syncthreads();
    auto b_column = [&](int n, int j0) {   // eight positions of a state
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = split[0][j0 + e][n];
        return v;
    };
    // C as [row block of 16][32 states][lane of an MFMA operand], with the states in the order the state's accumulators publish them
    for (int idx = tid; idx < kQ * N / 8; idx += THREADS) {
        const int ln = idx % 64, f = idx / 64;
        const int i = (f / (N / 32)) * 16 + ln % 16, n0 = (f % (N / 32)) * 32 + 16 * ((ln / 16) % 2) + 4 * (ln / 32);
        const bf16x4 lo = *reinterpret_cast<const bf16x4*>(&split[2][i][n0]), hi = *reinterpret_cast<const bf16x4*>(&split[2][i][n0 + 8]);
        *reinterpret_cast<bf16x8*>(&a.c_rows[(tile * kQ * N / 8 + idx) * 8]) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        if constexpr (!kFromRegisters) {
            const int n2 = (f / 4) * 32 + ln % 32, j0 = (f % 4) * 16 + 8 * (ln / 32);
            *reinterpret_cast<bf16x8*>(&a.b_t[(tile * kQ * N / 8 + idx) * 8]) = b_column(n2, j0);
        }
    }
    // Score tile B_j . C_i on the matrix cores, one 32 x 32 block per wave; only the three blocks on or below the
    // diagonal are kept.  Each fp32 operand is split into a bf16 head and a bf16 remainder and the three significant
    // cross products are accumulated in fp32, which keeps about 16 bits of the products.  With B rows as operand A
    // and C rows as operand B, accumulator register r of lane l is row j%32 = 8*(r/4) + 4*(l/32) + r%4 of column
    // i%32 = l%32, block pairs (0,0), (1,0), (1,1).
    const int wave = tid / 64, lane = tid % 64;
    // Sixteen waves deal a block's N / 16 contraction steps to four waves and adds their accumulators through LDS.
    constexpr int kSplit = THREADS > 256 ? 4 : 1;
    constexpr int kSteps = N / 16 / kSplit;
    const int blk = wave / kSplit, kpart = wave % kSplit;
    f32x16 acc = {0};
    if (blk < 3) {
        const int iblk = blk > 0, jblk = blk > 1;
        const int rj = jblk * 32 + lane % 32, ri = iblk * 32 + lane % 32, koff = 8 * (lane / 32);
        for (int ks = kpart * kSteps; ks < (kpart + 1) * kSteps; ks++) {
            const int k0 = 16 * ks + koff;
            const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&split[0][rj][k0]), al = *reinterpret_cast<const bf16x8*>(&split[1][rj][k0]);
            const bf16x8 bh = *reinterpret_cast<const bf16x8*>(&split[2][ri][k0]), bl = *reinterpret_cast<const bf16x8*>(&split[3][ri][k0]);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
        }
    }
    if constexpr (kSplit > 1) {
        float* const sums = reinterpret_cast<float*>(split + 4);   // [12][64][16]
        if (blk < 3 && kpart > 0) {
#pragma unroll
            for (int q = 0; q < 4; q++)
                *reinterpret_cast<float4*>(&sums[((size_t)wave * 64 + lane) * 16 + 4 * q]) =
                    make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        }
        __syncthreads();
        if (blk < 3 && kpart == 0) {
            for (int o = 1; o < kSplit; o++) {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const float4 v = *reinterpret_cast<const float4*>(&sums[((size_t)(wave + o) * 64 + lane) * 16 + 4 * q]);
                    acc[4 * q] += v.x; acc[4 * q + 1] += v.y; acc[4 * q + 2] += v.z; acc[4 * q + 3] += v.w;
                }
            }
        }
    }
    if (blk < 3 && kpart == 0) {
        // [block][16 rows i][lane][8]: slot 4t + e of lane l holds row i = l%16 of column j = 16t + 4(l/16) + e; zero above the diagonal
        float* const dst = a.score_op + tile * kScoreOp;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = blk != 1 && 8 * q + 4 * (lane / 32) + e > lane % 32 ? 0.0f : acc[4 * q + e];
            const int sl = (2 * (q % 2) + lane / 32) * 16 + lane % 16;
            *reinterpret_cast<float4*>(dst + ((blk * 2 + (lane / 16) % 2) * 64 + sl) * 8 + 4 * (q / 2)) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
}

// Output modes of the chunk walk (ssd_wide.h).
enum { kSsdFinalOnly = 0, kSsdPartial = 1, kSsdPartialRaw = 2, kSsdFinalAdd = 3, kSsdFinalAddRaw = 4 };
// Its forms.
constexpr int kSsdWhole = 0, kSsdParts = 1, kSsdFarParts = 2, kSsdMeet = 3;

struct SsdArgs {
    TensorArg x, z, dt;
    const float *conv_w, *conv_b, *A, *D, *dt_bias;
    const __bf16* c_rows;
    const __bf16* b_t;
    const float* score_op;
    void* out;
    long long out_sb, out_st;
    void* partial;        // [batch][L][Dn]: bf16 where an item is walked whole, fp32 in the form for time parts (ssd_wide.h)
    const float* h_in;    // [batch][Dn][N] or null
    float* h_out;         // or null
    const void* tail_in;  // bf16 [batch][K-1][tail_ch] or null (causal direction only)
    int L, Dn, H, HG, G, K, tail_ch, nchunk;
    int dir, mode, out_ch_off, dt_softplus, d_per_head;
    int far;              // z or out rows are too far apart for a chunk's 32-bit row offsets (kSsdFarParts)
    // Time parts (calls with too few (batch, head) items to fill the chip): the chunks are dealt to `parts` workgroups
    // per item, part_chunks each, in scan order.  A part is part_subs sub-parts of sub_chunks chunks;
    // ssd_state_kernel leaves every sub-part's end state from a zero start and the product of its chunk decays (all
    // but the scan-last one), ssd_carry_kernel turns those into the state entering each sub-part, and the output launch
    // starts part p from the entry state of sub-part p * part_subs.
    int parts, part_chunks, part_subs, sub_chunks;
    float* part_state;    // [subs][batch][Dn][N]
    float* part_decay;    // [subs][batch][H]
    // Directions that meet in the middle (kSsdMeet): the launch walks part_chunks chunks from first_chunk on, from h_in to h_out.
    int meet, first_chunk;
    int lead;             // positions before the sequence that the first chunk starts with: both directions' chunks hold the same tokens
};

struct SsdCarryArgs {
    float* part_state[2];
    const float* part_decay[2];
    const float* h_in;    // forward direction's initial state or null
    int batch, Dn, P, H, parts;   // parts: the number of sub-parts to fold over
};

// One thread per (direction, batch, channel, four states): entry state of sub-part p+1 = decay_p * entry_p + end_p.
template <int N>
__global__ __launch_bounds__(256) void ssd_carry_kernel(const SsdCarryArgs a)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long per_dir = (long long)a.batch * a.Dn * N / 4;
    if (idx >= 2 * per_dir) return;
    const int s = (int)(idx / per_dir);
    const long long e = (idx % per_dir) * 4;            // element offset inside one part's [batch][Dn][N]
    const int ch = (int)((e / N) % a.Dn), b = (int)(e / ((long long)N * a.Dn));
    float4 h = (s == 0 && a.h_in) ? *reinterpret_cast<const float4*>(a.h_in + e) : make_float4(0.f, 0.f, 0.f, 0.f);
    for (int p = 0; p < a.parts; p++) {
        float4* slot = reinterpret_cast<float4*>(a.part_state[s] + (size_t)p * per_dir * 4 + e);
        const bool more = p + 1 < a.parts;
        const float4 end = more ? *slot : make_float4(0.f, 0.f, 0.f, 0.f);
        *slot = h;
        if (more) {
            const float dk = a.part_decay[s][((size_t)p * a.batch + b) * a.H + ch / a.P];
            h = make_float4(fmaf(dk, h.x, end.x), fmaf(dk, h.y, end.y), fmaf(dk, h.z, end.z), fmaf(dk, h.w, end.w));
        }
    }
}

// LDS-only barrier: waits for this wave's LDS traffic, not for global loads that were issued ahead on purpose.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Inclusive prefix sum over the 64 lanes with DPP moves: shifts inside each row of 16 lanes, then the last lane of
// row 0 / 2 is added to row 1 / 3 and the last lane of row 1 to rows 2 and 3.
__device__ __forceinline__ float wave_inclusive_sum(float v)
{
#define BM_DPP_ADD(ctrl, rows) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xF, false))
    BM_DPP_ADD(0x111, 0xF);  // row_shr:1
    BM_DPP_ADD(0x112, 0xF);  // row_shr:2
    BM_DPP_ADD(0x114, 0xF);  // row_shr:4
    BM_DPP_ADD(0x118, 0xF);  // row_shr:8
    BM_DPP_ADD(0x142, 0xA);  // row_bcast:15 into rows 1 and 3
    BM_DPP_ADD(0x143, 0xC);  // row_bcast:31 into rows 2 and 3
#undef BM_DPP_ADD
    return v;
}

struct SsdStatePair {
    SsdArgs dir[2];   // forward, reverse: one launch walks both
};

// State pass of the time parts.  grid (H, subs - 1, 2 * batch), block 256, static LDS; blockIdx.z / batch selects the
// direction and blockIdx.y the sub-part: sub_chunks chunks in scan order, walked from a zero state.  Leaves the
// sub-part's end state in part_state[sub] and the product of its chunk decays in part_decay[sub] for
// ssd_carry_kernel.  The end state needs neither the score tile nor C nor the gate, so this is the conv + SiLU of x,
// the chunk's decay weights and the state-update product only, in a workgroup light enough (four waves, 19 KB of LDS)
// that three or four of them share a CU; the sub-parts are what gives the chip that many workgroups.  All four
// waves run the short scan for themselves, convolve a quarter of the chunk's positions each, and own 1/4 of the
// 32 x 32 blocks of H, whose B^T operand they read straight from the prepared tile in global memory.
template <int N, int P>
__global__ __launch_bounds__(256, 4) void ssd_state_kernel(const SsdStatePair both)
{
    constexpr int kPB = P / 32, kNB = N / 32, kBlocks = kNB * kPB, kOwn = (kBlocks + 3) / 4;
    constexpr int kRowT = kQ + kPadK;
    constexpr int kCP = P / 2;                // channel pairs of the head
    constexpr int kPos = kQ * kCP / 256;      // chunk positions per thread in the conv (8 or 4)
    using T = unsigned short;
    __shared__ __attribute__((aligned(16))) __bf16 s_xw[2][P * kRowT];   // conv output times end-of-chunk weight, transposed
    __shared__ __attribute__((aligned(16))) float s_wgt[4][kQ];          // wave-private: end-of-chunk weight of each position

    // (a compare, not a division by the batch size: integer division runs on the vector ALU)
    const int batch = gridDim.z >> 1;
    const int reverse = (int)blockIdx.z >= batch ? 1 : 0;
    const SsdArgs& a = both.dir[reverse];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int head = blockIdx.x, b = (int)blockIdx.z - reverse * batch, sub = blockIdx.y;
    const int grp = head / a.HG, ch0 = head * P;
    // (the host never hands this pass the sequence's last sub-part, so every chunk here is a full one)
    const int c_first = sub * a.sub_chunks, c_stop = min(a.L / kQ, c_first + a.sub_chunks);
    const int last = a.L - 1;
    auto token_of = [&](int tau) { return a.dir > 0 ? tau : last - tau; };

    const int cp = tid % kCP, tg = tid / kCP;   // conv role: channels 2cp, 2cp+1; positions kPos*tg .. of each chunk
    const float a2 = a.A[head] * kLog2e;
    const float dtb = (a.dt_softplus && a.dt_bias) ? a.dt_bias[head] : 0.0f;
    float w4[2][4], cbias[2];
#pragma unroll
    for (int h2 = 0; h2 < 2; h2++) {
        load_taps(a.conv_w + (size_t)(ch0 + 2 * cp + h2) * a.K, a.K, w4[h2]);
        cbias[h2] = a.conv_b ? a.conv_b[ch0 + 2 * cp + h2] : 0.0f;
    }
    const T* xb = (const T*)a.x.p + (size_t)b * a.x.sb + ch0 + 2 * cp;
    const T* dtp = (const T*)a.dt.p + (size_t)b * a.dt.sb + head;
    float* const wgt = s_wgt[wave];

    // matrix role: blocks kOwn * wave + o of the kNB x kPB blocks of H, channel block fastest, so that the blocks of a
    // wave share their rows of B^T (kSameB: one operand load serves both)
    constexpr bool kSameB = kOwn == 2 && kPB == 2;
    constexpr int kLoadB = kSameB ? 1 : kOwn;
    const int cl = lane & 31, half = lane >> 5;
    f32x16 hacc[kOwn];
#pragma unroll
    for (int o = 0; o < kOwn; o++)
#pragma unroll
        for (int r = 0; r < 16; r++) hacc[o][r] = 0.0f;

    // channel pair at positions kPos*tg - 3 .. kPos*tg + kPos - 1 and Delta of position `lane`, as requested for the
    // chunk after the one being worked on
    unsigned xnext[kPos + 3];
    T dtraw;
    auto issue_dt = [&](int c) { dtraw = dtp[(long long)token_of(min(c * kQ + lane, last)) * a.dt.st]; };
    // A chunk inside the sequence is read through a raw buffer range anchored at the chunk's lowest token row: the
    // row of register q is a wave-uniform offset, the thread's rows and channel pair a 32-bit offset that never
    // changes (no per-row vector address arithmetic, no address registers).  The host keeps 67 rows within 2^32 bytes.
    const unsigned st_bytes = (unsigned)a.x.st * (unsigned)sizeof(T);
    const unsigned x_lane_off = (unsigned)(a.dir > 0 ? kPos * tg : kQ - kPos * (tg + 1)) * st_bytes + 4u * cp;
    const T* const x_head = (const T*)a.x.p + (size_t)b * a.x.sb + ch0;
    auto issue_x_inside = [&](int c) {   // chunks 1 .. L / kQ - 1
        {
            const Rsrc rows = raw_range(x_head + (long long)(a.dir > 0 ? c * kQ - 3 : last - (c * kQ + kQ - 1)) * a.x.st);
            // register q holds scan position q of the thread, so the rows run backwards in the reverse direction.
            // (The offsets are formed in scalar registers for every chunk anew: carried across the loop, the compiler
            // keeps them in vector registers and loops over the lanes to read them back for each load.)
            int row_step = __builtin_amdgcn_readfirstlane(a.dir * (int)st_bytes);
            asm volatile("" : "+s"(row_step));
            const int row_0 = ((1 - a.dir) >> 1) * (kPos + 2) * (a.dir * row_step);
#pragma unroll
            for (int q = 0; q < kPos + 3; q++)
                xnext[q] = __builtin_amdgcn_raw_buffer_load_b32(rows, x_lane_off, row_0 + q * row_step, 0);
        }
    };
    auto issue_x_first = [&]() {   // chunk 0: positions before the sequence are clamped here and zeroed in the conv
        const int tau0 = kPos * tg - 3;
#pragma unroll
        for (int q = 0; q < kPos + 3; q++)
            xnext[q] = *reinterpret_cast<const unsigned*>(xb + (long long)token_of(min(max(tau0 + q, 0), last)) * a.x.st);
    };
    if (c_first >= c_stop) return;   // (never: see above)
    issue_dt(c_first);
    if (c_first == 0) issue_x_first(); else issue_x_inside(c_first);
    float decay_product = 1.0f;
    // The walk is bound by the latency of its loads (a row piece of 128 bytes per token, each from another DRAM page),
    // not by its arithmetic: what chunk c + 1 needs is requested at the top of chunk c, a whole chunk of work ahead,
    // and on every path alike (the walk's last chunk re-requests a valid chunk), so that the waits below count the
    // same loads in flight whichever way the loop was entered.
    const int c_inside = a.L / kQ - 1;   // the last chunk that is certainly a full one
    for (int c = c_first; c < c_stop; c++) {
        const int buf = (c - c_first) & 1;
        const int cn = max(1, min(c + 1, c_inside));
        // take over what was requested for this chunk
        unsigned xraw[kPos + 3];
#pragma unroll
        for (int q = 0; q < kPos + 3; q++) xraw[q] = xnext[q];
        float dl = IoBF16::cvt(dtraw);
        issue_dt(cn);
        // this wave's B^T operands straight from the prepared tile (whole pieces in lane order), used after the barrier
        bf16x8 ab[kLoadB][4];
        {
            const bf16x8* bsrc = reinterpret_cast<const bf16x8*>(a.b_t + ((((size_t)b * a.nchunk + c) * a.G + grp) * N) * kQ) + lane;
#pragma unroll
            for (int o = 0; o < kLoadB; o++) {
                const int id = kOwn * wave + o, nblk = id / kPB;
                if (kBlocks % 4 == 0 || id < kBlocks) {
#pragma unroll
                    for (int kb = 0; kb < 4; kb++) ab[o][kb] = bsrc[(nblk * 4 + kb) * 64];
                }
            }
        }
        issue_x_inside(cn);
        // Delta, inclusive cumulative log2-decay, end-of-chunk weight of position `lane`
        if (a.dt_softplus) dl = softplus(dl + dtb);
        if (c * kQ + lane > last) dl = 0.0f;
        const float l2 = wave_inclusive_sum(dl * a2);
        const float l2_end = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l2), 63));
        wgt[lane] = fast_exp2(l2_end - l2) * dl;
        const float decay_q = fast_exp2(l2_end);
        __builtin_amdgcn_wave_barrier();
        // conv + SiLU of two channels at kPos positions, weighted
        if (c == 0) {
#pragma unroll
            for (int q = 0; q < 3; q++)
                if (kPos * tg + q - 3 < 0) xraw[q] = 0u;
            if (a.dir > 0 && a.tail_in && tg == 0 && a.K > 1) {
                unsigned cached[3];
#pragma unroll
                for (int q = 0; q < 3; q++) {   // 3 - q tokens before the block (a tap beyond the conv width has a zero weight)
                    const T* tp = (const T*)a.tail_in + ((size_t)b * (a.K - 1) + max(a.K - 1 - (3 - q), 0)) * a.tail_ch + ch0 + 2 * cp;
                    cached[q] = (unsigned)tp[0] | ((unsigned)tp[1] << 16);
                }
                // (consumed here, so that no load is pending on xraw where the two paths join: the conv must not
                // wait for the younger B^T loads)
#pragma unroll
                for (int q = 0; q < 3; q++) asm volatile("" : "+v"(cached[q]));
#pragma unroll
                for (int q = 0; q < 3; q++)
                    if (3 - q <= a.K - 1) xraw[q] = cached[q];
            }
        }
        float wq[kPos];
#pragma unroll
        for (int q = 0; q < kPos; q += 4) {
            const float4 w = *reinterpret_cast<const float4*>(&wgt[kPos * tg + q]);
            wq[q] = w.x; wq[q + 1] = w.y; wq[q + 2] = w.z; wq[q + 3] = w.w;
        }
#pragma unroll
        for (int h2 = 0; h2 < 2; h2++) {
            typedef __attribute__((__vector_size__(kPos * sizeof(__bf16)))) __bf16 bf16run;
            float xr[kPos + 3];
#pragma unroll
            for (int q = 0; q < kPos + 3; q++) xr[q] = __uint_as_float(h2 == 0 ? xraw[q] << 16 : xraw[q] & 0xffff0000u);
            bf16run vw;
#pragma unroll
            for (int q = 0; q < kPos; q++) {
                float pre = cbias[h2];
                pre = fmaf(w4[h2][0], xr[q], pre);
                pre = fmaf(w4[h2][1], xr[q + 1], pre);
                pre = fmaf(w4[h2][2], xr[q + 2], pre);
                pre = fmaf(w4[h2][3], xr[q + 3], pre);
                vw[q] = (__bf16)(silu(pre) * wq[q]);
            }
            *reinterpret_cast<bf16run*>(&s_xw[buf][(2 * cp + h2) * kRowT + kPos * tg]) = vw;
        }
        lds_barrier();   // one per chunk: the other buffer is rewritten only after every wave has passed this one
        decay_product *= decay_q;
#pragma unroll
        for (int o = 0; o < kOwn; o++) {
            const int id = kOwn * wave + o, pblk = id % kPB;
            if (kBlocks % 4 == 0 || id < kBlocks) {
#pragma unroll
                for (int r = 0; r < 16; r++) hacc[o][r] *= decay_q;
#pragma unroll
                for (int kb = 0; kb < 4; kb++) {
                    const bf16x8 bw = *reinterpret_cast<const bf16x8*>(&s_xw[buf][(pblk * 32 + cl) * kRowT + 16 * kb + 8 * half]);
                    hacc[o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ab[kSameB ? 0 : o][kb], bw, hacc[o], 0, 0, 0);
                }
            }
        }
    }
    if (tid == 0) a.part_decay[((size_t)sub * batch + b) * a.H + head] = decay_product;
    float* const state_out = a.part_state + (size_t)sub * batch * a.Dn * N;
#pragma unroll
    for (int o = 0; o < kOwn; o++) {
        const int id = kOwn * wave + o, nblk = id / kPB, pblk = id % kPB;
        if (kBlocks % 4 == 0 || id < kBlocks) {
            // registers 4q .. 4q+3 hold four adjacent states of channel pblk*32 + cl
            float* hrow = state_out + ((size_t)b * a.Dn + ch0 + pblk * 32 + cl) * N + nblk * 32 + 4 * half;
#pragma unroll
            for (int q = 0; q < 4; q++)
                *reinterpret_cast<float4*>(hrow + 8 * q) =
                    make_float4(hacc[o][4 * q], hacc[o][4 * q + 1], hacc[o][4 * q + 2], hacc[o][4 * q + 3]);
        }
    }
}

}  // namespace bm
