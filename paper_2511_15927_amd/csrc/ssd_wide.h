// The chunk walk of ssd_kernels.h dealt to short instruction streams of up to sixteen waves.
//
// A wave issues at most one instruction every six to seven cycles whatever the instruction is, while a SIMD's vector
// ALU accepts a 64-lane instruction every four, so a workgroup is as fast as its longest instruction stream, not as its
// total work.  A workgroup walks the chunks of one head, or of two heads of a group in turn (HEADS = 2); a period is one
// (chunk, head), and its work is
//   y waves     (two sets of P/16): the intra-chunk product, the inter-chunk product C H and the epilogue of a 32 x 32 output
//               block each.  The sets take the periods in turn: a set runs a period's matrix products while its tiles are in
//               LDS and its epilogue (gate, combine, stores) a period later, while the other set multiplies;
//   state waves (4): the state update, whose B^T operand comes straight from global memory in operand order, the bf16 operand
//               copy of the new state, and the masked, decayed score operand of the next period.  Each of them scans every fourth
//               period's Delta, two periods ahead, for all waves;
//   conv waves  (4): conv + SiLU of x for the next period.
// One LDS barrier per period.
//
// What bounds it is the bytes a CU takes in: with all global accesses but the first ones removed a launch at batch 8 x 8192
// tokens of 64 heads x 64, 128 states takes 0.28 ms, with them 0.50 (reverse) and 0.69 (forward), and the tiles that every
// head of a group reads again (C 16 KB, B^T 16, scores 12 per chunk, all from L2) cost more than x, z and the output.  Hence two heads
// to a workgroup, which share them, where that leaves no CU idle: 0.43 and 0.51 ms.
//
// Layouts.  The y waves multiply with the 16x16x32 MFMA (operand A lane l: row l%16, eight contraction slots of group l/16;
// accumulator register r: row 4*(l/16) + r, column l%16): two row tiles by two column tiles, where column tile ct holds
// channels 2*(l%16) + ct, so that a lane owns adjacent channels and moves 4-byte pairs (of any alignment) of z, of the parked
// result and of the output.  The state update uses the 32x32x16 MFMA with the same channel order, column j = channel 2*(j%16) + j/16.
// Contraction over positions: slot 4t + e of group g is position 16t + 4g + e of a 32-position block, which makes a
// lane's own output rows its slots of the xc operand (the skip term reads no LDS).  Contraction over states: slot 4u + e of group
// g is state 16*(g%2) + 8u + 4*(g/2) + e of a 32-state block, the order in which the state's accumulators publish it.
//
// The result one direction parks for the other crosses global memory as bf16: in the paper's precision (bf16 autocast,
// App. A) each direction's output is a bf16 tensor before the two are added (eq. 6).  In time parts it stays fp32.
//
// grid (H / HEADS, directions * parts, batch).  Calls of several chunks; z / out token strides up to 2^24 elements but in the form for rows far apart.
#pragma once
#include "ssd_kernels.h"

namespace bm {

template <int N, int P, int HEADS>
struct SsdWide {
    static constexpr int kPB = P / 32, kNB = N / 32;
    static constexpr int kYWaves = 2 * kPB;                  // of one set
    static constexpr int kThreads = 64 * (2 * kYWaves + 8);
    // LDS: two buffers of xc, xw (operand order) and of the score operand, two of the state operand (the chunks of one head in
    // turn, or one for each of two heads), of C where two heads share it, four slots of tables
    static constexpr int kX = kQ * P, kM = 3 * 2 * 64 * 8, kTile = 2 * kX + kM, kHT = N * P;
    static constexpr int kTable = 4 * kQ + 4, kSlots = 4;    // e_i, f_j Delta_j, end-of-chunk weight, exp(l_i); separable flag
    static constexpr int kC = HEADS == 2 ? kQ * N : 0;
    static constexpr size_t bytes() { return 2 * (size_t)(kTile + kHT + kC) * sizeof(__bf16) + (size_t)kSlots * kTable * sizeof(float); }
};

// MODE: the output mode, compiled apart (the registers of one mode are not held through another's loop); kSsdFinalOnly walks
// both directions in one launch (see launch_ssd_scan), the others one.
// FORM: kSsdWhole: a workgroup walks an item's chunks.  kSsdParts: the launch deals them to several in scan order (blockIdx.y: the part,
// then the direction), each from the state that ssd_state_kernel and ssd_carry_kernel left for it, and what one direction parks for
// the other stays fp32.  kSsdFarParts: the same, one part or more, every row addressed by itself, for calls whose z or out rows lie
// too far apart for 32-bit offsets within a chunk.  (A form of its own: asked per chunk in the other, whether the offsets serve
// cost calls whose rows are near 1.6 %, 64 heads x 32, N 64, 1 x 16384 tokens.)
// kSsdMeet: calls that leave at least half of the CUs empty and have directions to add, in two launches of both directions.  In the
// first each walks the half of the chunks that it scans first, parks its results and leaves its state, in the second each takes the
// other half from there and adds what the other direction parked there.  The reverse direction's chunks start before the sequence
// where that is ragged, so that both directions' chunks hold the same tokens (positions that do not exist have Delta = 0 and are not
// stored).
// Against one walk of eight waves a part, calls of 64 heads x 64, N 128: 1 x 32768 tokens 953 -> 890 us, 1 x 8192 279 -> 255, 2 x 8192
// 476 -> 440, 1 x 2048 103 -> 90; 64 heads x 32, N 64, 1 x 16384 340 -> 258.
template <int N, int P, int HEADS, int MODE, int FORM>
__global__ __launch_bounds__((SsdWide<N, P, HEADS>::kThreads)) void ssd_wide_kernel(const std::conditional_t<(MODE > 0 && FORM != 3), SsdArgs, SsdStatePair> launch)
{
    constexpr bool kParts = FORM != kSsdWhole, kMeet = FORM == kSsdMeet;
    static_assert(kSsdMeet == 3);
    // (the parameter's type names no enumerator: those of an unnamed enumeration are spelt differently in a kernel's host and device name)
    static_assert(kSsdFinalOnly == 0);
    const SsdArgs& a = [&]() -> const SsdArgs& {
        if constexpr (kMeet) return launch.dir[blockIdx.y];
        else if constexpr (MODE != kSsdFinalOnly) return launch;
        else return launch.dir[kParts ? (int)blockIdx.y >= launch.dir[0].parts : blockIdx.y];
    }();
    using W = SsdWide<N, P, HEADS>;
    constexpr int kPB = W::kPB, kNB = W::kNB;
    using T = unsigned short;
    extern __shared__ __attribute__((aligned(16))) unsigned char ssd_lds[];
    __bf16* const tiles = reinterpret_cast<__bf16*>(ssd_lds);
    __bf16* const sHT = tiles + 2 * W::kTile;
    __bf16* const sC = sHT + 2 * W::kHT;
    float* const tables = reinterpret_cast<float*>(sC + 2 * W::kC);
    auto sXc = [&](int buf) { return tiles + buf * W::kTile; };
    auto sXw = [&](int buf) { return tiles + buf * W::kTile + W::kX; };
    auto sM = [&](int buf) { return tiles + buf * W::kTile + 2 * W::kX; };
    auto table = [&](int p) { return tables + (p & (W::kSlots - 1)) * W::kTable; };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups go to the 8 XCDs round-robin by linear id and each XCD has its own L2.  All heads of a batch element read the same
    // C / B^T / score tiles, so the (batch, head) items are dealt out such that an XCD receives a contiguous, batch-major run of
    // them and fetches each tile from HBM once instead of once per XCD.
    int head = blockIdx.x, b = blockIdx.z;
    {
        const unsigned total = gridDim.x * gridDim.z, id = blockIdx.x + gridDim.x * blockIdx.z;
        if (total % 8 == 0) {
            const unsigned item = (id % 8) * (total / 8) + id / 8;
            head = (int)(item % gridDim.x);
            b = (int)(item / gridDim.x);
        }
    }
    head *= HEADS;                          // the workgroup's first; two heads are of one group (the host checks)
    const int grp = head / a.HG;
    const int ch0 = head * P;
    // this workgroup's chunks [c0, c0 + nchunk), below by their place in it; period p: chunk p / HEADS, head p % HEADS
    const int part = !kParts || kMeet ? 0 : (int)blockIdx.y - ((int)blockIdx.y >= a.parts ? a.parts : 0);
    const int c0 = kMeet ? a.first_chunk : !kParts ? 0 : part * a.part_chunks;
    const int nchunk = kMeet ? a.part_chunks : !kParts ? a.nchunk : min(a.nchunk - c0, a.part_chunks), periods = nchunk * HEADS;
    const int q0 = c0 * kQ - (kMeet ? a.lead : 0);
    const float* const state_in = !kParts || kMeet ? a.h_in : a.part_state + (size_t)part * a.part_subs * gridDim.z * a.Dn * N;
    float* const state_out = !kParts || kMeet || part == a.parts - 1 ? a.h_out : nullptr;
    const int last = a.L - 1;
    auto token_of = [&](int tau) { return a.dir > 0 ? tau : last - tau; };
    // the prepared tiles of (chunk c, this group)
    auto tile_of = [&](int c) { return ((size_t)b * a.nchunk + c0 + c) * a.G + grp; };

    if (wave >= 2 * W::kYWaves + 4) {
        // ------------------------------------------------------------------ conv waves
        // (the conv and state waves' streams are what a period waits for: they go before the y waves on their SIMD)
        __builtin_amdgcn_s_setprio(1);
        constexpr int kCP = P / 2;                  // channel pairs of the head
        constexpr int kPos = kQ * kCP / 256;        // chunk positions per thread (8 or 4)
        const int ptid = tid - 64 * (2 * W::kYWaves + 4);
        const int cp = ptid % kCP, tg = ptid / kCP;
        float w4[HEADS][2][4], cbias[HEADS][2];
#pragma unroll
        for (int hd = 0; hd < HEADS; hd++)
#pragma unroll
            for (int h2 = 0; h2 < 2; h2++) {
                const int ch = ch0 + hd * P + 2 * cp + h2;
                load_taps(a.conv_w + (size_t)ch * a.K, a.K, w4[hd][h2]);
                cbias[hd][h2] = a.conv_b ? a.conv_b[ch] : 0.0f;
            }
        const T* xb = (const T*)a.x.p + (size_t)b * a.x.sb + ch0 + 2 * cp;
        const long long xstep = a.dir * a.x.st;
        const auto edge_chunk = [&](int c) { return (kMeet ? q0 + c * kQ < 3 : c0 + c == 0) || q0 + c * kQ + kQ - 1 > last; };
        unsigned xraw[2][kPos + 3];   // of the periods of either parity, requested two periods ahead
        auto issue_x = [&](int c, int hd, unsigned (&xraw)[kPos + 3]) {
            const int tau0 = q0 + c * kQ + kPos * tg - 3;
            const T* const xh = xb + hd * P;
            if (!edge_chunk(c)) {
                const T* xp = xh + (long long)token_of(tau0) * a.x.st;
#pragma unroll
                for (int q = 0; q < kPos + 3; q++) xraw[q] = *reinterpret_cast<const unsigned*>(xp + q * xstep);
            } else {
#pragma unroll
                for (int q = 0; q < kPos + 3; q++)
                    xraw[q] = *reinterpret_cast<const unsigned*>(xh + (long long)token_of(min(max(tau0 + q, 0), last)) * a.x.st);
            }
        };
        // this thread's pieces of the operand tiles (elements): its kPos positions of channels 2cp, 2cp + 1
        const int pblk = cp / 16, pos0 = kPos * tg;
        unsigned xc_at[kPos / 4], xw_at;
#pragma unroll
        for (int u = 0; u < kPos / 4; u++) {
            const int pos = pos0 + 4 * u;   // slot 4t of group g in 32-position block pos/32
            xc_at[u] = (unsigned)((((pos / 32) * kPB + pblk) * 2 * 64 + ((pos % 16) / 4) * 16 + cp % 16) * 8 + 4 * ((pos % 32) / 16));
        }
        xw_at = (unsigned)((((pos0 / 16) * kPB + pblk) * 64 + ((pos0 % 16) / 8) * 32 + cp % 16) * 8 + pos0 % 8);
        // conv + SiLU of period p (of parity odd) into its tile buffer; requests x of period p + 2 the moment its registers are free
        auto finish = [&](int p, auto odd_c) {
            constexpr int odd = decltype(odd_c)::value, hd = odd % HEADS;
            const int c = p / HEADS, cn = min((p + 2) / HEADS, nchunk - 1);
            unsigned(&xraw_p)[kPos + 3] = xraw[odd];
            float xr[2][kPos + 3];
#pragma unroll
            for (int q = 0; q < kPos + 3; q++) {
                xr[0][q] = __uint_as_float(xraw_p[q] << 16);
                xr[1][q] = __uint_as_float(xraw_p[q] & 0xffff0000u);
            }
            asm volatile("" ::: "memory");
            // (two heads' rows are neighbours in memory and are requested together: 0.5 % at 64 heads x 64)
            if constexpr (HEADS == 1) issue_x(cn, hd, xraw_p);
            else if constexpr (odd == 1) {
                issue_x(cn, 0, xraw[0]);
                issue_x(cn, 1, xraw[1]);
            }
            if (edge_chunk(c)) {
#pragma unroll
                for (int q = 0; q < kPos + 3; q++) {
                    const int tau = q0 + c * kQ + kPos * tg + q - 3;
                    if (tau < 0 || tau > last) xr[0][q] = xr[1][q] = 0.0f;
                }
                if (c0 + c == 0 && a.dir > 0 && a.tail_in && tg == 0 && a.K > 1) {
                    T cached[3][2];
#pragma unroll
                    for (int q = 0; q < 3; q++) {   // 3 - q tokens before the block; a tap beyond the conv width has a zero weight
                        const T* tp = (const T*)a.tail_in + ((size_t)b * (a.K - 1) + max(a.K - 1 - (3 - q), 0)) * a.tail_ch + ch0 + hd * P + 2 * cp;
                        cached[q][0] = tp[0];
                        cached[q][1] = tp[1];
                    }
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        if (3 - q <= a.K - 1) {
                            xr[0][q] = IoBF16::cvt(cached[q][0]);
                            xr[1][q] = IoBF16::cvt(cached[q][1]);
                        }
                    }
                }
            }
            const float* const wgt = table(p) + 2 * kQ + pos0;
            float wq[kPos];
#pragma unroll
            for (int q = 0; q < kPos; q += 4) {
                const float4 w = *reinterpret_cast<const float4*>(wgt + q);
                wq[q] = w.x; wq[q + 1] = w.y; wq[q + 2] = w.z; wq[q + 3] = w.w;
            }
            const int buf = p & 1;
#pragma unroll
            for (int h2 = 0; h2 < 2; h2++) {
                typedef __attribute__((__vector_size__(kPos * sizeof(__bf16)))) __bf16 bf16run;
                bf16run vw;
                bf16x4 vx[kPos / 4];
#pragma unroll
                for (int q = 0; q < kPos; q++) {
                    float pre = cbias[hd][h2];
                    pre = fmaf(w4[hd][h2][0], xr[h2][q], pre);
                    pre = fmaf(w4[hd][h2][1], xr[h2][q + 1], pre);
                    pre = fmaf(w4[hd][h2][2], xr[h2][q + 2], pre);
                    pre = fmaf(w4[hd][h2][3], xr[h2][q + 3], pre);
                    const float xc = silu(pre);
                    vx[q / 4][q % 4] = (__bf16)xc;
                    vw[q] = (__bf16)(xc * wq[q]);
                }
#pragma unroll
                for (int u = 0; u < kPos / 4; u++) *reinterpret_cast<bf16x4*>(&sXc(buf)[xc_at[u] + h2 * 64 * 8]) = vx[u];
                *reinterpret_cast<bf16run*>(&sXw(buf)[xw_at + h2 * 16 * 8]) = vw;
            }
        };
        // C of a chunk to LDS for two heads: requested two periods before it is written
        constexpr int kCopy = HEADS == 2 ? kQ * N / 8 / 256 : 1;
        bf16x8 ctile[kCopy];
        auto issue_c = [&](int c) {
            const bf16x8* src = reinterpret_cast<const bf16x8*>(a.c_rows + tile_of(c) * N * kQ) + ptid;
#pragma unroll
            for (int i = 0; i < kCopy; i++) ctile[i] = src[i * 256];
        };
        auto put_c = [&](int c) {
            bf16x8* dst = reinterpret_cast<bf16x8*>(sC + (c & 1) * W::kC) + ptid;
#pragma unroll
            for (int i = 0; i < kCopy; i++) dst[i * 256] = ctile[i];
        };
        using Even = std::integral_constant<int, 0>;
        using Odd = std::integral_constant<int, 1>;
        if constexpr (HEADS == 2) issue_c(0);
        issue_x(0, 0, xraw[0]);
        issue_x(min(1 / HEADS, nchunk - 1), HEADS - 1, xraw[1]);
        lds_barrier();   // the tables of the first two periods
        if constexpr (HEADS == 2) {
            put_c(0);
            asm volatile("" ::: "memory");
            issue_c(1);
        }
        finish(0, Even{});
        lds_barrier();
        for (int p = 0; p < periods; p += 2) {
            if constexpr (HEADS == 2) {
                const int c = p / 2;
                if (c + 1 < nchunk) {   // (the slot's last readers were in the period before this one)
                    put_c(c + 1);
                    asm volatile("" ::: "memory");
                    issue_c(min(c + 2, nchunk - 1));
                }
            }
            if (p + 1 < periods) finish(p + 1, Odd{});
            lds_barrier();
            if (HEADS == 1 && p + 1 >= periods) break;
            if (p + 2 < periods) finish(p + 2, Even{});
            lds_barrier();
        }
        return;
    }

    if (wave >= 2 * W::kYWaves) {
        // ------------------------------------------------------------------ state waves
        __builtin_amdgcn_s_setprio(1);
        constexpr int kBlocks = kNB * kPB, kOwn = (kBlocks + 3) / 4;   // 32 x 32 blocks of H; of one wave: one row of blocks
        const int sw = wave - 2 * W::kYWaves, ptid = tid - 64 * 2 * W::kYWaves;
        const bool owner = kOwn * sw < kBlocks;
        const int nblk = kOwn * sw / kPB, pblk0 = kOwn * sw % kPB;
        const int cl = lane & 31, half = lane >> 5;
        const int ch_of_lane = ch0 + 2 * (cl % 16) + cl / 16;          // + 32 per channel block
        // a wave scans every fourth period: always the same head's
        const int scan_head = head + sw % HEADS;
        const float a2 = a.A[scan_head] * kLog2e;
        const float dtb = (a.dt_softplus && a.dt_bias) ? a.dt_bias[scan_head] : 0.0f;
        const T* dtp = (const T*)a.dt.p + (size_t)b * a.dt.sb + scan_head;
        T dtraw;
        auto issue_dt = [&](int p) {
            const int tau = min(q0 + p / HEADS * kQ + lane, last);
            dtraw = dtp[(long long)token_of(kMeet ? max(tau, 0) : tau) * a.dt.st];
        };
        // A period's scan: Delta; the inclusive cumulative log2-decay; what the waves read of them.  With two heads a wave does these
        // in successive periods (whole, it lengthens one wave's stream in every period: 0.8 % at 8 x 8192 tokens); with one head's
        // shorter periods the branches cost more than that (2 % at 1 x 1024).
        float dl = 0.0f, l2 = 0.0f;
        auto scan_delta = [&](int p) {
            dl = IoBF16::cvt(dtraw);
            issue_dt(p + 4);   // (clamped to the sequence)
            if (a.dt_softplus) dl = softplus(dl + dtb);
            if (q0 + p / HEADS * kQ + lane > last || (kMeet && q0 + p / HEADS * kQ + lane < 0)) dl = 0.0f;
        };
        auto scan_decay = [&]() { l2 = wave_inclusive_sum(dl * a2); };
        auto scan_tables = [&](int p) {
            const float l2_end = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l2), 63));
            // separable decay exp(l_i - l_j) = e_i f_j around the chunk's middle unless the chunk decays too fast
            const float l2_first = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l2), 0));
            const float l2_mid = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l2), kQ / 2 - 1));
            const bool separable = l2_first - l2_end <= 100.0f;
            float* const t = table(p);
            t[lane] = separable ? fast_exp2(l2 - l2_mid) : l2;
            t[kQ + lane] = separable ? fast_exp2(l2_mid - l2) * dl : dl;
            t[2 * kQ + lane] = fast_exp2(l2_end - l2) * dl;
            t[3 * kQ + lane] = fast_exp2(l2);
            if (lane == 0) t[4 * kQ] = separable ? 1.0f : 0.0f;
        };
        float4 gt[3];
        auto issue_score = [&](int c, int m) {
            gt[m] = reinterpret_cast<const float4*>(a.score_op + tile_of(c) * kScoreOp)[m * 256 + ptid];
        };
        bf16x8 bt[4];
        auto issue_bt = [&](int c) {
            const bf16x8* src = reinterpret_cast<const bf16x8*>(a.b_t + tile_of(c) * N * kQ) + (owner ? nblk * 4 * 64 : 0) + lane;
#pragma unroll
            for (int kb = 0; kb < 4; kb++) bt[kb] = src[kb * 64];
        };
        // (B_j . C_i) exp(l_i - l_j) Delta_j of a period, for the blocks (i, j) = (0, 0), (1, 0), (1, 1) of 32 x 32: this
        // thread holds row i of four adjacent columns j in each.  The prepared scores are zero above the diagonal.
        const int i32 = (ptid / 128) * 16 + (ptid / 2) % 16, j32 = 16 * (ptid % 2) + 4 * ((ptid / 32) % 4);
        auto score = [&](int p, int cn) {   // cn: the chunk whose scores to request then, -1: they are needed again
            const float* const t = table(p);
            const bool separable = __builtin_amdgcn_readfirstlane(__float_as_int(t[4 * kQ])) != 0;
            const float li[2] = {t[i32], t[32 + i32]};
            // (block by block, each one's scores requested again as soon as they are used: the state leaves few registers)
#pragma unroll
            for (int m = 0; m < 3; m++) {
                const float4 d4 = *reinterpret_cast<const float4*>(t + kQ + 32 * (m > 1) + j32);
                const float dj[4] = {d4.x, d4.y, d4.z, d4.w}, sv[4] = {gt[m].x, gt[m].y, gt[m].z, gt[m].w};
                bf16x4 v;
                if (separable) {
#pragma unroll
                    for (int e = 0; e < 4; e++) v[e] = (__bf16)(sv[e] * li[m > 0] * dj[e]);
                } else {
                    const float4 l4 = *reinterpret_cast<const float4*>(t + 32 * (m > 1) + j32);
                    const float lj[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const float val = sv[e] * fast_exp2(li[m > 0] - lj[e]) * dj[e];
                        v[e] = (__bf16)((m != 1 && j32 + e > i32) ? 0.0f : val);
                    }
                }
                *reinterpret_cast<bf16x4*>(&sM(p & 1)[(m * 256 + ptid) * 4]) = v;
                asm volatile("" ::: "memory");
                if (cn >= 0) issue_score(cn, m);
            }
        };
        f32x16 hacc[HEADS][kOwn];
#pragma unroll
        for (int hd = 0; hd < HEADS; hd++)
#pragma unroll
            for (int o = 0; o < kOwn; o++) {
#pragma unroll
                for (int r = 0; r < 16; r++) hacc[hd][o][r] = 0.0f;
                if (state_in && owner) {   // registers 4q .. 4q+3: four adjacent states of the lane's channel
                    const float* hrow = state_in + ((size_t)b * a.Dn + ch_of_lane + hd * P + (pblk0 + o) * 32) * N + nblk * 32 + 4 * half;
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const float4 v = *reinterpret_cast<const float4*>(hrow + 8 * q);
                        hacc[hd][o][4 * q] = v.x; hacc[hd][o][4 * q + 1] = v.y; hacc[hd][o][4 * q + 2] = v.z; hacc[hd][o][4 * q + 3] = v.w;
                    }
                }
            }
        auto publish_state = [&](auto head_c, int which) {
            constexpr int hd = decltype(head_c)::value;
            if (!owner) return;
#pragma unroll
            for (int o = 0; o < kOwn; o++) {
#pragma unroll
                for (int u = 0; u < 2; u++) {
                    bf16x8 v;
#pragma unroll
                    for (int e = 0; e < 8; e++) v[e] = (__bf16)hacc[hd][o][8 * u + e];
                    *reinterpret_cast<bf16x8*>(&sHT[which * W::kHT + (((nblk * kPB + pblk0 + o) * 2 + cl / 16) * 64 + (2 * half + u) * 16 + cl % 16) * 8]) = v;
                }
            }
        };
        auto update = [&](auto head_c, int c) {
            constexpr int hd = decltype(head_c)::value;
            const int p = c * HEADS + hd;
            // the state after the last chunk matters only if it is committed
            if (!owner || (c + 1 >= nchunk && state_out == nullptr)) return;
            const float decay_q = table(p)[3 * kQ + kQ - 1];
            const bf16x8* xw = reinterpret_cast<const bf16x8*>(sXw(p & 1)) + lane;
#pragma unroll
            for (int o = 0; o < kOwn; o++)
#pragma unroll
                for (int r = 0; r < 16; r++) hacc[hd][o][r] *= decay_q;
#pragma unroll
            for (int kb = 0; kb < 4; kb++) {
                // (two heads' states leave no registers for operands that wait)
                if (HEADS == 2 && kb % 2 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int o = 0; o < kOwn; o++)
                    hacc[hd][o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bt[kb], xw[(kb * kPB + pblk0 + o) * 64], hacc[hd][o], 0, 0, 0);
            }
            if (HEADS == 2) __builtin_amdgcn_sched_barrier(0);
        };
        // tables of period p + 2 in period p, by wave (p + 2) % 4
        auto scan_ahead = [&](int p) {
            const int ahead = (sw - p) & 3;
            if constexpr (HEADS == 1) {
                if (ahead != 2) return;
                scan_delta(p + 2);
                scan_decay();
                scan_tables(p + 2);
            } else {
                if (ahead == 2) scan_tables(p + 2);
                else if (ahead == 3) scan_decay();
                else if (ahead == 0) scan_delta(p + 4);
            }
        };
        using Head0 = std::integral_constant<int, 0>;
        using Head1 = std::integral_constant<int, HEADS - 1>;
        issue_dt(sw);
#pragma unroll
        for (int m = 0; m < 3; m++) issue_score(0, m);
        issue_bt(0);
        if (HEADS == 2 || sw < 2) {
            scan_delta(sw);
            scan_decay();
        }
        if (sw < 2) scan_tables(sw);
        lds_barrier();   // the tables of the first two periods
        score(0, HEADS == 1 ? min(1, nchunk - 1) : -1);
        publish_state(Head0{}, 0);
        if constexpr (HEADS == 2) publish_state(Head1{}, 1);
        lds_barrier();
        for (int c = 0; c < nchunk; c++) {
            const int cn = min(c + 1, nchunk - 1);
            if constexpr (HEADS == 1) {
                scan_ahead(c);
                update(Head0{}, c);
                asm volatile("" ::: "memory");
                issue_bt(cn);
                if (c + 1 < nchunk) {
                    score(c + 1, min(c + 2, nchunk - 1));
                    publish_state(Head0{}, (c + 1) & 1);   // (the chunk's own copy is still being read)
                }
                lds_barrier();
            } else {
                // a head's new state is published in the other head's period, when nothing reads its copy
                scan_ahead(2 * c);
                if (c > 0) publish_state(Head1{}, 1);
                update(Head0{}, c);
                score(2 * c + 1, cn);
                lds_barrier();
                scan_ahead(2 * c + 1);
                publish_state(Head0{}, 0);
                update(Head1{}, c);
                asm volatile("" ::: "memory");
                issue_bt(cn);
                if (c + 1 < nchunk) score(2 * c + 2, -1);
                lds_barrier();
            }
        }
        if (state_out && owner) {
#pragma unroll
            for (int hd = 0; hd < HEADS; hd++)
#pragma unroll
                for (int o = 0; o < kOwn; o++) {
                    float* hrow = state_out + ((size_t)b * a.Dn + ch_of_lane + hd * P + (pblk0 + o) * 32) * N + nblk * 32 + 4 * half;
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        *reinterpret_cast<float4*>(hrow + 8 * q) =
                            make_float4(hacc[hd][o][4 * q], hacc[hd][o][4 * q + 1], hacc[hd][o][4 * q + 2], hacc[hd][o][4 * q + 3]);
                }
        }
        return;
    }

    // ---------------------------------------------------------------------- y waves: one 32 x 32 block of every other period's output
    constexpr bool need_z = MODE != kSsdPartialRaw;
    constexpr bool need_p = MODE == kSsdFinalAdd || MODE == kSsdFinalAddRaw;
    constexpr bool parks = MODE == kSsdPartialRaw || MODE == kSsdPartial;
    const int set = wave / W::kYWaves, iblk = (wave / kPB) % 2, pblk = wave % kPB;
    const int col = lane & 15, g4 = lane >> 4;
    const int po = pblk * 32 + 2 * col;        // this lane's channel pair
    const int i0 = iblk * 32 + 4 * g4;         // output row of row tile 0, register 0
    const int my_head = head + (HEADS == 2 ? set : 0), my_ch0 = my_head * P;
    const float dval[2] = {a.D[a.d_per_head ? my_head : my_ch0 + po], a.D[a.d_per_head ? my_head : my_ch0 + po + 1]};
    // rows of a chunk that lies inside the sequence, relative to the chunk's lowest-address token: row 16 rt + r of
    // the lane is group[rt] (in the lane offset) plus step[r] (a scalar offset): no vector address arithmetic
    const int fwd = a.dir > 0;
    const unsigned zs = (unsigned)a.z.st * 2u, os = (unsigned)a.out_st * 2u;
    using Park = std::conditional_t<kParts, float, T>;   // what one direction leaves for the other: bf16 where a call is walked whole
    const unsigned ps = (unsigned)a.Dn * (unsigned)sizeof(Park);
    unsigned zoff[2], ooff[2], poff[2];
#pragma unroll
    for (int rt = 0; rt < 2; rt++) {
        const unsigned rows = (unsigned)(fwd ? i0 + 16 * rt : kQ - 4 - i0 - 16 * rt);
        zoff[rt] = rows * zs + 2u * (unsigned)po;
        ooff[rt] = rows * os + 2u * (unsigned)po;
        poff[rt] = rows * ps + (unsigned)sizeof(Park) * (unsigned)po;
    }
    // (scalar registers by construction: left to the compiler the direction select lands in vector registers and
    // every access loops over the lanes to read its offset back)
    int zstep[4], ostep[4], pstep[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int m = fwd ? e : 3 - e;
        zstep[e] = __builtin_amdgcn_readfirstlane(m * (int)zs);
        ostep[e] = __builtin_amdgcn_readfirstlane(m * (int)os);
        pstep[e] = __builtin_amdgcn_readfirstlane(m * (int)ps);
    }
    const T* const zhead = (const T*)a.z.p + (size_t)b * a.z.sb + my_ch0;
    Park* const phead = (Park*)a.partial + (size_t)b * a.L * a.Dn + my_ch0;
    T* const ohead = (T*)a.out + (size_t)b * a.out_sb + a.out_ch_off + my_ch0;
    auto chunk_low_token = [&](int c) { return (long long)(fwd ? q0 + c * kQ : last - (q0 + c * kQ + kQ - 1)); };
    auto inside = [&](int c) { return FORM != kSsdFarParts && q0 + c * kQ + kQ - 1 <= last && (!kMeet || q0 + c * kQ >= 0); };
    auto token_at = [&](int c, int k) {
        const int tau = min(q0 + c * kQ + i0 + 16 * (k / 4) + k % 4, last);
        return (long long)token_of(kMeet ? max(tau, 0) : tau);
    };

    typedef unsigned __attribute__((ext_vector_type(2))) uint2v;
    using ParkPair = std::conditional_t<kParts, uint2v, unsigned>;
    unsigned zraw[8];   // register k: row 16 (k / 4) + k % 4 of the lane, a channel pair
    ParkPair praw[8];
    auto issue_z = [&](int c) {
        if constexpr (!need_z) return;
        if (inside(c)) {
            const Rsrc zr = raw_range(zhead + chunk_low_token(c) * a.z.st);
#pragma unroll
            for (int k = 0; k < 8; k++) zraw[k] = __builtin_amdgcn_raw_buffer_load_b32(zr, zoff[k / 4], zstep[k % 4], 0);
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const T* zp = zhead + token_at(c, k) * a.z.st + po;
                zraw[k] = *reinterpret_cast<const bf16_pair*>(zp);
            }
        }
    };
    auto issue_p = [&](int c) {
        if constexpr (!need_p) return;
        if (inside(c)) {
            const Rsrc pr = raw_range(phead + chunk_low_token(c) * a.Dn);
#pragma unroll
            for (int k = 0; k < 8; k++) {
                if constexpr (kParts) praw[k] = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(pr, poff[k / 4], pstep[k % 4], 0));
                else praw[k] = __builtin_amdgcn_raw_buffer_load_b32(pr, poff[k / 4], pstep[k % 4], 0);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++) praw[k] = *reinterpret_cast<const ParkPair*>(phead + token_at(c, k) * a.Dn + po);
        }
    };
    bf16x8 cf[HEADS == 1 ? kNB : 1][2];   // one head: C operand straight from global memory, [32 states][row tile]
    auto issue_c = [&](int c) {
        if constexpr (HEADS == 2) return;
        const bf16x8* src = reinterpret_cast<const bf16x8*>(a.c_rows + tile_of(c) * N * kQ) + iblk * 2 * kNB * 64 + lane;
#pragma unroll
        for (int nb = 0; nb < kNB; nb++)
#pragma unroll
            for (int rt = 0; rt < 2; rt++) cf[HEADS == 1 ? nb : 0][rt] = src[(rt * kNB + nb) * 64];
    };
    auto lo = [](unsigned v) { return __uint_as_float(v << 16); };
    auto hi = [](unsigned v) { return __uint_as_float(v & 0xffff0000u); };

    const int mine = HEADS == 2 ? 0 : min(set, nchunk - 1);
    issue_c(mine);
    issue_z(mine);
    issue_p(mine);
    lds_barrier();
    lds_barrier();
    if (set == 1) lds_barrier();   // period 0 belongs to the other set
    const int buf = set;           // of the set's tiles and of its state operand
    for (int p = set; p < periods; p += 2) {
        const int c = p / HEADS, cn = p + 2 < periods ? (p + 2) / HEADS : c;
        f32x4 y1[2][2], y2[2][2];
#pragma unroll
        for (int rt = 0; rt < 2; rt++)
#pragma unroll
            for (int ct = 0; ct < 2; ct++) y1[rt][ct] = y2[rt][ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (c > 0 || state_in != nullptr) {
            const bf16x8* c_t = reinterpret_cast<const bf16x8*>(sC + (c & 1) * W::kC) + iblk * 2 * kNB * 64 + lane;
            const bf16x8* h_t = reinterpret_cast<const bf16x8*>(sHT + buf * W::kHT) + pblk * 2 * 64 + lane;
#pragma unroll
            for (int nb = 0; nb < kNB; nb++)
#pragma unroll
                for (int ct = 0; ct < 2; ct++) {
                    const bf16x8 bh = h_t[(nb * kPB * 2 + ct) * 64];
#pragma unroll
                    for (int rt = 0; rt < 2; rt++) {
                        const bf16x8 ac = HEADS == 1 ? cf[HEADS == 1 ? nb : 0][rt] : c_t[(rt * kNB + nb) * 64];
                        y2[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ac, bh, y2[rt][ct], 0, 0, 0);
                    }
                }
        }
        bf16x8 bx[2];        // after the loop: the diagonal block's
#pragma unroll
        for (int jblk = 0; jblk < 2; jblk++) {
            if (jblk > iblk) break;
            const bf16x8* m_t = reinterpret_cast<const bf16x8*>(sM(buf)) + (iblk + jblk) * 2 * 64 + lane;
            const bf16x8* x_t = reinterpret_cast<const bf16x8*>(sXc(buf)) + (jblk * kPB + pblk) * 2 * 64 + lane;
            bf16x8 am[2];
#pragma unroll
            for (int k = 0; k < 2; k++) { am[k] = m_t[k * 64]; bx[k] = x_t[k * 64]; }
#pragma unroll
            for (int rt = 0; rt < 2; rt++)
#pragma unroll
                for (int ct = 0; ct < 2; ct++) y1[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[rt], bx[ct], y1[rt][ct], 0, 0, 0);
        }
        asm volatile("" ::: "memory");
        issue_c(cn);
        // inter-chunk and skip term
        float y[8][2];
        const float* const e_l = table(p) + 3 * kQ + i0;
#pragma unroll
        for (int rt = 0; rt < 2; rt++) {
            const float4 v = *reinterpret_cast<const float4*>(e_l + 16 * rt);
            const float el[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int r = 0; r < 4; r++)
#pragma unroll
                for (int ct = 0; ct < 2; ct++)
                    y[4 * rt + r][ct] = y1[rt][ct][r] + el[r] * y2[rt][ct][r] + dval[ct] * (float)bx[ct][4 * rt + r];
        }
        lds_barrier();
        // epilogue: gate, combine, round, a channel pair at a time
        using Result = std::conditional_t<parks, ParkPair, unsigned>;
        Result res[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            float v[2];
#pragma unroll
            for (int ct = 0; ct < 2; ct++) {
                float pv = 0.0f;
                if constexpr (need_p && kParts) pv = __uint_as_float(praw[k][ct]);
                else if constexpr (need_p) pv = ct == 0 ? lo(praw[k]) : hi(praw[k]);
                if constexpr (!need_z) v[ct] = y[k][ct];
                else {
                    const float zg = silu(ct == 0 ? lo(zraw[k]) : hi(zraw[k]));
                    v[ct] = MODE == kSsdFinalAddRaw ? (y[k][ct] + pv) * zg : need_p ? y[k][ct] * zg + pv : y[k][ct] * zg;
                }
            }
            if constexpr (parks && kParts) {
                res[k] = Result{__float_as_uint(v[0]), __float_as_uint(v[1])};
            } else {
                const bf16x2 pair = {(__bf16)v[0], (__bf16)v[1]};
                res[k] = __builtin_bit_cast(unsigned, pair);
            }
        }
        if (inside(c)) {
            const long long t0 = chunk_low_token(c);
            const Rsrc orr = raw_range(parks ? (const void*)(phead + t0 * a.Dn) : (const void*)(ohead + t0 * a.out_st));
#pragma unroll
            for (int k = 0; k < 8; k++) {
                if constexpr (parks && kParts) __builtin_amdgcn_raw_buffer_store_b64(res[k], orr, poff[k / 4], pstep[k % 4], 0);
                else if constexpr (parks) __builtin_amdgcn_raw_buffer_store_b32(res[k], orr, poff[k / 4], pstep[k % 4], 0);
                else __builtin_amdgcn_raw_buffer_store_b32(res[k], orr, ooff[k / 4], ostep[k % 4], 0);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const int tau = q0 + c * kQ + i0 + 16 * (k / 4) + k % 4;
                if (tau <= last && (!kMeet || tau >= 0)) {
                    const long long t = token_of(tau);
                    if constexpr (parks) *reinterpret_cast<Result*>(phead + t * a.Dn + po) = res[k];
                    else {
                        T* const o = ohead + t * a.out_st + po;
                        *reinterpret_cast<bf16_pair*>(o) = res[k];
                    }
                }
            }
        }
        issue_z(cn);
        issue_p(cn);
        if (p + 1 < periods) lds_barrier();   // (the other set's period)
    }
}

}  // namespace bm
